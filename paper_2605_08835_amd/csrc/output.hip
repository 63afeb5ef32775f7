// The step's last stage in one kernel (bf16 path): the UNet's output
// convolution (3x3, zero padding 1, C -> 4 channels) for a request's
// conditional and, under CFG, unconditional row, the classifier-free
// guidance combine eps = eps_u + w (eps_c - eps_u) (eps = eps_c under
// Skip-CFG, whose unconditional branch is bypassed: Sec. II-B, Sec. III-B)
// and the DDIM update x' = A x + B eps (eta = 0), all in registers.  The
// per-row eps never reaches memory.
//
// The convolution is computed per input pixel rather than per output pixel:
// for every pixel p of the block's tile (plus one image row and one pixel of
// halo on either side) the MFMAs form the 36 partial products
//     Y[p][tap][o] = sum_c x[p][c] w[o][tap][c]      (tap = 3 ky + kx)
// with the pixel's channels read once.  The
// output pixel then sums its 9 taps from LDS,
//     eps[p][o] = b[o] + sum over in-image taps of Y[p + (ky-1) W + (kx-1)][tap][o],
// so the zero padding is the taps that are skipped, and the K reduction over
// channels happens across the lanes of each MFMA.
//
// MFMA v_mfma_f32_16x16x32_bf16 with the weights as the first operand (16
// of the 36 (tap, o) columns per tile, 3 tiles, zero rows past 36) and 16
// pixels as the second; step s takes channels 32 s .. 32 s + 31, eight to a
// lane group g = lane / 16, so a load reads 64 contiguous bytes of each pixel.
// (With a contiguous quarter of the channels per group, a load touched 64
// cache lines, and the 40 KB that four waves had in flight passed through the
// 32 KB of L1 several times: 32 guided requests 56.1
// us, now 40.2.)  The weights of a lane stay in registers
// for the whole block.
#include "device_common.h"
#include "kernels.h"

namespace sd {

// WIDE: 8 waves, four on each of a request's two rows at the same time, each
// row with its own Y; threads 0..255 gather the conditional, 256..511 the
// unconditional eps.  Under Skip-CFG all eight take the only row where a block
// has 64 pixels, else four (the others' weight loads cost more than their tiles
// save: 10 requests of 64x64 15.3 us with eight, 14.6 with four).
// Not WIDE: 4 waves, one row after the other, two blocks per CU.  a.P output
// pixels per block.
template <int S, bool WIDE>  // S = C / 32 MFMA steps over the channels
__global__ __launch_bounds__(WIDE ? 512 : 256, WIDE ? 1 : 2) void out_cfg_ddim_kernel(OutArgs a) {
  extern __shared__ __attribute__((aligned(16))) float Ys[];  // (two of) [pixel - q0][9 taps][4], eps_u
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, pl = lane & 15;
  const int W = a.W, HW = a.H * a.W, C = a.C;
  const int ri = blockIdx.x / a.tiles, tile = blockIdx.x - ri * a.tiles;
  const int r = a.order ? a.order[ri] : ri;
  const int ru = a.req_row_u[r];
  const int p0 = tile * a.P, p1 = min(HW, p0 + a.P);
  const int q0 = max(0, p0 - W - 1), q1 = min(HW, p1 + W + 1);

  // what the last lines need is read first
  const int p = p0 + (tid & 255);
  const float A = a.req_coef[3 * r], B = a.req_coef[3 * r + 1], w = a.req_coef[3 * r + 2];
  float lat[4], bias[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    bias[c] = a.bias[c];
    lat[c] = p < p1 ? a.lat_in[((long)r * 4 + c) * HW + p] : 0.f;
  }
  const int nw1 = WIDE && a.P < 128 ? 8 : 4;  // waves on the only row of a request
  const bool idle = WIDE && ru < 0 && wave >= nw1;
  // weight fragments: tile t, row pl is column j = 16 t + pl = (tap j / 4, output j % 4)
  bf16x8 wf[3][S];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int j = 16 * t + pl, tap = j >> 2, o = j & 3;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      bf16x8 v = {};
      if (j < 36 && !idle) v = *reinterpret_cast<const bf16x8*>(a.w + (long)o * 9 * C + tap * C + 32 * s + 8 * g);
      wf[t][s] = v;
    }
  }

  // Y over pixels [q0, q1) of one row: 16-pixel tiles dealt round-robin to
  // the waves, the next tile's loads issued before the current one's MFMAs.
  auto compute_y = [&](int row, float* Y, int w0, int nw) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(a.x + (long)row * HW * C, (long)HW * C * 2);
    const int ntile = (q1 - q0 + 15) >> 4;
    bf16x8 cur[S], nxt[S];
    auto fetch = [&](int tt, bf16x8(&v)[S]) {
      const int px = q0 + 16 * tt + pl;
      const bool ok = px < q1;
      const int off = (px * C + 8 * g) * 2;
#pragma unroll
      for (int s = 0; s < S; ++s) v[s] = buf_load16(rs, ok ? off + 64 * s : OOB);
    };
    if (w0 < ntile) fetch(w0, cur);
    for (int tt = w0; tt < ntile; tt += nw) {
      if (tt + nw < ntile) fetch(tt + nw, nxt);
      f32x4 acc[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int t = 0; t < 3; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[t][s], cur[s], acc[t], 0, 0, 0);
      // lane (g, pl) holds rows 4 g .. 4 g + 3 of each tile = tap 4 t + g, outputs 0..3, of pixel pl
      const int px = q0 + 16 * tt + pl;
      if (px < q1) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
          if (4 * t + g < 9)
            *reinterpret_cast<f32x4*>(&Y[(px - q0) * 36 + (4 * t + g) * 4]) = acc[t];
      }
#pragma unroll
      for (int s = 0; s < S; ++s) cur[s] = nxt[s];
    }
  };
  // eps of this thread's output pixel: bias plus its in-image taps
  auto gather = [&](const float* Y, float e[4]) {
#pragma unroll
    for (int o = 0; o < 4; ++o) e[o] = bias[o];
    if (p >= p1) return;
    const int y = p / W, x = p - y * W;
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const int yy = y + ky - 1;
      if (yy < 0 || yy >= a.H) continue;
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) {
        const int xx = x + kx - 1;
        if (xx < 0 || xx >= W) continue;
        const f32x4 v = *reinterpret_cast<const f32x4*>(&Y[(p + (ky - 1) * W + (kx - 1) - q0) * 36 + (3 * ky + kx) * 4]);
#pragma unroll
        for (int o = 0; o < 4; ++o) e[o] += v[o];
      }
    }
  };

  float ec[4], eu[4];
  if constexpr (WIDE) {
    const int ylen = (a.P + 2 * W + 2) * 36, half = wave >> 2;
    float* E = Ys + 2 * ylen;  // eps_u of the block's pixels
    if (ru >= 0)
      compute_y(half ? ru : r, Ys + half * ylen, wave & 3, 4);
    else if (!idle)
      compute_y(r, Ys, wave, nw1);
    __syncthreads();
    if (half == 0) {
      gather(Ys, ec);
    } else if (ru >= 0) {
      gather(Ys + ylen, eu);
      *reinterpret_cast<f32x4*>(&E[(tid & 255) * 4]) = f32x4{eu[0], eu[1], eu[2], eu[3]};
    }
    __syncthreads();
    if (half) return;
    if (ru >= 0) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&E[tid * 4]);
#pragma unroll
      for (int o = 0; o < 4; ++o) eu[o] = v[o];
    }
  } else {
    compute_y(r, Ys, wave, 4);
    __syncthreads();
    gather(Ys, ec);
    if (ru >= 0) {
      __syncthreads();  // every thread has read the conditional row's Y
      compute_y(ru, Ys, wave, 4);
      __syncthreads();
      gather(Ys, eu);
    }
  }
  if (p < p1) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float e = ec[c];
      if (ru >= 0) e = eu[c] + w * (e - eu[c]);
      const long o = ((long)r * 4 + c) * HW + p;
      a.lat_out[o] = A * lat[c] + B * e;
      if (a.eps_out) a.eps_out[o] = e;
    }
  }
}

bool out_cfg_ddim_ok(DType dt, int latent_c, int H, int W, int C) {
  return dt == BF16 && latent_c == 4 && H >= 1 && W >= 1 && W <= 128 && C >= 32 && C <= 320 && C % 32 == 0 &&
         (long)H * W * C * 2 < (1L << 31);
}

template <int S, bool WIDE>
static hipError_t launch_out_k(const OutArgs& a, unsigned blocks, hipStream_t s) {
  const size_t y = (size_t)(a.P + 2 * a.W + 2) * 36 * sizeof(float);
  const size_t lds = WIDE ? 2 * y + 256 * 4 * sizeof(float) : y;  // at most 152 KB (P 256, W 128)
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&out_cfg_ddim_kernel<S, WIDE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  out_cfg_ddim_kernel<S, WIDE><<<blocks, WIDE ? 512 : 256, lds, s>>>(a);
  return hipGetLastError();
}

// Blocks of 256 pixels, two per CU, once there are more of them than CUs; up to
// that many take the 8-wave form (one block per CU), with 128 or 64 pixels
// where that still leaves at most a block per CU (the halo of 2 W + 2 pixels is
// recomputed per block).  The pixels per block do not enter the arithmetic.
// 64x64x320, guided: one request 22.3 us with 256 pixels, 15.9 with 64; eight
// 23.0 with 256, 20.0 with 128; sixteen (256 blocks) 26.2 with 4 waves, 25.4
// with 8; past 256 blocks the 8-wave form needs a second round: 20 requests
// 45.1 us with 8 waves, 36.0 with 4; without guidance 29.2 and 22.4; at 64
// channels 13.6 and 10.9.
template <int S>
static hipError_t launch_out_s(OutArgs a, hipStream_t s) {
  const int HW = a.H * a.W;
  auto blocks = [&](int P) { return (long)a.n_req * ((HW + P - 1) / P); };
  const bool wide = blocks(256) <= 256;
  a.P = !wide ? 256 : (blocks(64) <= 256 ? 64 : (blocks(128) <= 256 ? 128 : 256));
  a.tiles = (HW + a.P - 1) / a.P;
  if (blocks(a.P) > 0x7FFFFFFFL) return hipErrorInvalidValue;
  return wide ? launch_out_k<S, true>(a, (unsigned)blocks(a.P), s) : launch_out_k<S, false>(a, (unsigned)blocks(a.P), s);
}

hipError_t launch_out_cfg_ddim(const OutArgs& args, hipStream_t s) {
  OutArgs a = args;
  if (!out_cfg_ddim_ok(BF16, 4, a.H, a.W, a.C) || a.n_req < 0) return hipErrorInvalidValue;
  if (a.n_req == 0) return hipSuccess;
  switch (a.C / 32) {
    case 1: return launch_out_s<1>(a, s);
    case 2: return launch_out_s<2>(a, s);
    case 3: return launch_out_s<3>(a, s);
    case 4: return launch_out_s<4>(a, s);
    case 5: return launch_out_s<5>(a, s);
    case 6: return launch_out_s<6>(a, s);
    case 7: return launch_out_s<7>(a, s);
    case 8: return launch_out_s<8>(a, s);
    case 9: return launch_out_s<9>(a, s);
    case 10: return launch_out_s<10>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sd
