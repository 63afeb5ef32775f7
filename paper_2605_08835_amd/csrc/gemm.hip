// Implicit-GEMM convolution / linear layers.
//
// C[M, N] = A[M, K] * B[K, N] where A is generated on the fly from NHWC
// activations (3x3 / 1x1 taps, stride 2, nearest-2x upsampling, two-source
// channel concat, fused GroupNorm affine + SiLU) and B is the packed weight
// matrix stored N-major with K contiguous.  bf16 runs on MFMA
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation); fp32 on v_mfma_f32_16x16x4_f32
// (true fp32, no reduced-precision products).
#include "device_common.h"
#include "kernels.h"

namespace sd {

struct RowPos {
  int img, oy, ox;
  bool ok;
};

__device__ inline RowPos decode_row(const ASeg& s, int m, int M) {
  RowPos r;
  r.ok = m < M;
  const int hw = s.Ho * s.Wo;
  const int mm = r.ok ? m : 0;
  r.img = mm / hw;
  const int p = mm - r.img * hw;
  r.oy = p / s.Wo;
  r.ox = p - r.oy * s.Wo;
  return r;
}

// Address of the 8-channel chunk (tap, c) of output pixel r, or null when
// the tap falls into the zero padding.
template <typename T>
__device__ inline const T* a_chunk_ptr(const ASeg& s, const RowPos& r, int tap, int c) {
  int ky = 1, kx = 1;
  if (s.ks == 3) {
    ky = tap / 3;
    kx = tap - ky * 3;
  }
  int iy = r.oy * s.stride + ky - 1, ix = r.ox * s.stride + kx - 1;
  const int Hs = s.up ? 2 * s.Hi : s.Hi, Ws = s.up ? 2 * s.Wi : s.Wi;
  if (!r.ok || iy < 0 || ix < 0 || iy >= Hs || ix >= Ws) return nullptr;
  if (s.up) {
    iy >>= 1;
    ix >>= 1;
  }
  const long pix = ((long)r.img * s.Hi + iy) * s.Wi + ix;
  if (c < s.c0) return reinterpret_cast<const T*>(s.src0) + pix * s.c0 + c;
  return reinterpret_cast<const T*>(s.src1) + pix * s.c1 + (c - s.c0);
}

// bf16 chunk: raw 16-byte copy when no transform applies.
__device__ inline bf16x8 a_chunk_bf16(const ASeg& s, const RowPos& r, int tap, int c) {
  bf16x8 z = {};
  const bf16* p = a_chunk_ptr<bf16>(s, r, tap, c);
  if (!p) return z;
  bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
  if (s.scale) {
    float sc[8], sh[8];
    load8f(s.scale + (long)r.img * s.cin + c, sc);
    load8f(s.shift + (long)r.img * s.cin + c, sh);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float f = (float)v[i] * sc[i] + sh[i];
      if (s.silu) f = silu_f(f);
      v[i] = (bf16)f;
    }
  }
  return v;
}

// Output row of GEMM row m (the upsample phases write every other pixel of
// every other image row).
__device__ inline long out_row(const Epi& e, int m) {
  if (!e.phase) return m;
  const int hw = e.ph_h * e.ph_w, img = m / hw, p = m - img * hw, y = p / e.ph_w, x = p - y * e.ph_w;
  const int py = (e.phase - 1) >> 1, px = (e.phase - 1) & 1;
  return (long)img * 4 * hw + (long)(2 * y + py) * (2 * e.ph_w) + 2 * x + px;
}

// Four consecutive output channels n..n+3 of row m (n % 4 == 0, N % 4 == 0).
template <typename T>
__device__ inline void store4(const Epi& e, int m, int n, const float x[4]) {
  const long r = out_row(e, m);
  if (e.out_f32) {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(e.out) + r * e.ldo + n) =
        make_float4(x[0], x[1], x[2], x[3]);
  } else {
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (bf16)x[i];
    *reinterpret_cast<bf16x4*>(reinterpret_cast<T*>(e.out) + r * e.ldo + n) = o;
  }
}

// Row scale (a folded LayerNorm's rstd); rows at or past M read nothing.
__device__ inline float row_scale(const Epi& e, int m, int M) {
  return (e.rowscale && m < M) ? e.rowscale[m] : 1.0f;
}

template <typename T>
__device__ inline void epilogue4(const Epi& e, int m, int n, float x[4]) {
  if (e.rowscale) {
    const float rs = e.rowscale[m];
    x[0] *= rs; x[1] *= rs; x[2] *= rs; x[3] *= rs;
  }
  if (e.bias) {
    const float4 b = *reinterpret_cast<const float4*>(e.bias + n);
    x[0] += b.x; x[1] += b.y; x[2] += b.z; x[3] += b.w;
  }
  if (e.tbias) {
    const float4 b = *reinterpret_cast<const float4*>(e.tbias + (long)(m / e.hw) * e.tb_ld + e.tb_off + n);
    x[0] += b.x; x[1] += b.y; x[2] += b.z; x[3] += b.w;
  }
  if (e.resid) {
    const bf16x4 r = *reinterpret_cast<const bf16x4*>(reinterpret_cast<const T*>(e.resid) + (long)m * e.ldr + n);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] += (float)r[i];
  }
  if (n < e.qcols) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] *= e.qscale;
  }
  store4<T>(e, m, n, x);
}

// ---------------------------------------------------------------- bf16 MFMA
// Block tile BM x BN x 64, 256 threads = WM x WN waves, each wave a
// (BM/WM) x (BN/WN) sub-tile of 32x32 MFMA accumulators.  Double-buffered
// LDS (one barrier per K step) with the next K tile prefetched into
// registers while the current one feeds the MFMAs.  Rows of both tiles are
// padded by 16 bytes so the 16-byte fragment reads of 8 consecutive rows hit
// distinct banks.  Blocks are renumbered so that the tiles sharing one A
// row band run on the same XCD (blocks are dealt round-robin over 8 XCDs).
template <int V>
struct IC {
  static constexpr int value = V;
};
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IC<I>{});
    static_for<I + 1, N>(f);
  }
}

// The MFMAs compute C^T tiles (weights as the first operand), so element r
// of lane l is (output channel 8*(r/4) + 4*(l/32) + r%4, pixel l%32): each
// lane owns runs of 4 consecutive channels of one pixel and stores them with
// one 8-byte (bf16) or 16-byte (fp32) write.  Tiles are visited with
// compile-time indices so the accumulators stay in registers.
template <int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void epilogue_tiles(const GemmArgs& a, const f32x16 (&acc)[TM][TN], int m0, int n0,
                                               int wm, int wn, int lane) {
  const int lr = lane & 31, hq = 4 * (lane >> 5);
  static_for<0, TM>([&](auto I) {
    static_for<0, TN>([&](auto J) {
      const f32x16 v = acc[I.value][J.value];
      const int m = m0 + wm * (BM / WM) + I.value * 32 + lr;
      const int nt = n0 + wn * (BN / WN) + J.value * 32;
      if (m < a.M) {
        if (a.epi.geglu) {
          // packed columns 32t + u (a) and 32t + 16 + u (gate) -> channel 16t + u
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int n = nt + 8 * q + hq;
            if (n < a.N) {
              float x[4], g[4];
              const float rs = row_scale(a.epi, m, a.M);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                x[e] = fmaf(v[4 * q + e], rs, a.epi.bias[n + e]);
                g[e] = fmaf(v[4 * (q + 2) + e], rs, a.epi.bias[n + 16 + e]);
                x[e] *= gelu_as(g[e]);
              }
              store4<bf16>(a.epi, m, nt / 2 + 8 * q + hq, x);
            }
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = nt + 8 * q + hq;
            if (n < a.N) {
              float x[4] = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
              if (a.epi.vt_out && n >= a.epi.vt_col0) {
                // transposed store: lanes l and l+1 hold consecutive tokens
                const float rs = row_scale(a.epi, m, a.M);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] *= rs;
                const int img = m / a.epi.vt_hw, tok = m - img * a.epi.vt_hw;
                bf16* o = reinterpret_cast<bf16*>(a.epi.vt_out) + (long)img * a.epi.vt_img +
                          (long)(n - a.epi.vt_col0) * a.epi.vt_ld + tok;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[(long)e * a.epi.vt_ld] = (bf16)x[e];
              } else {
                epilogue4<bf16>(a.epi, m, n, x);
              }
            }
          }
        }
      }
    });
  });
}

// Epilogue through LDS for bf16 outputs with no transposed part: each wave
// finishes its values in registers (bias, time bias, GEGLU, residual, query
// scale), writes 32 rows of its tile as bf16 into a private LDS region, then
// stores them back row-contiguous, 16 bytes per lane, so a wave writes whole
// runs instead of 32 scattered 8-byte pieces.  A residual is first copied
// into the same region row-contiguous, and each lane picks up its own
// elements there before overwriting them with the result (one rounding).
// Row stride of the region: the wave's columns plus 8 (16 bytes), which
// keeps rows 16-byte aligned and the 8-byte writes of 32 consecutive rows at
// most two to a bank.
template <int OW>
constexpr int STAGED_LD = OW + 8;

template <int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void epilogue_staged(const GemmArgs& a, const f32x16 (&acc)[TM][TN], int m0, int n0,
                                                int wm, int wn, int lane, bf16* R) {
  constexpr int WC = BN / WN;  // the wave's accumulator columns
  constexpr int LD = STAGED_LD<WC>;
  const Epi& e = a.epi;
  const bool geglu = e.geglu;
  const int OW = geglu ? WC / 2 : WC;  // output columns of the wave
  const int ncol0 = (geglu ? n0 / 2 : n0) + wn * OW;
  const int lr = lane & 31, hq = 4 * (lane >> 5);
  const bf16* resid = reinterpret_cast<const bf16*>(e.resid);
  // Residual rows (never with GEGLU, so a row has WC / 8 chunks): every load
  // of a 32-row group is issued before the first is used, and the next
  // group's loads are in flight while this group is stored, so the epilogue
  // waits for memory about once instead of once per chunk.
  constexpr int RCH = WC / 8, RPL = 32 * RCH / 64;
  static_assert((32 * RCH) % 64 == 0, "residual chunks spread evenly over the lanes");
  bf16x8 rres[RPL];
  auto load_resid = [&](int mrow0) {
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      const int c = lane + 64 * u, row = c / RCH, ch = c - row * RCH;
      const int m = mrow0 + row;
      bf16x8 r = {};
      if (m < a.M) r = *reinterpret_cast<const bf16x8*>(resid + (long)m * e.ldr + ncol0 + ch * 8);
      rres[u] = r;
    }
  };
  if (resid) load_resid(m0 + wm * (BM / WM));
  // The bias of the columns the lane finishes in 32-column tile J (columns
  // nt + 8 q + hq + [0, 4); with GEGLU q = 0, 1 are the value and q = 2, 3
  // the gate columns), loaded one tile ahead of its use.
  auto load_bias = [&](int J, float4 (&b)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      b[q] = e.bias ? *reinterpret_cast<const float4*>(e.bias + n0 + wn * WC + J * 32 + 8 * q + hq)
                    : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  static_for<0, TM>([&](auto I) {
    const int mrow0 = m0 + wm * (BM / WM) + I.value * 32;
    if (resid) {  // (not with GEGLU)
#pragma unroll
      for (int u = 0; u < RPL; ++u) {
        const int c = lane + 64 * u, row = c / RCH, ch = c - row * RCH;
        *reinterpret_cast<bf16x8*>(R + row * LD + ch * 8) = rres[u];
      }
      asm volatile("" ::: "memory");  // (one wave's LDS accesses complete in order)
    }
    static_for<0, TN>([&](auto J) {
      float4 bj[4];
      load_bias(J.value, bj);
      const f32x16 v = acc[I.value][J.value];
      const int nt = n0 + wn * WC + J.value * 32;
      const int m = mrow0 + lr;
      const float rs = row_scale(e, m, a.M);
      if (geglu) {
        // packed columns 32t + u (a) and 32t + 16 + u (gate) -> channel 16t + u
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float ba[4] = {bj[q].x, bj[q].y, bj[q].z, bj[q].w};
          const float bg[4] = {bj[q + 2].x, bj[q + 2].y, bj[q + 2].z, bj[q + 2].w};
          float x[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float av = fmaf(v[4 * q + k], rs, ba[k]);
            const float g = fmaf(v[4 * (q + 2) + k], rs, bg[k]);
            x[k] = av * gelu_as(g);
          }
          bf16x4 o;
#pragma unroll
          for (int k = 0; k < 4; ++k) o[k] = (bf16)x[k];
          *reinterpret_cast<bf16x4*>(R + lr * LD + J.value * 16 + 8 * q + hq) = o;
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = nt + 8 * q + hq;
          // (one rounding for scale and bias, written out so that it does not
          // depend on the compiler's contraction choices; bj is 0 without a bias)
          float x[4] = {fmaf(v[4 * q], rs, bj[q].x), fmaf(v[4 * q + 1], rs, bj[q].y),
                        fmaf(v[4 * q + 2], rs, bj[q].z), fmaf(v[4 * q + 3], rs, bj[q].w)};
          if (e.tbias && m < a.M) {
            const float4 b = *reinterpret_cast<const float4*>(e.tbias + (long)(m / e.hw) * e.tb_ld + e.tb_off + n);
            x[0] += b.x; x[1] += b.y; x[2] += b.z; x[3] += b.w;
          }
          bf16* slot = R + lr * LD + J.value * 32 + 8 * q + hq;
          if (resid) {
            const bf16x4 r = *reinterpret_cast<const bf16x4*>(slot);
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] += (float)r[k];
          }
          if (n < e.qcols) {
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] *= e.qscale;
          }
          bf16x4 o;
#pragma unroll
          for (int k = 0; k < 4; ++k) o[k] = (bf16)x[k];
          *reinterpret_cast<bf16x4*>(slot) = o;
        }
      }
    });
    asm volatile("" ::: "memory");
    if (resid && I.value + 1 < TM) load_resid(mrow0 + 32);
    // Every LDS read of a run of chunks is issued before its first store,
    // so the stores wait for the LDS once per run rather than once per
    // chunk; the row width in chunks is a compile-time constant per case.
    auto store_rows = [&](auto cpc) {
      constexpr int CP = decltype(cpc)::value, NCH = 32 * CP / 64, SH = (NCH + 1) / 2;
      static_assert((32 * CP) % 64 == 0, "row chunks spread evenly over the lanes");
      const int nout = geglu ? a.N / 2 : a.N;
#pragma unroll
      for (int h = 0; h < NCH; h += SH) {
        bf16x8 ob[SH];
#pragma unroll
        for (int u = 0; u < SH; ++u) {
          if (h + u < NCH) {
            const int c = lane + 64 * (h + u), row = c / CP, ch = c - row * CP;
            ob[u] = *reinterpret_cast<const bf16x8*>(R + row * LD + ch * 8);
          }
        }
#pragma unroll
        for (int u = 0; u < SH; ++u) {
          if (h + u < NCH) {
            const int c = lane + 64 * (h + u), row = c / CP, ch = c - row * CP;
            const int m = mrow0 + row;
            if (m < a.M && ncol0 + ch * 8 < nout)
              *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16*>(e.out) + out_row(e, m) * e.ldo + ncol0 + ch * 8) =
                  ob[u];
          }
        }
      }
    };
    if (geglu)
      store_rows(IC<WC / 16>{});
    else
      store_rows(IC<WC / 8>{});
    asm volatile("" ::: "memory");
  });
}

// The transposed part of a QKV projection (V written [image][channel][token]
// for the attention kernel): the wave stages its 32 tokens x WC channels
// channel-major, then stores 16-byte runs of 8 consecutive tokens.  Needs
// the 32 tokens in one image at a multiple of 32 (vt_hw % 32 == 0) and
// 16-byte aligned channel rows (vt_ld % 8 == 0).
template <int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void epilogue_staged_vt(const GemmArgs& a, const f32x16 (&acc)[TM][TN], int m0, int n0,
                                                   int wm, int wn, int lane, bf16* R) {
  constexpr int WC = BN / WN;
  const Epi& e = a.epi;
  const int lr = lane & 31, hq = 4 * (lane >> 5);
  const int c0 = n0 + wn * WC - e.vt_col0;  // first V channel of the wave
  static_for<0, TM>([&](auto I) {
    const int mrow0 = m0 + wm * (BM / WM) + I.value * 32;
    const float rs = row_scale(e, mrow0 + lr, a.M);
    static_for<0, TN>([&](auto J) {
      const f32x16 v = acc[I.value][J.value];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) R[(J.value * 32 + 8 * q + hq + k) * 32 + lr] = (bf16)(v[4 * q + k] * rs);
    });
    asm volatile("" ::: "memory");  // (one wave's LDS accesses complete in order)
    const int img = mrow0 / e.vt_hw, tok0 = mrow0 - img * e.vt_hw;
    bf16* dst = reinterpret_cast<bf16*>(e.vt_out) + (long)img * e.vt_img + (long)c0 * e.vt_ld + tok0;
    for (int c = lane; c < WC * 4; c += 64) {
      const int ch = c >> 2, part = c & 3;
      if (mrow0 + 8 * part < a.M)  // (M is a multiple of vt_hw, hence of 32)
        *reinterpret_cast<bf16x8*>(dst + (long)ch * e.vt_ld + 8 * part) =
            *reinterpret_cast<const bf16x8*>(R + ch * 32 + 8 * part);
    }
    asm volatile("" ::: "memory");
  });
}

// Loader modes.
//  0: per-thread addressing of any layer (incl. the GroupNorm affine on load).
//  1: every segment is a stride-1 3x3 or 1x1 layer on an image of the
//     output's size with cin and the source split c0 multiples of BK, so a
//     K tile lies in one (segment, tap, source) and the input pixel of row m
//     under tap (ky, kx) is m + (ky-1) W + (kx-1): the tile's addressing is
//     uniform and each row keeps only m and a 9-bit mask of in-image taps.
//  2: one stride-2 or upsampling 3x3 segment with cin a multiple of BK:
//     uniform tap per tile, rows keep (image base pixel, oy, ox).
// Modes 1 and 2 read through buffer resources: a masked-off element gets an
// out-of-range offset, which the hardware returns as zero, so the loads are
// branch-free.

template <int BM, int BN, int BK, int WM, int WN, int MODE, int MINB>
__global__ __launch_bounds__(256, MINB) void gemm_bf16_kernel(GemmArgs a) {
  constexpr int LDS_LD = BK + 8;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;  // 32x32 tiles per wave
  constexpr int CPR = BK / 8, RPP = 256 / CPR;         // chunks per row, rows per pass
  constexpr int AR = (BM + RPP - 1) / RPP, BR = (BN + RPP - 1) / RPP;  // 16-byte chunks per thread
  static_assert(BM % RPP == 0, "A tile rows must be a multiple of the rows per loader pass");
  __shared__ __attribute__((aligned(16))) bf16 As[2][BM * LDS_LD];
  __shared__ __attribute__((aligned(16))) bf16 Bs[2][BN * LDS_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_n = (a.N + BN - 1) / BN;
  int bid = blockIdx.x;
  const int nb = gridDim.x;
  if ((nb & 7) == 0) bid = (bid & 7) * (nb >> 3) + (bid >> 3);
  const int tm = bid / tiles_n, tn = bid - tm * tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;

  const int kc = tid % CPR, lrow = tid / CPR;  // loader: chunk kc of rows lrow + RPP j
  constexpr int NR = MODE == 0 ? 1 : AR;
  RowPos rp[MODE == 0 ? AR : 1];
  int ra0[NR], ra1[NR];  // mode 1: (m, tap mask); mode 2: (image base pixel, oy << 16 | ox)
  const int Ho = a.seg[0].Ho, Wo = a.seg[0].Wo, hwo = Ho * Wo;
  if constexpr (MODE == 1) {
#pragma unroll
    for (int j = 0; j < AR; ++j) {
      const int m = m0 + lrow + RPP * j;
      const int p = m % hwo, oy = p / Wo, ox = p - oy * Wo;
      int mk = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int iy = oy + t / 3 - 1, ix = ox + t % 3 - 1;
        if (iy >= 0 && iy < Ho && ix >= 0 && ix < Wo) mk |= 1 << t;
      }
      ra0[j] = m;
      ra1[j] = m < a.M ? mk : 0;
    }
  } else if constexpr (MODE == 2) {
#pragma unroll
    for (int j = 0; j < AR; ++j) {
      const int m = m0 + lrow + RPP * j;
      const int img = m / hwo, p = m - img * hwo, oy = p / Wo, ox = p - oy * Wo;
      ra0[j] = img * a.seg[0].Hi * a.seg[0].Wi;
      ra1[j] = m < a.M ? (oy << 16) | ox : -1;
    }
  } else {
#pragma unroll
    for (int j = 0; j < AR; ++j) rp[j] = decode_row(a.seg[0], m0 + lrow + RPP * j, a.M);
  }
  const __amdgpu_buffer_rsrc_t bres = make_rsrc(a.B, (long)a.N * a.ldb * 2);
  int boff[BR];
#pragma unroll
  for (int j = 0; j < BR; ++j) {
    const int n = n0 + lrow + RPP * j;
    boff[j] = (n < a.N && lrow + RPP * j < BN) ? n * a.ldb * 2 : OOB;
  }

  bf16x8 ra[AR], rb[BR];
  // Uniform loader state of the next K tile (modes 1, 2): segment, tap and
  // channel base, advanced by BK per tile without divisions.
  int st_seg = 0, st_tap = 0, st_cb = 0;
  auto gload = [&](int kt) {
    const int k = kt * BK + kc * 8;
    const bf16x8 z = {};
    if constexpr (MODE != 0) {
      // (fields are picked one by one: selecting a whole kernel-argument
      // struct by a runtime condition would copy it to scratch)
      const int k0 = kt * BK;
      const bool s1 = MODE == 1 && st_seg;
      const int gcin = s1 ? a.seg[1].cin : a.seg[0].cin, gks = s1 ? a.seg[1].ks : a.seg[0].ks;
      const int gc0 = s1 ? a.seg[1].c0 : a.seg[0].c0, gc1 = s1 ? a.seg[1].c1 : a.seg[0].c1;
      const void* gs0 = s1 ? a.seg[1].src0 : a.seg[0].src0;
      const void* gs1 = s1 ? a.seg[1].src1 : a.seg[0].src1;
      const int tap = st_tap, cb = st_cb;
      st_cb += BK;
      if (st_cb >= gcin) {
        st_cb = 0;
        if (++st_tap == gks * gks) {
          st_tap = 0;
          st_seg = 1;
        }
      }
      const bool in0 = cb < gc0;
      const int cs = in0 ? gc0 : gc1, c2 = 2 * ((in0 ? cb : cb - gc0) + kc * 8);
      const bool live = k0 < a.K;
      if constexpr (MODE == 1) {
        const long npix = a.M;
        const __amdgpu_buffer_rsrc_t ares = make_rsrc(in0 ? gs0 : gs1, npix * cs * 2);
        // tap offset (dy, dx) and its bit in the 3x3 in-image mask (a 1x1 tap
        // is the centre; an upsample phase's 2x2 taps are four of the nine)
        const int gpy = s1 ? a.seg[1].py : a.seg[0].py, gpx = s1 ? a.seg[1].px : a.seg[0].px;
        const int tdy = gks == 3 ? tap / 3 - 1 : (gks == 2 ? gpy - 1 + (tap >> 1) : 0);
        const int tdx = gks == 3 ? tap % 3 - 1 : (gks == 2 ? gpx - 1 + (tap & 1) : 0);
        const int t9 = (tdy + 1) * 3 + tdx + 1;
        const int dpix = tdy * Wo + tdx;
#pragma unroll
        for (int j = 0; j < AR; ++j) {
          const bool ok = live && ((ra1[j] >> t9) & 1);
          ra[j] = buf_load16(ares, ok ? (ra0[j] + dpix) * cs * 2 + c2 : OOB);
        }
      } else {
        const ASeg& g = a.seg[0];
        const long npix = (long)(a.M / hwo) * g.Hi * g.Wi;
        const __amdgpu_buffer_rsrc_t ares = make_rsrc(in0 ? gs0 : gs1, npix * cs * 2);
        const int ky = tap / 3 - 1, kx = tap % 3 - 1;
#pragma unroll
        for (int j = 0; j < AR; ++j) {
          const int oy = ra1[j] >> 16, ox = ra1[j] & 0xFFFF;
          int iy, ix;
          bool ok;
          if (g.up) {
            iy = oy + ky;
            ix = ox + kx;
            ok = iy >= 0 && iy < 2 * g.Hi && ix >= 0 && ix < 2 * g.Wi;
            iy >>= 1;
            ix >>= 1;
          } else {
            iy = oy * g.stride + ky;
            ix = ox * g.stride + kx;
            ok = iy >= 0 && iy < g.Hi && ix >= 0 && ix < g.Wi;
          }
          ok = ok && live && ra1[j] >= 0;
          ra[j] = buf_load16(ares, ok ? (ra0[j] + iy * g.Wi + ix) * cs * 2 + c2 : OOB);
        }
      }
    } else if (k < a.seg[0].K) {
      const int tap = k / a.seg[0].cin, c = k - tap * a.seg[0].cin;
#pragma unroll
      for (int j = 0; j < AR; ++j) ra[j] = a_chunk_bf16(a.seg[0], rp[j], tap, c);
    } else if (k < a.K) {
      const int kk = k - a.seg[0].K;
      const int tap = kk / a.seg[1].cin, c = kk - tap * a.seg[1].cin;
#pragma unroll
      for (int j = 0; j < AR; ++j) {
        const bf16* p = a_chunk_ptr<bf16>(a.seg[1], rp[j], tap, c);
        ra[j] = p ? *reinterpret_cast<const bf16x8*>(p) : z;
      }
    } else {
#pragma unroll
      for (int j = 0; j < AR; ++j) ra[j] = z;
    }
    const bool kin = k < a.K;
#pragma unroll
    for (int j = 0; j < BR; ++j) rb[j] = buf_load16(bres, kin ? boff[j] + 2 * k : OOB);
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int j = 0; j < AR; ++j) *reinterpret_cast<bf16x8*>(&As[buf][(lrow + RPP * j) * LDS_LD + kc * 8]) = ra[j];
#pragma unroll
    for (int j = 0; j < BR; ++j)
      if (BN % RPP == 0 || lrow + RPP * j < BN)
        *reinterpret_cast<bf16x8*>(&Bs[buf][(lrow + RPP * j) * LDS_LD + kc * 8]) = rb[j];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = (a.K + BK - 1) / BK;
  gload(0);
  sstore(0);
  __syncthreads();
  const int lr = lane & 31, lk = 8 * (lane >> 5);
  const int arow = wm * (BM / WM) + lr, brow = wn * (BN / WN) + lr;
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) gload(kt + 1);
    const bf16* Ab = As[cur];
    const bf16* Bb = Bs[cur];
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        af[i] = *reinterpret_cast<const bf16x8*>(&Ab[(arow + i * 32) * LDS_LD + ks * 16 + lk]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bfr[j] = *reinterpret_cast<const bf16x8*>(&Bb[(brow + j * 32) * LDS_LD + ks * 16 + lk]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) sstore(cur ^ 1);
    __syncthreads();
  }

  epilogue_tiles<BM, BN, WM, WN>(a, acc, m0, n0, wm, wn, lane);
}

// ------------------------------------------------- bf16 MFMA, direct-to-LDS
// The C^T tiles of the uniform-tap loader modes (1, 2), with the operand tiles
// fetched by buffer_load ... lds: each 64-lane load writes 1 KB of LDS
// contiguously (lane l at byte 16 l), so the loads need no registers.  A tile
// row holds the CPR = DK / 8 16-byte chunks of a DK-deep K slice; chunk c of
// row r sits in slot c ^ swz(r), which keeps the fragment reads of 16
// consecutive rows on distinct banks.  Lane l of a load writes (row
// (64 / CPR) i + l / CPR, slot l % CPR) and fetches the chunk of that slot.
//
// No one unit bounds these kernels: at 196608 x 320 x 2880 the products with their
// LDS reads take 241 us without the loads, the loads 210 us without the products,
// both together 341 (12288 x 1280 x 11520 in 2 splits 235, 208 and 344; 24576 x
// 640 x 2560 69, 64 and 90): the two streams overlap by a quarter to a third.
// A row of 64 bytes (DK = 32) moves a whole 128-byte line from L2 for half of it:
// 66 B/ns per CU against 130 for rows of 128 bytes (DK = 64; a loop of such loads
// over 2.6 MB).  So every layer whose channels are multiples of 64 takes 64-deep
// stages; DKS-deep ones serve the rest (conv_in, padded to 32 channels) and short
// 1x1 layers.  Against 32-deep stages with the addresses formed per tile, in one
// process: 196608 x 320 x 2880 389 -> 318 us, 12288 x 1280 x 11520 (2 splits) 359
// -> 318 us, 512 x 1280 x 5120 100 -> 25 us.
constexpr int DKS = 32;  // the smallest stage depth (the granule of split K and of the loader modes)

// Slot swizzle of a tile row's 16-byte chunks: the fragment reads of rows
// r..r+15 at one logical chunk land on distinct 16-byte bank groups (4
// chunks per row: 64-byte rows; 8 chunks: 128-byte rows).
template <int CPR>
__device__ __forceinline__ int swz(int r) {
  return CPR == 4 ? (r >> 2) & 3 : (r >> 1) & 7;
}

// Position of the operand loads in the K tiles, all wave-uniform.  Tiles come
// in runs: with TI (images larger than 8x8) a run is one DK-channel block
// under all taps of its layer, otherwise one tap (or 1x1 layer) over the
// channels of one source.  Inside a run a tile only adds constants to the
// source pointer, the weight offset and the tap number, so the refill beside
// the products is a handful of scalar instructions plus two vector ones per
// A load (the per-tile selects and divisions it replaces cost about 140
// instructions, as long as the tile's products).
struct KPos {
  const char* ab;    // source + (tap displacement * channels + channel) elements
  int boff;          // byte offset of the tile's weight columns
  int sh;            // 31 - tap (0..8; 9 = every row masked)
  int dead;          // bit 31: past the last tile
  int left, tp;      // tiles until the next run; tap step within the run
  int da, daw, db;   // per-tile steps: source bytes (daw where a kernel row ends), weight bytes
  int dsh, dshw, wm; // tap steps likewise; wm: bit tp set where a kernel row ends
  int togo;          // tiles until the end of this block's K range
  int seg, cb, tap;  // of the run
  int cs2;           // bytes per pixel of the run's source
  bool ti;           // the run steps through taps
};

// A wave-uniform value the compiler would otherwise keep in vector registers
// (what divisions and their users leave there).
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const char* uni(const char* p) {
  const uint64_t v = (uint64_t)p;
  return (const char*)(((uint64_t)(uint32_t)uni((int)(v >> 32)) << 32) | (uint32_t)uni((int)v));
}

template <typename T>
__device__ __forceinline__ T pick(bool c, T a, T b) {
  return c ? a : b;
}

// A and B tiles of DK-deep K slices in DNS LDS stages, one barrier per tile.
// All stages are in flight; fragments are read ahead of their products (a
// 16-deep substep, or a tile for the smallest wave tiles), the next tile's
// first ones after its wait and the barrier, beside this tile's last products,
// and with them goes the refill of the stage this tile has freed.
// UP: the layer upsamples its input (nearest 2x), so the input pixel of a tap
// depends on the row's parity and is formed per tile.
// LIN: a 1x1 layer of one source, so a row is its input pixel, no tap is masked
// and the K tiles are one run.  The general form's setup costs a short layer
// much, above all between other kernels, where its instructions come from beyond
// the caches: 131072 x 320 x 320 in 256x160 tiles 69 us with the general setup and
// 61 with this one (77 and 71 after four other kernels), 512 x 1280 x 1280 18.2 and
// 15.8 (13.8 and 11.6), 49152 x 5120 x 640 451 and 424.
template <int BM, int BN, int WM, int WN, bool UP, int DK, int DNS, int MINB, bool TI, bool LIN = false>
__global__ __launch_bounds__(64 * WM * WN, MINB) void gemm_bf16_dma_kernel(GemmArgs a) {
  constexpr int NWV = WM * WN;                          // waves per block
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int CPR = DK / 8, RPL = 64 / CPR;           // 16-byte chunks per row, rows per load
  constexpr int AI = BM / RPL, BI = BN / RPL;           // 1 KB loads per tile
  constexpr int AW = AI / NWV, BW = (BI + NWV - 1) / NWV;  // ... per wave
  constexpr int LPT = AW + BW;
  static_assert(DNS >= 2 && (DNS - 1) * LPT < 64, "pipeline depth, vmcnt range");
  static_assert(AI % NWV == 0, "A tile must split evenly over the waves");
  // Operand stages (A then B; where the B loads do not split evenly over the
  // waves, the surplus ones write zeros to a spare slot, so that every wave
  // counts the same loads per tile); after the K loop the same LDS stages
  // the output tile for the row-contiguous stores of the epilogue.
  constexpr bool SPARE = BI % NWV != 0;
  constexpr int OPS = DNS * (BM + BN) * DK + (SPARE ? 512 : 0);
  constexpr int STG = NWV * 32 * STAGED_LD<BN / WN>;
  __shared__ __attribute__((aligned(1024))) bf16 smem[OPS > STG ? OPS : STG];
  bf16* const As = smem;
  bf16* const Bs = smem + DNS * BM * DK;
  bf16* const spare = smem + DNS * (BM + BN) * DK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uni(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_n = (a.N + BN - 1) / BN;
  // consecutive tiles on one XCD (blocks are dealt round-robin over 8)
  int bid = blockIdx.x;
  {
    const int nb = gridDim.x, q = nb >> 3, r = nb & 7, x = bid & 7;
    bid = x * q + min(x, r) + (bid >> 3);
  }
  // split-K: blocks split * tiles .. cover K tiles [kb, ke) of their output tile
  const int tiles = gridDim.x / a.ksplit, split = uni(bid / tiles);
  bid -= split * tiles;
  const int tm = bid / tiles_n, tn = bid - tm * tiles_n;
  const int m0 = uni(tm * BM), n0 = uni(tn * BN);

  // Rows and chunks this lane fetches: A load j of this wave is tile load
  // i = wave * AW + j (rows RPL i ..); B load j is i = wave + NWV j.  A row
  // keeps its input pixel under the centre tap (UP: image base and output
  // position) and the taps outside the image (bit 9: a tap that always is).
  const int lrow = lane / CPR, lslot = lane % CPR;
  const int Hi = a.seg[0].Hi, Wi = a.seg[0].Wi, Ho = a.seg[0].Ho, Wo = a.seg[0].Wo, hwo = Ho * Wo;
  const int stride = a.seg[0].stride;
  int pix[AW], pyx[UP ? AW : 1], nmask[AW], voffA[AW];
#pragma unroll
  for (int j = 0; j < AW; ++j) {
    const int m = m0 + RPL * (wave * AW + j) + lrow;
    if constexpr (LIN) {
      pix[j] = m;
      continue;
    }
    const int img = m / hwo, p = m - img * hwo, oy = p / Wo, ox = p - oy * Wo;
    int mk = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int iy = oy * stride + t / 3 - 1, ix = ox * stride + t % 3 - 1;
      if (iy >= 0 && iy < (UP ? 2 * Hi : Hi) && ix >= 0 && ix < (UP ? 2 * Wi : Wi)) mk |= 1 << t;
    }
    nmask[j] = m < a.M ? ~mk : -1;
    pix[j] = UP ? img * Hi * Wi : img * Hi * Wi + oy * stride * Wi + ox * stride;
    if constexpr (UP) pyx[j] = (oy << 16) | ox;
  }
  // byte of the 16-byte chunk this lane fetches in tile load i
  auto chunk16 = [&](int i) __attribute__((always_inline)) { return 16 * (lslot ^ swz<CPR>(RPL * i + lrow)); };
  const __amdgpu_buffer_rsrc_t bres = make_rsrc(a.B, (long)a.N * a.ldb * 2);
  int voffB[BW];
#pragma unroll
  for (int j = 0; j < BW; ++j) {
    const int i = wave + NWV * j, n = n0 + RPL * i + lrow;
    voffB[j] = (i < BI && n < a.N) ? n * a.ldb * 2 + chunk16(i) : OOB;
  }

  const int nk_all = (a.K + DK - 1) / DK;  // K is a multiple of DK
  const int per = uni((nk_all + a.ksplit - 1) / a.ksplit);
  const int kb = split * per, nk = max(min(nk_all, kb + per) - kb, 0);

  // The segment fields the runs read, read once and selected as values
  // (selecting between lvalues would keep them in scratch).
  const void *g0s0 = a.seg[0].src0, *g0s1 = a.seg[0].src1, *g1s0 = a.seg[1].src0, *g1s1 = a.seg[1].src1;
  const int g0ks = a.seg[0].ks, g0cin = a.seg[0].cin, g0c0 = a.seg[0].c0, g0c1 = a.seg[0].c1, g0py = a.seg[0].py,
            g0px = a.seg[0].px, g0K = a.seg[0].K;
  const int g1ks = a.seg[1].ks, g1cin = a.seg[1].cin, g1c0 = a.seg[1].c0, g1c1 = a.seg[1].c1;
  KPos s;
  auto set_source = [&](int cs2) __attribute__((always_inline)) {
    s.cs2 = cs2;
    if constexpr (!UP) {
#pragma unroll
      for (int j = 0; j < AW; ++j) {
        voffA[j] = pix[j] * cs2 + chunk16(wave * AW + j);
        if (LIN && pix[j] >= a.M) voffA[j] = OOB;
      }
    }
  };
  // Start the run that holds (segment, tap, channel).
  auto place = [&](int seg, int tap, int cb) __attribute__((always_inline)) {
    const bool s1 = seg != 0;
    const int ks = pick(s1, g1ks, g0ks), cin = pick(s1, g1cin, g0cin), c0 = pick(s1, g1c0, g0c0);
    const int c1 = pick(s1, g1c1, g0c1);
    const int py = g0py, px = g0px;  // (an upsample phase has one segment)
    const bool in0 = cb < c0;
    const char* src = (const char*)pick(in0, pick(s1, g1s0, g0s0), pick(s1, g1s1, g0s1));
    const int cs = pick(in0, c0, c1);
    // tap displacement; its bit in the 3x3 in-image mask (a 1x1 tap is the
    // centre; an upsample phase's 2x2 taps are four of the nine)
    const int ky = ks == 1 ? 1 : (ks == 3 ? tap / 3 : py + (tap >> 1));
    const int kx = ks == 1 ? 1 : (ks == 3 ? tap % 3 : px + (tap & 1));
    const int dpix = UP ? 0 : (ky - 1) * Wi + kx - 1;
    s.ab = src + ((long)dpix * cs + (in0 ? cb : cb - c0)) * 2;
    s.boff = (pick(s1, g0K, 0) + tap * cin + cb) * 2;
    s.sh = 31 - (3 * ky + kx);
    s.ti = TI && ks > 1;
    if (s.ti) {
      s.left = ks * ks - tap;
      s.tp = tap;
      s.da = UP ? 0 : 2 * cs;
      s.daw = UP ? 0 : (Wi - ks + 1) * 2 * cs;
      s.db = 2 * cin;
      s.dsh = 1;
      s.dshw = 4 - ks;
      s.wm = ks == 3 ? 0x24 : 0x2;
    } else {
      s.left = (pick(in0, c0, cin) - cb) / DK;
      s.tp = 0;
      s.da = s.daw = s.db = 2 * DK;
      s.dsh = s.dshw = s.wm = 0;
    }
    s.ab = uni(s.ab);
    s.boff = uni(s.boff);
    s.sh = uni(s.sh);
    s.da = uni(s.da);
    s.daw = uni(s.daw);
    s.db = uni(s.db);
    s.dsh = uni(s.dsh);
    s.dshw = uni(s.dshw);
    s.wm = uni(s.wm);
    s.left = uni(min(s.left, s.togo));
    s.seg = seg;
    s.cb = cb;
    s.tap = tap;
    if (s.cs2 != 2 * cs) set_source(2 * cs);
  };
  // The run after the current one, or past the end.
  auto next_run = [&]() __attribute__((always_inline)) {
    if (s.togo == 0) {
      s.dead = OOB;
      s.sh = 31 - 9;
      s.da = s.daw = s.db = s.dsh = s.dshw = 0;
      s.left = 0x7FFFFFFF;
      return;
    }
    const bool s1 = s.seg != 0;
    const int ks = pick(s1, g1ks, g0ks), cin = pick(s1, g1cin, g0cin), c0 = pick(s1, g1c0, g0c0);
    int seg = s.seg, tap = 0, cb = 0;
    if (s.ti) {
      cb = s.cb + DK;
      if (cb == cin) {
        cb = 0;
        ++seg;
      }
    } else {
      tap = s.tap;
      cb = pick(s.cb < c0, c0, cin);
      if (cb == cin) {
        cb = 0;
        if (++tap == ks * ks) {
          tap = 0;
          ++seg;
        }
      }
    }
    place(seg, tap, cb);
  };
  // Issue the loads of the next K tile into stage `stg`.
  auto issue = [&](int stg) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t ares = make_rsrc(s.ab, 0x7FFFFFFF);
    bf16* adst = As + stg * BM * DK + wave * AW * 512;
#pragma unroll
    for (int j = 0; j < AW; ++j) {
      int v = voffA[j];
      if constexpr (UP) {
        const int t9 = 31 - s.sh, ky = t9 / 3 - 1, kx = t9 % 3 - 1;
        const int iy = ((pyx[j] >> 16) + ky) >> 1, ix = ((pyx[j] & 0xFFFF) + kx) >> 1;
        v = (pix[j] + iy * Wi + ix) * s.cs2 + chunk16(wave * AW + j);
      }
      dma16(ares, adst + j * 512, LIN ? v | s.dead : ((nmask[j] << s.sh) & OOB) | (UP ? v & 0x7FFFFFFF : v), 0);
    }
    bf16* bdst = Bs + stg * BN * DK;
    const int boff = uni(s.boff);
#pragma unroll
    for (int j = 0; j < BW; ++j) {
      const int i = wave + NWV * j;
      dma16(bres, (SPARE && i >= BI) ? spare : bdst + i * 512, voffB[j] | s.dead, boff);
    }
  };
  auto advance = [&]() __attribute__((always_inline)) {
    if constexpr (LIN) {
      s.ab += 2 * DK;
      s.boff += 2 * DK;
      if (--s.togo <= 0) s.dead = OOB;
      return;
    }
    --s.togo;
    if (--s.left == 0) {
      next_run();
    } else {
      const bool w = (s.wm >> (s.tp & 31)) & 1;  // (wm is 0 in the runs of more than 9 tiles)
      s.ab += pick(w, s.daw, s.da);
      s.sh -= pick(w, s.dshw, s.dsh);
      s.boff += s.db;
      ++s.tp;
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  s.cs2 = -1;
  s.dead = 0;
  s.togo = nk;
  if constexpr (LIN) {  // (never split)
    s.ab = uni((const char*)g0s0);
    s.boff = 0;
    set_source(2 * g0c0);
  } else if (nk > 0) {  // the run at K tile kb
    int kk = kb * DK, seg = 0;
    if (kk >= g0K) {
      seg = 1;
      kk -= g0K;
    }
    const int ks = pick(seg != 0, g1ks, g0ks), cin = pick(seg != 0, g1cin, g0cin), taps = ks * ks;
    if (TI && taps > 1) {
      const int i = kk / DK, c = i / taps;
      place(seg, uni(i - c * taps), uni(c * DK));
    } else {
      const int tap = uni(kk / cin);
      place(seg, tap, kk - tap * cin);
    }
  } else {
    s.ab = (const char*)g0s0;
    s.boff = s.tp = 0;
    s.seg = s.cb = s.tap = 0;
    s.ti = false;
    set_source(0);
    next_run();
  }

  const int lr = lane & 31, lh = lane >> 5;
  const int arow = wm * (BM / WM) + lr, brow = wn * (BN / WN) + lr;
  // fragment of row r, chunk c: element r DK + 8 (c ^ swz(r)); rows 32 apart share the swizzle
  constexpr int KS = DK / 16;  // 16-deep substeps per tile
  int fa_off[KS], fb_off[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    fa_off[k] = arow * DK + 8 * ((2 * k + lh) ^ swz<CPR>(arow));
    fb_off[k] = brow * DK + 8 * ((2 * k + lh) ^ swz<CPR>(brow));
  }
  // Fragment sets: the smallest wave tiles (at most two products a substep)
  // hold a whole tile's fragments twice, so an LDS read has a tile's products
  // to land; the others two substeps', unless two blocks of 64 x 160 waves
  // share a CU, which leaves no registers for a second set.
  constexpr bool WT = TM * TN <= 2, PF = !WT && !(TM * TN == 10 && MINB > 1);
  constexpr int NF = WT ? 2 * KS : (PF ? 2 : 1);
  bf16x8 fa[NF][TM], fb[NF][TN];
  auto readf = [&](int stg, int ks, bf16x8 (&af)[TM], bf16x8 (&bfr)[TN]) {
    const bf16* Ab = As + stg * BM * DK + fa_off[ks];
    const bf16* Bb = Bs + stg * BN * DK + fb_off[ks];
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8*>(Ab + i * 32 * DK);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[j] = *reinterpret_cast<const bf16x8*>(Bb + j * 32 * DK);
  };
  auto products = [&](int cur) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][j], fa[cur][i], acc[i][j], 0, 0, 0);
  };
  auto prologue = [&](int n) __attribute__((always_inline)) {
#pragma unroll 1
    for (int p = 0; p < n; ++p) {
      issue(p);
      advance();
    }
  };
  // The wait and barrier after which tile kt + 1 may be read and the stage of
  // tile kt refilled: its loads have landed (DNS - 2 tiles stay in flight) and
  // this wave's reads of tile kt are complete.
  auto next_ready = [&]() __attribute__((always_inline)) {
    wait_vmcnt<(DNS - 2) * LPT>();
    wait_lgkm0();
    stage_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  int st = 0;  // stage of the tile
  if constexpr (WT) {
    prologue(DNS);
    wait_vmcnt<(DNS - 1) * LPT>();  // tile 0 has landed
    stage_barrier();
    static_for<0, KS>([&](auto K) { readf(0, K.value, fa[K.value], fb[K.value]); });
    auto tile = [&](auto CUR) __attribute__((always_inline)) {
      constexpr int cur = CUR.value * KS, nxt = KS - cur;
      const int nst = st + 1 == DNS ? 0 : st + 1;
      next_ready();
      static_for<0, KS>([&](auto K) { readf(nst, K.value, fa[nxt + K.value], fb[nxt + K.value]); });
      issue(st);
      static_for<0, KS>([&](auto K) { products(cur + K.value); });
      advance();
      st = nst;
    };
    for (int kt = 0; kt < nk; kt += 2) {
      tile(IC<0>{});
      if (kt + 1 < nk) tile(IC<1>{});
    }
  } else if constexpr (PF) {
    prologue(DNS);
    wait_vmcnt<(DNS - 1) * LPT>();  // tile 0 has landed
    stage_barrier();
    readf(0, 0, fa[0], fb[0]);
    for (int kt = 0; kt < nk; ++kt) {
      const int nst = st + 1 == DNS ? 0 : st + 1;
      static_for<0, KS>([&](auto KSI) {
        constexpr int ks = KSI.value, cur = ks & 1, nxt = cur ^ 1;
        if constexpr (ks + 1 < KS) {
          readf(st, ks + 1, fa[nxt], fb[nxt]);
          if constexpr (TM * TN > 4) __builtin_amdgcn_sched_barrier(0);  // the reads go out before the products
          products(cur);
        } else {
          if constexpr (TM * TN > 4) __builtin_amdgcn_sched_barrier(0);  // the previous products stay above
          next_ready();
          readf(nst, 0, fa[nxt], fb[nxt]);
          issue(st);
          products(cur);
          if constexpr (TM * TN > 4) {
            // the fragment reads, then the refill loads, spread over the products
            constexpr int NP = TM * TN, NR = TM + TN;
            constexpr int LP = NP > NR ? NP - NR : 1;  // products left for the loads
            static_for<0, NP>([&](auto Q) {
              constexpr int q = Q.value, l = q - (NP - LP);
              if constexpr (q < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
              if constexpr (l >= 0 && (l + 1) * LPT / LP > l * LPT / LP)
                __builtin_amdgcn_sched_group_barrier(0x020, (l + 1) * LPT / LP - l * LPT / LP, 0);  // VMEM read
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            });
          }
          advance();
        }
      });
      st = nst;
    }
  } else {
    prologue(DNS - 1);
    for (int kt = 0; kt < nk; ++kt) {
      next_ready();  // (here: tile kt may be read, the stage of tile kt - 1 refilled)
      static_for<0, KS>([&](auto KSI) {
        constexpr int ks = KSI.value;
        readf(st, ks, fa[0], fb[0]);
        if constexpr (ks == 0) issue(st == 0 ? DNS - 1 : st - 1);
        products(0);
      });
      advance();
      st = st + 1 == DNS ? 0 : st + 1;
    }
  }
  wait_vmcnt<0>();  // the refills past the last tile have landed
  if (a.ksplit > 1) {
    // raw fp32 partial sums; the reduction kernel applies the epilogue
    const int lr = lane & 31, hq = 4 * (lane >> 5);
    float* P = a.partial + (long)split * a.M * a.N;
    static_for<0, TM>([&](auto I) {
      static_for<0, TN>([&](auto J) {
        const f32x16 v = acc[I.value][J.value];
        const int m = m0 + wm * (BM / WM) + I.value * 32 + lr;
        const int nt = n0 + wn * (BN / WN) + J.value * 32;
        if (m < a.M) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = nt + 8 * q + hq;
            if (n < a.N)
              *reinterpret_cast<float4*>(P + (long)m * a.N + n) =
                  make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
          }
        }
      });
    });
    return;
  }
  {
    static_assert(32 * (BN / WN) <= 32 * STAGED_LD<BN / WN>, "transposed staging fits the region");
    const bool vt_ok = a.epi.vt_out && a.epi.vt_col0 % (BN / WN) == 0 && a.epi.vt_hw % 32 == 0 && a.epi.vt_ld % 8 == 0;
    if ((!a.epi.vt_out || vt_ok) && !a.epi.out_f32 && (!a.epi.resid || !a.epi.geglu)) {
      __syncthreads();  // every wave is done with the operand stages
      bf16* R = smem + wave * 32 * STAGED_LD<BN / WN>;
      if (a.epi.vt_out && n0 + wn * (BN / WN) >= a.epi.vt_col0)
        epilogue_staged_vt<BM, BN, WM, WN>(a, acc, m0, n0, wm, wn, lane, R);
      else
        epilogue_staged<BM, BN, WM, WN>(a, acc, m0, n0, wm, wn, lane, R);
      return;
    }
    epilogue_tiles<BM, BN, WM, WN>(a, acc, m0, n0, wm, wn, lane);
  }
}

// Sum of the split-K partials in split order, then the epilogue.
__global__ void splitk_reduce_kernel(GemmArgs a) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;  // one run of 4 columns
  const int nv = a.N / 4;
  if (i >= (long)a.M * nv) return;
  const int m = (int)(i / nv), n = (int)(i - (long)m * nv) * 4;
  float x[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < a.ksplit; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(a.partial + ((long)s * a.M + m) * a.N + n);
    x[0] += v.x; x[1] += v.y; x[2] += v.z; x[3] += v.w;
  }
  epilogue4<bf16>(a.epi, m, n, x);
}

// ---------------------------------------------------------------- fp32 MFMA
// v_mfma_f32_16x16x4_f32: fp32 products and sums.  The fp32 path runs narrow
// layers (the test UNet: 192-768 rows, 4-512 columns, K 32-1152) whose time is
// latency, so a block is one (16 T) x (16 T) output tile with K split over its
// NW waves in 16-deep chunks (wave w takes chunks w, w + NW, ...).  A lane
// loads four consecutive k of its row or column straight into the registers
// the products read (lane l: row l % 16, k 4 (l / 16) .. + 3; element j of
// every lane is MFMA j's k slice), four chunks in flight, no LDS and no barrier
// until the NW partial tiles are added in wave order.  The chunks a wave
// takes and the order of the sums depend on K alone, so a row's bits do not
// depend on the tile or on its batch-mates.  Against 64x64 SIMT tiles with a
// barrier every 16 k (event to event, some 5 us of it the launch): 192 x 64 x
// 576 50 -> 8.9 us, 192 x 64 x 1152 93 -> 11.4 us, 768 x 32 x 32 10.5 -> 6.5 us.
// (tap, channel) of k: k / cin by a float quotient corrected by one (exact below 2^24)
__device__ __forceinline__ void split_k(int k, int cin, float inv_cin, int& tap, int& c) {
  tap = (int)((float)k * inv_cin);
  c = k - tap * cin;
  if (c < 0) {
    --tap;
    c += cin;
  } else if (c >= cin) {
    ++tap;
    c -= cin;
  }
}

template <typename T4>
__device__ __forceinline__ void a_quad(const ASeg& s, const RowPos& r, int k, float inv_cin, T4& v) {
  v = T4{0.f, 0.f, 0.f, 0.f};
  int tap, c;
  split_k(k, s.cin, inv_cin, tap, c);
  const float* p = a_chunk_ptr<float>(s, r, tap, c);
  if (!p) return;
  v = *reinterpret_cast<const T4*>(p);
  if (s.scale) {
    const T4 sc = *reinterpret_cast<const T4*>(s.scale + (long)r.img * s.cin + c);
    const T4 sh = *reinterpret_cast<const T4*>(s.shift + (long)r.img * s.cin + c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = v[i] * sc[i] + sh[i];
      if (s.silu) v[i] = silu_f(v[i]);
    }
  }
}

template <int T, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmArgs a) {
  constexpr int BT = 16 * T, U = 4;  // tile edge; chunks in flight
  __shared__ float part[NW][BT * BT];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles_n = (a.N + BT - 1) / BT;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
  const int m0 = tm * BT, n0 = tn * BT, lr = lane & 15, lk = 4 * (lane >> 4);
  RowPos rp[T];
  const float* bp[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    rp[t] = decode_row(a.seg[0], m0 + 16 * t + lr, a.M);
    const int n = n0 + 16 * t + lr;
    bp[t] = n < a.N ? reinterpret_cast<const float*>(a.B) + (long)n * a.ldb : nullptr;
  }
  // the epilogue's operands are on their way while the products run
  constexpr int OPT = (BT * BT + 64 * NW - 1) / (64 * NW);  // outputs per thread
  float eb[OPT], et[OPT], er[OPT];
#pragma unroll
  for (int i = 0; i < OPT; ++i) {
    const int o = tid + 64 * NW * i, row = m0 + o / BT, col = n0 + o % BT;
    const bool in = o < BT * BT && row < a.M && col < a.N;
    eb[i] = in && a.epi.bias ? a.epi.bias[col] : 0.f;
    et[i] = in && a.epi.tbias ? a.epi.tbias[(long)(row / a.epi.hw) * a.epi.tb_ld + a.epi.tb_off + col] : 0.f;
    er[i] = in && a.epi.resid ? reinterpret_cast<const float*>(a.epi.resid)[(long)row * a.epi.ldr + col] : 0.f;
  }
  const int K0 = a.seg[0].K;
  const float inv0 = 1.0f / (float)a.seg[0].cin, inv1 = a.seg[1].K ? 1.0f / (float)a.seg[1].cin : 0.f;
  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 16 * wave; k0 < a.K; k0 += 16 * NW * U) {
    f32x4 av[U][T], bv[U][T];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 16 * NW * u + lk;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        av[u][t] = bv[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (k < a.K) {
          if (k < K0)
            a_quad(a.seg[0], rp[t], k, inv0, av[u][t]);
          else
            a_quad(a.seg[1], rp[t], k - K0, inv1, av[u][t]);
          if (bp[t]) bv[u][t] = *reinterpret_cast<const f32x4*>(bp[t] + k);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][i][e], bv[u][j][e], acc[i][j], 0, 0, 0);
  }
  // lane l holds rows 4 (l / 16) + r, column l % 16 of each 16x16 tile
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][(16 * i + lk + r) * BT + 16 * j + lr] = acc[i][j][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < OPT; ++i) {
    const int o = tid + 64 * NW * i, row = m0 + o / BT, col = n0 + o % BT;
    if (o < BT * BT && row < a.M && col < a.N) {
      float v = part[0][o];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += part[w][o];
      v = v + eb[i] + et[i] + er[i];
      if (col < a.epi.qcols) v *= a.epi.qscale;
      reinterpret_cast<float*>(a.epi.out)[(long)row * a.epi.ldo + col] = v;
    }
  }
}

// The same sums for large layers, where the form above is bound by its operand
// traffic (a 32x32 tile reads 256 bytes per k for 1024 products): a block of 4
// waves is one 64x64 tile whose 16-deep chunks go through LDS, two to a stage,
// the next stage's loads in flight beside the products.  Chunk c adds to partial
// sum c mod NW of each output, and the NW partial sums are added in order at the
// end, so an output has the bits of the form above.  A thread fetches one quad
// of A and one of B per chunk; a chunk lies in LDS as [row][16 k], so both the
// quads' writes and the fragment reads are contiguous.  What bounds it is issue:
// 16 products (512 cycles) a chunk beside the addressing of two quads, two waves
// per SIMD; 62 TFLOP/s at 32768 x 1280 x 320, 73 at 4096 x 512 x 4608.
template <int NW>
__global__ __launch_bounds__(256, 2) void gemm_f32_tiled_kernel(GemmArgs a) {
  constexpr int BT = 64, CH = 2;  // tile edge; chunks per stage
  __shared__ __attribute__((aligned(16))) float As[2][CH][BT * 16], Bs[2][CH][BT * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles_n = (a.N + BT - 1) / BT;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
  const int m0 = tm * BT, n0 = tn * BT;
  const int kq = 4 * (tid & 3);  // of the quad this thread fetches, in row tid / 4
  const RowPos rp = decode_row(a.seg[0], m0 + (tid >> 2), a.M);
  const bool bok = n0 + (tid >> 2) < a.N;
  const float* bp = reinterpret_cast<const float*>(a.B) + (bok ? (long)(n0 + (tid >> 2)) * a.ldb : 0);
  const int K0 = a.seg[0].K;
  const float inv0 = 1.0f / (float)a.seg[0].cin, inv1 = a.seg[1].K ? 1.0f / (float)a.seg[1].cin : 0.f;
  const int nst = (a.K + 16 * CH - 1) / (16 * CH);

  // The loads have no branches: a masked quad reads the start of its buffer
  // and becomes zero, and the GroupNorm affine is applied, when the stage goes
  // to LDS behind the products.
  const float* ap[CH];
  int ac[CH];  // channel, or -1 where the quad is zero
  auto locate = [&](const ASeg& s, int k, float inv, int c) __attribute__((always_inline)) {
    int tap, ch;
    split_k(k, s.cin, inv, tap, ch);
    int ky = 1, kx = 1;
    if (s.ks == 3) {
      ky = tap / 3;
      kx = tap - ky * 3;
    }
    int iy = rp.oy * s.stride + ky - 1, ix = rp.ox * s.stride + kx - 1;
    const bool ok = rp.ok && iy >= 0 && ix >= 0 && iy < (s.up ? 2 * s.Hi : s.Hi) && ix < (s.up ? 2 * s.Wi : s.Wi);
    iy >>= s.up ? 1 : 0;
    ix >>= s.up ? 1 : 0;
    const bool in0 = ch < s.c0;
    const float* src = reinterpret_cast<const float*>(in0 ? s.src0 : s.src1);
    const long off = (((long)rp.img * s.Hi + iy) * s.Wi + ix) * (in0 ? s.c0 : s.c1) + (in0 ? ch : ch - s.c0);
    ap[c] = src + (ok ? off : 0);
    ac[c] = ok ? ch : -1;
  };
  f32x4 av[CH], bv[CH], asc[CH], ash[CH];
  auto gload = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int k = 16 * (st * CH + c) + kq, kk = min(k, a.K - 4);
      if (kk < K0)
        locate(a.seg[0], kk, inv0, c);
      else
        locate(a.seg[1], kk - K0, inv1, c);
      if (k >= a.K) ac[c] = -1;
      av[c] = *reinterpret_cast<const f32x4*>(ap[c]);
      bv[c] = *reinterpret_cast<const f32x4*>(bp + kk);
      if (a.seg[0].scale) {  // (only ever on a layer of one segment)
        const long o = (long)rp.img * a.seg[0].cin + max(ac[c], 0);
        asc[c] = *reinterpret_cast<const f32x4*>(a.seg[0].scale + o);
        ash[c] = *reinterpret_cast<const f32x4*>(a.seg[0].shift + o);
      }
    }
  };
  auto sstore = [&](int st, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      f32x4 v = av[c], w = bv[c];
      if (a.seg[0].scale) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[i] = v[i] * asc[c][i] + ash[c][i];
          if (a.seg[0].silu) v[i] = silu_f(v[i]);
        }
      }
      const bool kin = 16 * (st * CH + c) + kq < a.K && bok;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = ac[c] >= 0 ? v[i] : 0.f;
        w[i] = kin ? w[i] : 0.f;
      }
      *reinterpret_cast<f32x4*>(&As[buf][c][4 * tid]) = v;
      *reinterpret_cast<f32x4*>(&Bs[buf][c][4 * tid]) = w;
    }
  };
  f32x4 acc[NW][2][2];
#pragma unroll
  for (int w = 0; w < NW; ++w)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[w][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  gload(0);
  sstore(0, 0);
  __syncthreads();
  for (int s0 = 0; s0 < nst; s0 += NW / CH) {
    static_for<0, NW / CH>([&](auto S) {
      const int st = s0 + S.value, buf = st & 1;
      if (st < nst) {  // (uniform)
        if (st + 1 < nst) gload(st + 1);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          // fragment: lane l holds row l % 16, k 4 (l / 16) .. + 3
          f32x4 fa[2], fb[2];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            fa[t] = *reinterpret_cast<const f32x4*>(&As[buf][c][(32 * wm + 16 * t + (lane & 15)) * 16 + 4 * (lane >> 4)]);
            fb[t] = *reinterpret_cast<const f32x4*>(&Bs[buf][c][(32 * wn + 16 * t + (lane & 15)) * 16 + 4 * (lane >> 4)]);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                acc[S.value * CH + c][i][j] =
                    __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[i][e], acc[S.value * CH + c][i][j], 0, 0, 0);
        }
        if (st + 1 < nst) sstore(st + 1, buf ^ 1);
        __syncthreads();
      }
    });
  }
  // (weights as the first operand: lane l holds row l % 16, columns 4 (l / 16) +
  // [0, 4) of each 16x16 tile)
  const Epi& e = a.epi;
  const float* resid = reinterpret_cast<const float*>(e.resid);
  float* out = reinterpret_cast<float*>(e.out);
  const bool vec = !((a.N | e.ldo | (resid ? e.ldr : 0) | (e.tbias ? e.tb_ld | e.tb_off : 0)) & 3) &&
                   !(((uint64_t)out | (uint64_t)resid | (uint64_t)e.bias | (uint64_t)e.tbias) & 15);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = m0 + 32 * wm + 16 * i + (lane & 15);
    if (row >= a.M) continue;
    const float* tb = e.tbias ? e.tbias + (long)(row / e.hw) * e.tb_ld + e.tb_off : nullptr;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + 32 * wn + 16 * j + 4 * (lane >> 4);
      f32x4 v = acc[0][i][j];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += acc[w][i][j];
      f32x4 b{}, t{}, r{};
      if (vec && col < a.N) {
        if (e.bias) b = *reinterpret_cast<const f32x4*>(e.bias + col);
        if (tb) t = *reinterpret_cast<const f32x4*>(tb + col);
        if (resid) r = *reinterpret_cast<const f32x4*>(resid + (long)row * e.ldr + col);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (col + q < a.N) {
            if (e.bias) b[q] = e.bias[col + q];
            if (tb) t[q] = tb[col + q];
            if (resid) r[q] = resid[(long)row * e.ldr + col + q];
          }
      }
      v = v + b + t + r;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (col + q < e.qcols) v[q] *= e.qscale;
      float* o = out + (long)row * e.ldo + col;
      if (vec) {
        if (col < a.N) *reinterpret_cast<f32x4*>(o) = v;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (col + q < a.N) o[q] = v[q];
      }
    }
  }
}

// K split over 8 waves from K = 256 on, else 4 or 2 (a function of K alone);
// 32x32 tiles (half the operand traffic) once 16x16 ones would give the chip
// over four blocks per CU; 64x64 tiles through LDS once they give every CU one,
// unless at most 16 columns use them.  Small form against the LDS one, us: 160
// blocks of 64x64 (512 x 1280 x 1280) 51 and 57, 192 (12288 x 32 x 288) 13.7 and
// 16.8; 256 (16384 x 64 x 576) 36.5 and 27.0, 320 (2048 x 640 x 5760) 346 and
// 323, 640 (8192 x 320 x 320) 65 and 38, 10240 (32768 x 1280 x 320) 1007 and 431;
// 65536 x 8 x 1152 120 and 134.
template <int NW>
static void launch_f32(const GemmArgs& a, hipStream_t s) {
  auto blocks = [&](long bt) { return ((a.M + bt - 1) / bt) * ((a.N + bt - 1) / bt); };
  const bool affine2 = a.seg[1].K && (a.seg[0].scale || a.seg[1].scale);  // (the tiled form's affine is for one segment)
  if (blocks(64) >= 256 && a.N > 16 && !affine2)
    gemm_f32_tiled_kernel<NW><<<dim3((unsigned)blocks(64)), dim3(256), 0, s>>>(a);
  else if (blocks(16) > 1024)
    gemm_f32_kernel<2, NW><<<dim3((unsigned)blocks(32)), dim3(64 * NW), 0, s>>>(a);
  else
    gemm_f32_kernel<1, NW><<<dim3((unsigned)blocks(16)), dim3(64 * NW), 0, s>>>(a);
}

static bool fast_seg(const ASeg& g, int Ho, int Wo, int BK) {
  return g.stride == 1 && !g.up && (g.ks == 1 || g.ks == 2 || g.ks == 3) && g.Hi == Ho && g.Wi == Wo &&
         g.cin % BK == 0 && (g.c1 == 0 || g.c0 % BK == 0) && g.scale == nullptr;
}

// Loader mode of a GEMM (see the kernel); modes 1 and 2 address each source
// with 32-bit byte offsets, so its bytes must stay below 2^31.
static int loader_mode(const GemmArgs& a, int BK) {
  const ASeg& g0 = a.seg[0];
  const long hwo = (long)g0.Ho * g0.Wo;
  if (hwo <= 0 || g0.scale) return 0;
  auto small = [&](const ASeg& g, long npix) {
    return npix * (long)g.c0 * 2 < (1L << 31) && npix * (long)g.c1 * 2 < (1L << 31);
  };
  if (fast_seg(g0, g0.Ho, g0.Wo, BK) && (a.seg[1].K == 0 || fast_seg(a.seg[1], g0.Ho, g0.Wo, BK)) && small(g0, a.M) &&
      (a.seg[1].K == 0 || small(a.seg[1], a.M)) && (long)a.N * a.ldb * 2 < (1L << 31))
    return 1;
  if (a.seg[1].K == 0 && g0.ks == 3 && (g0.stride == 2 || g0.up) && g0.c1 == 0 && g0.cin % BK == 0 &&
      (a.M / hwo) * (long)g0.Hi * g0.Wi * g0.c0 * 2 < (1L << 31) && (long)a.N * a.ldb * 2 < (1L << 31) &&
      g0.Ho < 65536 && g0.Wo < 65536)
    return 2;
  return 0;
}

template <int BM, int BN, int BK, int WM, int WN, int MINB = 1>
static void launch_bf16(const GemmArgs& a, hipStream_t s) {
  const long blocks = (long)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 g((unsigned)blocks), b(256);
  switch (loader_mode(a, BK)) {
    case 1: gemm_bf16_kernel<BM, BN, BK, WM, WN, 1, MINB><<<g, b, 0, s>>>(a); break;
    case 2: gemm_bf16_kernel<BM, BN, BK, WM, WN, 2, MINB><<<g, b, 0, s>>>(a); break;
    default: gemm_bf16_kernel<BM, BN, BK, WM, WN, 0, MINB><<<g, b, 0, s>>>(a); break;
  }
}

// Direct-to-LDS kernel for the uniform-tap modes; false if the layer needs
// the register-staged loader.
template <int BM, int BN, int WM, int WN, int DK, int DNS, int MINB>
static bool launch_dma(const GemmArgs& a, hipStream_t s) {
  // (whole tiles of columns only: the staged epilogues do not mask columns)
  if (loader_mode(a, DK) == 0 || a.N % BN) return false;
  const long blocks = (long)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) * a.ksplit;
  const dim3 g((unsigned)blocks), b(64 * WM * WN);
  // K order (see the kernel): channel block outer, taps inner on images
  // larger than 8x8.
  const bool ti = (long)a.seg[0].Ho * a.seg[0].Wo > 64, up = a.seg[0].up != 0;
  if (a.seg[0].ks == 1 && a.seg[0].c1 == 0 && a.seg[1].K == 0 && a.ksplit == 1)  // (mode 1: stride 1, no upsampling)
    gemm_bf16_dma_kernel<BM, BN, WM, WN, false, DK, DNS, MINB, false, true><<<g, b, 0, s>>>(a);
  else if (!up && ti)
    gemm_bf16_dma_kernel<BM, BN, WM, WN, false, DK, DNS, MINB, true><<<g, b, 0, s>>>(a);
  else if (!up)
    gemm_bf16_dma_kernel<BM, BN, WM, WN, false, DK, DNS, MINB, false><<<g, b, 0, s>>>(a);
  else if (ti)
    gemm_bf16_dma_kernel<BM, BN, WM, WN, true, DK, DNS, MINB, true><<<g, b, 0, s>>>(a);
  else
    gemm_bf16_dma_kernel<BM, BN, WM, WN, true, DK, DNS, MINB, false><<<g, b, 0, s>>>(a);
  if (a.ksplit > 1) {
    const long n = (long)a.M * (a.N / 4);
    splitk_reduce_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(a);
  }
  return true;
}

// Split-K factor of a bf16 GEMM: long-K 3x3 convolutions on the small
// levels (16x16 and 8x8 images) have too few output tiles to fill 256 CUs.
// The factor depends only on K and the per-image output size, never on the
// number of rows, so a row's result does not depend on its batch-mates.
// Linear layers (1x1, the row count as image width) are never split: their
// "image" size is the row count.
int gemm_ksplit(const GemmArgs& a) {
  const long hw = (long)a.seg[0].Ho * a.seg[0].Wo;
  if (a.seg[0].ks != 3 || a.K < 5120 || hw > 256 || a.N % 160 || a.epi.geglu || a.epi.vt_out || a.epi.out_f32)
    return 1;
  if (loader_mode(a, DKS) == 0) return 1;
  return hw <= 64 ? 4 : 2;
}

// Tiles of the 64-deep direct-to-LDS kernel.  A block's time is modelled as
// eb + nk * t us for its nk K tiles, t1 for a block alone on its CU and tf
// when occ blocks share it, fitted to conv and linear shapes of 64 to 262144 rows.
// For the tiles of one block per CU (occ 1) t1 stands for a grid or last round of
// less than 256 blocks and tf for a full chip; what a full one adds is shared by
// all CUs, and sets in late: 192 blocks of 256 x 320 measure 1.5 to 1.6 us a tile
// (24576 x 640 x 2560 84 us, modelled 73).  A time in proportion to the filled share
// was tried instead: of 761 shapes 46 moved by over 3 %, between -11 and +15 %, and
// by +1.4 % in the mean, so the two values stay.  The tile never changes a row's
// K order, so every tile gives the same bits and the choice may follow the row count.
struct Tile64 {
  int bm, bn, occ;
  float t1, tf, eb;
};
static const Tile64 kTiles64[] = {
    {64, 64, 2, 0.224f, 0.402f, 4.6f},     // 4 waves of 32 x 32, four stages
    {128, 64, 2, 0.343f, 0.606f, 7.4f},    // 4 waves of 64 x 32, three stages
    {128, 128, 2, 0.594f, 0.979f, 10.9f},  // 4 waves of 64 x 64, two stages
    {128, 160, 2, 0.668f, 1.344f, 12.4f},  // 4 waves of 32 x 160, two stages
    {256, 256, 1, 1.130f, 1.861f, 16.9f},  // 8 waves of 128 x 64, two stages
    {256, 320, 1, 1.327f, 2.340f, 19.8f},  // 8 waves of 64 x 160, two stages
};

// Index of the tile with the smallest modelled time, -1 when none divides N.
static int pick_tile64(long M, long N, long K, int ksplit) {
  const float nk = (float)((K / 64 + ksplit - 1) / ksplit);
  int best = -1;
  float tbest = 0.f;
  for (int i = 0; i < (int)(sizeof(kTiles64) / sizeof(kTiles64[0])); ++i) {
    const Tile64& t = kTiles64[i];
    if (N % t.bn) continue;
    const long blocks = (M + t.bm - 1) / t.bm * (N / t.bn) * ksplit, slots = 256L * t.occ;
    const long full = blocks / slots, rest = (blocks - full * slots + 255) / 256;  // rest: blocks per CU of the last round
    const float tr = t.occ > 1 ? t.t1 + (t.tf - t.t1) * (float)(rest - 1) / (float)(t.occ - 1) : t.t1;
    // (one block of 8 waves fills a CU: its rounds overlap only at their ends)
    const float us = (float)full * (nk * t.tf + t.eb) + (rest > 0 ? nk * tr + t.eb : 0.f);
    if (best < 0 || us < tbest) {
      best = i;
      tbest = us;
    }
  }
  return best;
}

static bool launch_tile64(const GemmArgs& a, hipStream_t s) {
  if (loader_mode(a, 64) == 0) return false;
  // Short-K GEGLU projections are as long in their epilogue (some 25 vector
  // instructions per output) as in their products, so two blocks per CU, one
  // in each, beat the deeper stages: K = 320, 196608 x 2560 564 against 622 us,
  // K = 640, 10240 x 5120 100 against 106 us (K = 1280 347 against 333).
  if (a.epi.geglu && a.K <= 640 && (long)((a.M + 255) / 256) * (a.N / 160) >= 512 &&
      launch_dma<256, 160, 4, 1, 32, 3, 2>(a, s))
    return true;
  // Short-K 1x1 layers of 128-column tiles spend their time in loads, epilogue and
  // stores, which two blocks per CU overlap (the 32-deep tile; a 1x1 layer has the
  // same bits in either depth): 64-deep choice and this one 98304 x 128 x 128 26.3
  // and 24.0 us, 65536 x 256 x 256 34.0 and 30.5; below the stated grid 65536 x 128
  // x 128 18.7 and 22.1, at K = 512 196608 x 512 x 512 equal.  (At the widths that
  // are multiples of 160 it depends on the surroundings: 49152 x 960 x 320 alone
  // 80.7 and 70.6, but in the 48-row step the 196608-row QKV 216 and 222, the query
  // projection 81 and 88.)
  if (a.seg[0].ks == 1 && (a.seg[1].K == 0 || a.seg[1].ks == 1) && !a.epi.geglu && a.ksplit == 1 && a.N % 160 &&
      a.K <= 256 && (long)((a.M + 255) / 256) * (a.N / 128) >= 384 && launch_dma<256, 128, 4, 1, 32, 3, 2>(a, s))
    return true;
  switch (pick_tile64(a.M, a.N, a.K, a.ksplit)) {
    case 0: return launch_dma<64, 64, 2, 2, 64, 4, 2>(a, s);
    case 1: return launch_dma<128, 64, 2, 2, 64, 3, 2>(a, s);
    case 2: return launch_dma<128, 128, 2, 2, 64, 2, 2>(a, s);
    case 3: return launch_dma<128, 160, 4, 1, 64, 2, 2>(a, s);
    case 4: return launch_dma<256, 256, 2, 4, 64, 2, 1>(a, s);
    case 5: return launch_dma<256, 320, 4, 2, 64, 2, 1>(a, s);
    default: return false;
  }
}

// Tile choice: 64-deep tiles (above) where the loader allows them; else the
// widest N tile that divides N, then the tallest M tile that still gives every
// CU about two blocks.  Only the split factor and the stage depth, functions
// of the layer shape, decide a row's K order and so its bits.
hipError_t launch_gemm(DType dt, const GemmArgs& args, hipStream_t s) {
  GemmArgs a = args;
  if (a.ksplit < 1) a.ksplit = 1;
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.ksplit > 1 && (dt != BF16 || !a.partial || a.epi.geglu || a.epi.vt_out || a.epi.out_f32 ||
                       a.N % 160 || loader_mode(a, DKS) == 0))
    return hipErrorInvalidValue;
  if (dt == BF16 && (a.N % 4 || a.epi.ldo % 4 || (a.epi.resid && a.epi.ldr % 4) || (a.epi.geglu && a.N % 32) ||
                     a.epi.qcols % 4))
    return hipErrorInvalidValue;
  if (dt != BF16 && (a.epi.geglu || a.epi.vt_out)) return hipErrorInvalidValue;
  if (a.epi.vt_out && (a.epi.vt_col0 % 8 || a.epi.resid || a.epi.tbias || a.epi.out_f32))
    return hipErrorInvalidValue;
  if (a.epi.rowscale && dt != BF16) return hipErrorInvalidValue;
  if ((long)a.N * a.ldb * (dt == BF16 ? 2 : 4) >= (1L << 31)) return hipErrorInvalidValue;
  // upsample phases (ks 2): bf16, the direct-to-LDS tiles (N % 160) with
  // the uniform-tap loader only
  const bool phased = a.seg[0].ks == 2 || (a.seg[1].K && a.seg[1].ks == 2);
  if (phased && (dt != BF16 || a.N % 160 || loader_mode(a, DKS) != 1 || a.ksplit > 1 || a.seg[1].K))
    return hipErrorInvalidValue;
  if (a.epi.phase && (a.epi.phase > 4 || a.epi.ph_h < 1 || a.epi.ph_w < 1 || a.M % (a.epi.ph_h * a.epi.ph_w) ||
                      a.epi.resid || a.epi.vt_out || a.epi.tbias || a.epi.geglu))
    return hipErrorInvalidValue;
  if (dt == BF16) {
    auto nblk = [&](int bm, int bn) { return (long)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
    const long want = 2 * 256;
    if (launch_tile64(a, s)) {
    } else if (a.N % 160 == 0) {
      // 32-deep stages: 256x160 tiles, three of them (2 x 80.9 KB of LDS: two
      // blocks per CU); otherwise register-staged 64-deep tiles, one block per CU
      if (a.ksplit == 1 && nblk(256, 160) < 256 && launch_dma<64, 160, 2, 1, 32, 2, 4>(a, s)) {
        // short M: 64-row tiles, four blocks per CU
      } else if (launch_dma<256, 160, 4, 1, 32, 3, 2>(a, s)) {
      } else if (nblk(256, 160) >= want) {  // (mode 0: the direct-to-LDS tiles take every other layer of these widths)
        gemm_bf16_kernel<256, 160, 64, 4, 1, 0, 1><<<dim3((unsigned)nblk(256, 160)), dim3(256), 0, s>>>(a);
      } else {
        gemm_bf16_kernel<128, 160, 64, 4, 1, 0, 1><<<dim3((unsigned)nblk(128, 160)), dim3(256), 0, s>>>(a);
      }
    } else if (a.N % 128 == 0 && a.ksplit == 1 && launch_dma<256, 128, 4, 1, 32, 3, 2>(a, s)) {
      // widths that are multiples of 128 but not of 160, channels of 32 but not
      // of 64: 256x128 tiles, waves of 64x128
    } else if (a.N % 128 == 0 || a.N > 64) {
      if (nblk(256, 128) >= want)
        launch_bf16<256, 128, 64, 2, 2>(a, s);
      else if (nblk(128, 128) >= want)
        launch_bf16<128, 128, 64, 2, 2>(a, s);
      else
        launch_bf16<64, 128, 64, 2, 2>(a, s);
    } else if (a.N > 32) {
      launch_bf16<128, 64, 64, 4, 1>(a, s);
    } else {
      launch_bf16<256, 32, 64, 4, 1>(a, s);
    }
  } else {
    if (a.K >= 256)
      launch_f32<8>(a, s);
    else if (a.K > 64)
      launch_f32<4>(a, s);
    else
      launch_f32<2>(a, s);
  }
  return hipGetLastError();
}

}  // namespace sd
