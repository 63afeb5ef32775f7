// Memory-bound kernels of the step: row packing, time-embedding inputs and
// small-M MLP, GroupNorm statistics, LayerNorm, GEGLU and the fused CFG
// combine + DDIM update.
#include <map>
#include <mutex>

#include "device_common.h"
#include "kernels.h"

namespace sd {

// ------------------------------------------------------------ row packing
// x0[row, p, c] = latents[row_req[row], c, p] for c < lc, 0 for lc <= c < cpad.
template <typename T>
__global__ void pack_latents_kernel(const float* lat, T* x0, int rows, int lc, int hw, int cpad,
                                    const int* row_req) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)rows * hw) return;
  const int row = (int)(i / hw), p = (int)(i - (long)row * hw);
  const int r = row_req[row];
  if (sizeof(T) == 2 && cpad % 8 == 0) {  // 16-byte runs of 8 channels
    for (int c0 = 0; c0 < cpad; c0 += 8) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = c0 + e < lc ? lat[((long)r * lc + c0 + e) * hw + p] : 0.f;
      store8f(x0 + i * cpad + c0, v);
    }
    return;
  }
  for (int c = 0; c < cpad; ++c) {
    const float v = c < lc ? lat[((long)r * lc + c) * hw + p] : 0.f;
    x0[i * cpad + c] = from_f<T>(v);
  }
}

hipError_t launch_pack_latents(DType dt, const float* lat, void* x0, int rows, int lc, int hw,
                               int cpad, const int* row_req, hipStream_t s) {
  const long n = (long)rows * hw;
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (dt == BF16)
    pack_latents_kernel<bf16><<<blocks, 256, 0, s>>>(lat, (bf16*)x0, rows, lc, hw, cpad, row_req);
  else
    pack_latents_kernel<float><<<blocks, 256, 0, s>>>(lat, (float*)x0, rows, lc, hw, cpad, row_req);
  return hipGetLastError();
}

__global__ void copy_rows_kernel(uint4* base, long row_vecs, int dst0, const int* src_rows) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= row_vecs) return;
  const int r = blockIdx.y;
  base[(long)(dst0 + r) * row_vecs + i] = base[(long)src_rows[r] * row_vecs + i];
}

hipError_t launch_copy_rows(void* base, long row_bytes, int dst0, int n, const int* src_rows, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (row_bytes % 16) return hipErrorInvalidValue;
  const long vecs = row_bytes / 16;
  copy_rows_kernel<<<dim3((unsigned)((vecs + 255) / 256), (unsigned)n), 256, 0, s>>>((uint4*)base, vecs, dst0,
                                                                                      src_rows);
  return hipGetLastError();
}

// ------------------------------------------------------ time-embedding inputs
// Sinusoid [cos(t f_i) | sin(t f_i)], f_i = 10000^(-i/half), evaluated in
// fp64 so the argument t f_i (up to ~1e3 rad) keeps full fp32 accuracy;
// thread `part` of `parts` takes i = part, part + parts, ...
__device__ inline void sinusoid(double t, int dim, float* out, int part = 0, int parts = 1) {
  const int half = dim / 2;
  for (int i = part; i < half; i += parts) {
    const double f = exp(-9.210340371976184 * (double)i / (double)half);  // ln(1e4)
    double sv, cv;
    sincos(t * f, &sv, &cv);
    out[i] = (float)cv;
    out[half + i] = (float)sv;
  }
}

__global__ void time_inputs_kernel(const float* row_t, int rows, int temb_in, float* e,
                                   const float* pooled_cond, const float* pooled_uncond,
                                   const int* row_req, const int* row_branch, int pooled_dim,
                                   const float* time_ids, int n_ids, int id_dim, float* a) {
  const int row = blockIdx.x;
  if (row >= rows) return;
  sinusoid((double)row_t[row], temb_in, e + (long)row * temb_in, threadIdx.x, blockDim.x);
  if (a) {
    const int add_in = pooled_dim + n_ids * id_dim;
    float* ar = a + (long)row * add_in;
    const float* pooled = row_branch[row] ? pooled_uncond : pooled_cond + (long)row_req[row] * pooled_dim;
    for (int i = threadIdx.x; i < pooled_dim; i += blockDim.x) ar[i] = pooled[i];
    for (int id = 0; id < n_ids; ++id)
      sinusoid((double)time_ids[id], id_dim, ar + pooled_dim + id * id_dim, threadIdx.x, blockDim.x);
  }
}

hipError_t launch_time_inputs(const float* row_t, int rows, int temb_in, float* e,
                              const float* pooled_cond, const float* pooled_uncond,
                              const int* row_req, const int* row_branch, int pooled_dim,
                              const float* time_ids_dev, int n_ids, int id_dim, float* a,
                              hipStream_t s) {
  if (rows == 0) return hipSuccess;
  time_inputs_kernel<<<rows, 64, 0, s>>>(row_t, rows, temb_in, e, pooled_cond, pooled_uncond,
                                         row_req, row_branch, pooled_dim, time_ids_dev, n_ids,
                                         id_dim, a);
  return hipGetLastError();
}

// ---------------------------------------------------------- small-M linear
// out[m, n] = act_out(sum_k act_in(in[m, k]) W[n, k] + bias[n] + add[m, n])
// for a few rows (the per-request time embedding: M = requests).  The
// weights are the traffic: each wave owns 4 columns and streams their rows
// with K spread over the lanes (lane l takes k = 4 l .. 4 l + 3 of each
// 256-wide chunk), so every weight load is one contiguous run per column.
// The input rows (32 per pass) are staged in LDS a chunk at a time and each
// 16-byte read of them feeds 16 FMAs (4 columns x 4 k).  The 4 x 32 partial
// dot products per lane are then summed across the wave by halving: six
// exchange steps leave lane l with entries 2 l and 2 l + 1 (column l / 16,
// rows 2 l % 32 and + 1), which it finishes and stores.
namespace sm {
constexpr int MB = 32, KC = 256, CPW = 4, NWV = 4;  // CPW * MB = 128 partial sums per lane
}

template <typename TW>
__device__ inline void load4w(const TW* p, float w[4]);
template <>
__device__ inline void load4w<bf16>(const bf16* p, float w[4]) {
  const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
  w[0] = (float)v[0]; w[1] = (float)v[1]; w[2] = (float)v[2]; w[3] = (float)v[3];
}
template <>
__device__ inline void load4w<float>(const float* p, float w[4]) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
}

template <typename TW>
__global__ __launch_bounds__(256) void linear_smallm_kernel(const float* in, int M, int K, const TW* W,
                                                            const float* bias, const float* add,
                                                            float* out, int N, int silu_in,
                                                            int silu_out) {
  using namespace sm;
  __shared__ __attribute__((aligned(16))) float xs[MB][KC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = (blockIdx.x * NWV + wave) * CPW;  // the wave's first column
  const int m0 = blockIdx.y * MB;
  const int mrows = min(MB, M - m0);
  float acc[CPW * MB];  // [column][row]
#pragma unroll
  for (int i = 0; i < CPW * MB; ++i) acc[i] = 0.f;
  for (int k0 = 0; k0 < K; k0 += KC) {
    __syncthreads();
    for (int idx = tid; idx < MB * (KC / 4); idx += 256) {
      const int m = idx / (KC / 4), kk = (idx - m * (KC / 4)) * 4;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m < mrows && k0 + kk < K) {
        v = *reinterpret_cast<const float4*>(in + (long)(m0 + m) * K + k0 + kk);
        if (silu_in) {
          v.x = silu_f(v.x); v.y = silu_f(v.y); v.z = silu_f(v.z); v.w = silu_f(v.w);
        }
      }
      *reinterpret_cast<float4*>(&xs[m][kk]) = v;
    }
    __syncthreads();
    const int k = k0 + 4 * lane;
    float w[CPW][4];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      if (k < K && n0 + c < N) {
        load4w<TW>(W + (long)(n0 + c) * K + k, w[c]);
      } else {
        w[c][0] = w[c][1] = w[c][2] = w[c][3] = 0.f;
      }
    }
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const float4 x = *reinterpret_cast<const float4*>(&xs[m][4 * lane]);
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        float t = acc[c * MB + m];
        t = fmaf(x.x, w[c][0], t);
        t = fmaf(x.y, w[c][1], t);
        t = fmaf(x.z, w[c][2], t);
        t = fmaf(x.w, w[c][3], t);
        acc[c * MB + m] = t;
      }
    }
  }
  // Sum over the wave by halving: at the step of lane bit b, a lane keeps
  // the half of its live entries selected by that bit and adds its
  // partner's copy of the same half.
#pragma unroll
  for (int st = 0; st < 6; ++st) {
    const int h = (CPW * MB) >> (st + 1);  // entries kept after this step
    const int off = 32 >> st;
    const bool hi = (lane & off) != 0;
#pragma unroll
    for (int i = 0; i < CPW * MB / 2; ++i) {
      if (i < h) {
        const float keep = hi ? acc[i + h] : acc[i];
        const float give = hi ? acc[i] : acc[i + h];
        acc[i] = keep + __shfl_xor(give, off, 64);
      }
    }
  }
  // lane l now holds entries 2 l, 2 l + 1: column 2 l / MB, rows 2 l % MB, + 1
  static_assert(CPW * MB == 128, "the halving leaves two entries per lane");
  const int n = n0 + 2 * lane / MB;
  if (n >= N) return;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int m = (2 * lane) % MB + e;
    if (m < mrows) {
      float v = acc[e] + (bias ? bias[n] : 0.f) + (add ? add[(long)(m0 + m) * N + n] : 0.f);
      if (silu_out) v = silu_f(v);
      out[(long)(m0 + m) * N + n] = v;
    }
  }
}

// Adds up H entries per lane over the wave by halving: a step keeps the half of
// a lane's entries that the lane bit OFF selects and adds the partner's copy of
// it, until one entry is left.
template <int H, int OFF, int E>
__device__ __forceinline__ void halve_entries(float (&acc)[E], int lane) {
  if constexpr (H > 1) {
    const bool hi = (lane & OFF) != 0;
#pragma unroll
    for (int i = 0; i < H / 2; ++i) {
      const float keep = hi ? acc[i + H / 2] : acc[i], give = hi ? acc[i] : acc[i + H / 2];
      acc[i] = keep + __shfl_xor(give, OFF, 64);
    }
    halve_entries<H / 2, OFF / 2>(acc, lane);
  }
}

// The same for at most MB rows (2, 4 or 8; a request or a few): the 32-row
// form multiplies and exchanges its empty rows too, and loads a chunk of
// weights between two barriers.  Here all of x is staged once and the weight
// loads of four chunks are in flight.  The order of the sums is that of the
// 32-row form (each lane's chunks in order, then lanes 32, 16, .. 1 apart), so
// a row's bits do not depend on which form runs.  The three launches of a
// step for one guided request of the SD-1.5 UNet: 101 -> 44 us.  Five blocks per
// CU (96 registers) up to 4 rows: 2 rows of 1280 x 20160 20.0 us with four.
template <typename TW, int MB>
__global__ __launch_bounds__(256, MB == 8 ? 4 : 5) void linear_fewm_kernel(const float* in, int M, int K, const TW* W,
                                                          const float* bias, const float* add, float* out, int N,
                                                          int silu_in, int silu_out) {
  using namespace sm;
  constexpr int U = 4;  // chunks in flight
  extern __shared__ __attribute__((aligned(16))) float xf[];  // [MB][K rounded up to KC]
  const int KR = (K + KC - 1) / KC * KC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = (blockIdx.x * NWV + wave) * CPW;
  for (int idx = tid; idx < MB * (KR / 4); idx += 256) {
    const int m = idx / (KR / 4), kk = (idx - m * (KR / 4)) * 4;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (m < M && kk < K) {
      v = *reinterpret_cast<const float4*>(in + (long)m * K + kk);
      if (silu_in) {
        v.x = silu_f(v.x); v.y = silu_f(v.y); v.z = silu_f(v.z); v.w = silu_f(v.w);
      }
    }
    *reinterpret_cast<float4*>(&xf[m * KR + kk]) = v;
  }
  __syncthreads();
  constexpr int E = CPW * MB;  // entries (column, row) = c * MB + m
  float acc[E];
#pragma unroll
  for (int i = 0; i < E; ++i) acc[i] = 0.f;
  for (int k0 = 0; k0 < K; k0 += U * KC) {
    float w[U][CPW][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        const int k = k0 + u * KC + 4 * lane;
        if (k < K && n0 + c < N)
          load4w<TW>(W + (long)(n0 + c) * K + k, w[u][c]);
        else
          w[u][c][0] = w[u][c][1] = w[u][c][2] = w[u][c][3] = 0.f;
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * KC + 4 * lane;
      if (k0 + u * KC < K) {
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const float4 x = *reinterpret_cast<const float4*>(&xf[m * KR + k]);
#pragma unroll
          for (int c = 0; c < CPW; ++c) {
            float t = acc[c * MB + m];
            t = fmaf(x.x, w[u][c][0], t);
            t = fmaf(x.y, w[u][c][1], t);
            t = fmaf(x.z, w[u][c][2], t);
            t = fmaf(x.w, w[u][c][3], t);
            acc[c * MB + m] = t;
          }
        }
      }
    }
  }
  // (a full exchange of each of the E entries took 6 E steps: 8 rows of 32 x 128
  // 12.7 us, now 4.4, the 32-row form 8.8)
  halve_entries<E, 32>(acc, lane);
  constexpr int LPE = 64 / E;  // lanes that hold the same entry, lane / LPE
  float v = acc[0];
#pragma unroll
  for (int o = LPE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int n = n0 + lane / (LPE * MB), m = lane / LPE % MB;
  if (lane % LPE == 0 && n < N && m < M) {
    v = v + (bias ? bias[n] : 0.f) + (add ? add[(long)m * N + n] : 0.f);
    if (silu_out) v = silu_f(v);
    out[(long)m * N + n] = v;
  }
}

template <typename TW>
static bool launch_linear_fewm(const float* in, int M, int K, const TW* W, const float* bias, const float* add,
                               float* out, int N, int silu_in, int silu_out, hipStream_t s) {
  const int mb = M <= 2 ? 2 : (M <= 4 ? 4 : 8);
  const size_t lds = (size_t)mb * ((K + sm::KC - 1) / sm::KC * sm::KC) * sizeof(float);
  if (M > 8 || lds > 64 * 1024) return false;
  const unsigned blocks = (unsigned)((N + sm::CPW * sm::NWV - 1) / (sm::CPW * sm::NWV));
  if (mb == 2)
    linear_fewm_kernel<TW, 2><<<blocks, 256, lds, s>>>(in, M, K, W, bias, add, out, N, silu_in, silu_out);
  else if (mb == 4)
    linear_fewm_kernel<TW, 4><<<blocks, 256, lds, s>>>(in, M, K, W, bias, add, out, N, silu_in, silu_out);
  else
    linear_fewm_kernel<TW, 8><<<blocks, 256, lds, s>>>(in, M, K, W, bias, add, out, N, silu_in, silu_out);
  return true;
}

hipError_t launch_linear_smallm(DType wdt, const float* in, int M, int K, const void* W,
                                const float* bias, const float* add, float* out, int N,
                                int silu_in, int silu_out, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (K <= 0 || K % 4) return hipErrorInvalidValue;
  if (wdt == BF16 ? launch_linear_fewm(in, M, K, (const bf16*)W, bias, add, out, N, silu_in, silu_out, s)
                  : launch_linear_fewm(in, M, K, (const float*)W, bias, add, out, N, silu_in, silu_out, s))
    return hipGetLastError();
  const dim3 grid((unsigned)((N + sm::CPW * sm::NWV - 1) / (sm::CPW * sm::NWV)), (unsigned)((M + sm::MB - 1) / sm::MB));
  if (wdt == BF16)
    linear_smallm_kernel<bf16><<<grid, 256, 0, s>>>(in, M, K, (const bf16*)W, bias, add, out, N,
                                                    silu_in, silu_out);
  else
    linear_smallm_kernel<float><<<grid, 256, 0, s>>>(in, M, K, (const float*)W, bias, add, out,
                                                     N, silu_in, silu_out);
  return hipGetLastError();
}

// --------------------------------------------------------- GroupNorm stats
// Pixel rows per block of the partial pass: enough threads to stream a
// block's pixels with several 16-byte loads in flight each.
static inline int gn_pp(int cin) {
  const int cv = cin / 8;
  return cv >= 512 ? 1 : 512 / cv;
}

// Splits of an image's pixels (about 16 pixels per thread): 16 measured 7 %
// faster than 8 per launch at the SD-1.5 widths (fewer blocks, the LDS
// reduction amortised over more loads).  At most 128: a batch fills the chip with
// 64, and more blocks only cost it their start and reduction (16 images of
// 128x128x960 101 us with 64 or 128, 111 with 256), but one or two images do not
// (2 of them 30, 20 and 19 us).  From 2^15 pixels on, the VAE decoder's large
// images, which come one or two at a time, at most 256, one block per CU
// (512x512x256 81 us with 64, 28 with 256; eight of 256x256x512 97 and 102).
// A function of the image alone, so its bits do not depend on the batch.
static inline int gn_splits(int hw, int cin, bool few = false) {
  const int s = hw / (gn_pp(cin) * 16), most = few ? 64 : (hw >= (1 << 15) ? 256 : 128);
  return s < 1 ? 1 : (s > most ? most : s);
}

size_t groupnorm_partial_floats(int imgs, int hw, int cin) {
  return (size_t)imgs * gn_splits(hw, cin) * cin * 2;
}

// What the entry point that allocates nothing counts against its scratch
// (64 splits an image at most); a call whose partials exceed the scratch at
// the full split count runs its images in several passes.
size_t groupnorm_noalloc_floats(int imgs, int hw, int cin) {
  return (size_t)imgs * gn_splits(hw, cin, true) * cin * 2;
}

// Pass 1: per (image, split, channel) sum and sum of squares (fp32 over at
// most a few hundred pixels; the finalize pass adds the splits in fp64).
// Thread (pp, cv) reads channels 8 cv .. 8 cv + 7 (one 16-byte load) of
// pixels pp, pp + PP, ..., four at a time so their loads overlap; the
// partial results are reduced over pp in LDS, laid out so that neighbouring
// lanes write and read neighbouring 16-byte pieces (written channel by channel,
// 16 lanes met in each bank: 48 images of 64x64x640 52.4 us, now 44.7).
template <typename T>
__global__ void gn_partial_kernel(const T* src0, int c0, const T* src1, int c1, int hw, int nsplit,
                                  int PP, float* partial) {
  extern __shared__ __attribute__((aligned(16))) float4 red[];  // [PP][4 channel pairs][CV]: sum, squares of each
  const int cin = c0 + c1, CV = cin / 8;
  const int img = blockIdx.y, split = blockIdx.x;
  const int chunk = (hw + nsplit - 1) / nsplit;
  const int p0 = split * chunk, p1 = min(hw, p0 + chunk);
  const int cv = threadIdx.x % CV, pp = threadIdx.x / CV;
  const int c = cv * 8;
  const T* base = c < c0 ? src0 + c : src1 + (c - c0);
  const int ld = c < c0 ? c0 : c1;
  float s[8] = {}, q[8] = {};
  if (pp < PP) {
    for (int p = p0 + pp; p < p1; p += 4 * PP) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int pu = p + u * PP;
        if (pu < p1) {
          load8f(base + ((long)img * hw + pu) * ld, v[u]);
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) v[u][i] = 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          s[i] += v[u][i];
          q[i] = fmaf(v[u][i], v[u][i], q[i]);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      red[(pp * 4 + j) * CV + cv] = make_float4(s[2 * j], q[2 * j], s[2 * j + 1], q[2 * j + 1]);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4 * CV; i += blockDim.x) {
    const int j = i / CV, v = i - j * CV;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < PP; ++k) {
      const float4 r = red[k * 4 * CV + i];
      t.x += r.x; t.y += r.y; t.z += r.z; t.w += r.w;
    }
    float2* o = reinterpret_cast<float2*>(partial + (((long)img * nsplit + split) * cin + 8 * v + 2 * j) * 2);
    o[0] = make_float2(t.x, t.y);
    o[1] = make_float2(t.z, t.w);
  }
}

// Pass 2: per (image, group) mean and rstd in fp64 -> the per-channel affine.
// One block per (group, image), a wave where a lane then adds at most 10
// partials, else four; the loads of a lane's partials are independent, so the
// loop is unrolled to keep them in flight together.
template <int NW>
__global__ __launch_bounds__(64 * NW) void gn_finalize_kernel(const float* partial, int cin, int nsplit, int hw,
                                                              int groups, float eps, const float* gamma,
                                                              const float* beta, float* scale, float* shift) {
  const int g = blockIdx.x, img = blockIdx.y, tid = threadIdx.x;
  const int cpg = cin / groups, n = nsplit * cpg;
  double s = 0.0, q = 0.0;
#pragma unroll 8
  for (int idx = tid; idx < n; idx += 64 * NW) {
    const int sp = idx / cpg, ch = g * cpg + (idx - sp * cpg);
    const float2 v = *reinterpret_cast<const float2*>(partial + (((long)img * nsplit + sp) * cin + ch) * 2);
    s += v.x;
    q += v.y;
  }
  s = wave_sum_d(s);
  q = wave_sum_d(q);
  if constexpr (NW > 1) {
    __shared__ double red[2][NW];
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = s;
      red[1][tid >> 6] = q;
    }
    __syncthreads();
    s = q = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      s += red[0][w];
      q += red[1][w];
    }
  }
  const double cnt = (double)cpg * hw;
  const double mean = s / cnt;
  double var = q / cnt - mean * mean;
  if (var < 0.0) var = 0.0;
  const float rstd = (float)(1.0 / sqrt(var + (double)eps));
  for (int ch = g * cpg + tid; ch < (g + 1) * cpg; ch += 64 * NW) {
    const float sc = gamma[ch] * rstd;
    scale[(long)img * cin + ch] = sc;
    shift[(long)img * cin + ch] = beta[ch] - (float)mean * sc;
  }
}

hipError_t launch_groupnorm_stats(DType dt, const void* src0, int c0, const void* src1, int c1,
                                  int imgs, int hw, int groups, float eps, const float* gamma,
                                  const float* beta, float* partial, float* scale, float* shift,
                                  hipStream_t s) {
  if (imgs == 0) return hipSuccess;
  const int cin = c0 + c1, CV = cin / 8;
  const int PP = gn_pp(cin);
  const int nsplit = gn_splits(hw, cin);
  const int threads = CV * PP;
  const size_t lds = (size_t)PP * cin * 2 * sizeof(float);
  if (threads > 1024 || lds > 64 * 1024) return hipErrorInvalidValue;
  dim3 grid(nsplit, imgs);
  if (dt == BF16)
    gn_partial_kernel<bf16><<<grid, threads, lds, s>>>((const bf16*)src0, c0, (const bf16*)src1, c1,
                                                       hw, nsplit, PP, partial);
  else
    gn_partial_kernel<float><<<grid, threads, lds, s>>>((const float*)src0, c0, (const float*)src1,
                                                        c1, hw, nsplit, PP, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nsplit * (cin / groups) <= 10 * 64)
    gn_finalize_kernel<1><<<dim3(groups, imgs), 64, 0, s>>>(partial, cin, nsplit, hw, groups, eps, gamma, beta,
                                                            scale, shift);
  else
    gn_finalize_kernel<4><<<dim3(groups, imgs), 256, 0, s>>>(partial, cin, nsplit, hw, groups, eps, gamma, beta,
                                                             scale, shift);
  return hipGetLastError();
}

// Library-owned scratch for the GroupNorm partial sums of callers that
// cannot allocate device memory (synerdiff_op_groupnorm_stats_noalloc):
// one array per device, held until the process ends.  In host code the name
// `gn_scratch` stands for a host-side shadow, not a device address, so host
// code never passes it to a kernel: it takes the device address from
// hipGetSymbolAddress, once per device (with that device current), and uses
// that pointer everywhere.  The partial-sum kernel writes every element the
// finalize kernel reads, so nothing needs clearing between calls; calls
// that overlap in time on one device share the array and race.
constexpr size_t GN_SCRATCH_FLOATS = (size_t)1 << 22;  // 16 MiB
static __device__ __align__(256) float gn_scratch[GN_SCRATCH_FLOATS];

size_t groupnorm_scratch_floats_max() { return GN_SCRATCH_FLOATS; }

hipError_t groupnorm_scratch(float** out) {
  static std::mutex mu;
  static std::map<int, float*> by_device;
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  auto it = by_device.find(dev);
  if (it == by_device.end()) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(gn_scratch));
    if (e != hipSuccess) return e;
    it = by_device.emplace(dev, static_cast<float*>(p)).first;
  }
  *out = it->second;
  return hipSuccess;
}

// Pass 3: y = act(x * scale + shift) into a materialised [imgs, hw, cin]
// tensor (the concat of the two sources when there are two); one 8-channel
// vector per thread, blockIdx.y the image (32-bit index arithmetic).
template <typename T>
__global__ void gn_apply_kernel(const T* src0, int c0, const T* src1, int c1, const float* scale,
                                const float* shift, T* out, int hw, int silu) {
  const int cin = c0 + c1, CV = cin / 8;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= hw * CV) return;
  const int img = blockIdx.y;
  const int p = i / CV;
  const int c = (i - p * CV) * 8;
  const long pix = (long)img * hw + p;
  float v[8], sc[8], sh[8];
  if (c < c0)
    load8f(src0 + pix * c0 + c, v);
  else
    load8f(src1 + pix * c1 + (c - c0), v);
  load8f(scale + (long)img * cin + c, sc);
  load8f(shift + (long)img * cin + c, sh);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v[k] = v[k] * sc[k] + sh[k];
    if (silu) v[k] = silu_f(v[k]);
  }
  store8f(out + pix * cin + c, v);
}

hipError_t launch_groupnorm_apply(DType dt, const void* src0, int c0, const void* src1, int c1, int imgs,
                                  int hw, const float* scale, const float* shift, int silu, void* out,
                                  hipStream_t s) {
  const long per_img = (long)hw * ((c0 + c1) / 8);
  if (imgs == 0 || per_img == 0) return hipSuccess;
  if (per_img >= (1L << 31) || imgs > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((per_img + 255) / 256), (unsigned)imgs);
  if (dt == BF16)
    gn_apply_kernel<bf16><<<grid, 256, 0, s>>>((const bf16*)src0, c0, (const bf16*)src1, c1, scale, shift,
                                               (bf16*)out, hw, silu);
  else
    gn_apply_kernel<float><<<grid, 256, 0, s>>>((const float*)src0, c0, (const float*)src1, c1, scale, shift,
                                                (float*)out, hw, silu);
  return hipGetLastError();
}

// Small images (at most 5120 four-channel vectors per (image, group), the
// 16x16 and 8x8 levels of the SD UNets): statistics and apply in one kernel,
// one block per (group, image).  The block keeps its group's values in
// registers (E vectors of W = 8 channels per thread, 16-byte loads, where
// the group width and the sources' widths are multiples of 8, else W = 4
// and 8-byte loads; a group's channels are consecutive, a vector never
// straddles the two sources), adds the fp32 per-thread sums in fp64 across
// the block, and writes act(x * scale + shift) with the same per-channel
// scale and shift as the three-pass form.  One launch instead of three, and
// one read of the input.
template <typename T, int W> struct bvec;
template <> struct bvec<bf16, 4> { typedef bf16x4 type; };
template <> struct bvec<bf16, 8> { typedef bf16x8 type; };
template <> struct bvec<float, 4> { typedef f32x4 type; };

template <typename T, int E, int W>
__global__ __launch_bounds__(256) void gn_fused_kernel(const T* src0, int c0, const T* src1, int c1,
                                                       int hw, int groups, float eps, const float* gamma,
                                                       const float* beta, int silu, T* out) {
  typedef typename bvec<T, W>::type vec;
  const int g = blockIdx.x, img = blockIdx.y, tid = threadIdx.x;
  const int cin = c0 + c1, cpg = cin / groups, V = cpg / W, n = hw * V, cg = g * cpg;
  float v[E][W];
  float s = 0.f, q = 0.f;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = tid + 256 * e;
    if (i < n) {
      const int p = i / V, c = cg + (i - p * V) * W;
      const T* src = c < c0 ? src0 + ((long)img * hw + p) * c0 + c : src1 + ((long)img * hw + p) * c1 + (c - c0);
      const vec a = *reinterpret_cast<const vec*>(src);
#pragma unroll
      for (int k = 0; k < W; ++k) {
        v[e][k] = (float)a[k];
        s += v[e][k];
        q = fmaf(v[e][k], v[e][k], q);
      }
    }
  }
  __shared__ double red[2][4];
  const double ws = wave_sum_d((double)s), wq = wave_sum_d((double)q);
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = ws;
    red[1][tid >> 6] = wq;
  }
  __syncthreads();
  const double ts = red[0][0] + red[0][1] + red[0][2] + red[0][3];
  const double tq = red[1][0] + red[1][1] + red[1][2] + red[1][3];
  const double cnt = (double)cpg * hw;
  const double mean = ts / cnt;
  double var = tq / cnt - mean * mean;
  if (var < 0.0) var = 0.0;
  const float rstd = (float)(1.0 / sqrt(var + (double)eps));
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = tid + 256 * e;
    if (i < n) {
      const int p = i / V, c = cg + (i - p * V) * W;
      vec o;
#pragma unroll
      for (int k = 0; k < W; ++k) {
        const float sc = gamma[c + k] * rstd;
        float y = v[e][k] * sc + (beta[c + k] - (float)mean * sc);
        if (silu) y = silu_f(y);
        o[k] = (T)y;
      }
      *reinterpret_cast<vec*>(out + ((long)img * hw + p) * cin + c) = o;
    }
  }
}

bool groupnorm_fused_ok(DType dt, int c0, int c1, int hw, int groups) {
  const int cin = c0 + c1;
  if (groups <= 0 || cin % groups || c0 % 4 || c1 % 4) return false;
  const int cpg = cin / groups;
  return cpg % 4 == 0 && (long)hw * (cpg / 4) <= 256L * 20;
}

hipError_t launch_groupnorm_fused(DType dt, const void* src0, int c0, const void* src1, int c1, int imgs, int hw,
                                  int groups, float eps, const float* gamma, const float* beta, int silu, void* out,
                                  hipStream_t s) {
  if (!groupnorm_fused_ok(dt, c0, c1, hw, groups) || imgs > 65535) return hipErrorInvalidValue;
  if (imgs == 0 || hw == 0) return hipSuccess;
  const int cpg = (c0 + c1) / groups;
  const dim3 grid(groups, imgs);
  if (dt == F32) {  // vectors of 4 channels (16 bytes)
    const float *a = (const float*)src0, *b = (const float*)src1;
    float* o = (float*)out;
    const long n = (long)hw * (cpg / 4);  // <= 5120
    if (n <= 256 * 4)
      gn_fused_kernel<float, 4, 4><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
    else
      gn_fused_kernel<float, 20, 4><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
    return hipGetLastError();
  }
  const bf16 *a = (const bf16*)src0, *b = (const bf16*)src1;
  bf16* o = (bf16*)out;
  if (cpg % 8 == 0 && c0 % 8 == 0 && c1 % 8 == 0) {
    const long n = (long)hw * (cpg / 8);  // <= 2560
    if (n <= 256 * 4)
      gn_fused_kernel<bf16, 4, 8><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
    else if (n <= 256 * 8)
      gn_fused_kernel<bf16, 8, 8><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
    else
      gn_fused_kernel<bf16, 10, 8><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
  } else {
    const long n = (long)hw * (cpg / 4);  // <= 5120
    if (n <= 256 * 4)
      gn_fused_kernel<bf16, 4, 4><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
    else if (n <= 256 * 8)
      gn_fused_kernel<bf16, 8, 4><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
    else
      gn_fused_kernel<bf16, 20, 4><<<grid, 256, 0, s>>>(a, c0, b, c1, hw, groups, eps, gamma, beta, silu, o);
  }
  return hipGetLastError();
}

// -------------------------------------------------------------- LayerNorm
// One wave per token; the token's C values stay in registers (C <= 2048).
template <typename T>
__global__ __launch_bounds__(256) void layernorm_kernel(const T* x, T* y, long tokens, int C,
                                                        const float* gamma, const float* beta,
                                                        float eps) {
  constexpr int MAXV = 4;
  const long t = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= tokens) return;
  const int CV = C / 8;
  float v[MAXV][8];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int cv = lane + 64 * j;
    if (cv < CV) {
      load8f(x + t * C + cv * 8, v[j]);
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[j][i];
    }
  }
  const float mean = wave_sum(s) / C;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < MAXV; ++j)
    if (lane + 64 * j < CV)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = v[j][i] - mean;
        q = fmaf(d, d, q);
      }
  const float rstd = rsqrtf(wave_sum(q) / C + eps);
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    const int cv = lane + 64 * j;
    if (cv < CV) {
      float g[8], b[8], o[8];
      load8f(gamma + cv * 8, g);
      load8f(beta + cv * 8, b);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = (v[j][i] - mean) * rstd * g[i] + b[i];
      store8f(y + t * C + cv * 8, o);
    }
  }
}

hipError_t launch_layernorm(DType dt, const void* x, void* y, long tokens, int C, const float* gamma,
                            const float* beta, float eps, hipStream_t s) {
  if (tokens == 0) return hipSuccess;
  if (C % 8 || C > 2048) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)((tokens + 3) / 4);
  if (dt == BF16)
    layernorm_kernel<bf16><<<blocks, 256, 0, s>>>((const bf16*)x, (bf16*)y, tokens, C, gamma, beta, eps);
  else
    layernorm_kernel<float><<<blocks, 256, 0, s>>>((const float*)x, (float*)y, tokens, C, gamma, beta,
                                                   eps);
  return hipGetLastError();
}

// The scale 1 / sqrt(var + eps) alone, for the projections that fold the
// rest of the normalisation into their weights.  One wave takes U
// consecutive tokens (lane l holds vectors l, l + 64, ... of each), issues
// all of their loads before the first reduction, then runs the two passes
// over its registers per token; the per-token sums are the same as with one
// token per wave.  U tokens of C <= 512 channels (MV = 1) are 4 loads per
// lane in flight: about 10 % faster than one token per wave.
template <typename T, int MV, int U>
__global__ __launch_bounds__(256) void layernorm_rstd_kernel(const T* x, float* rstd, long tokens, int C,
                                                             float eps) {
  const long t0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * U;
  const int lane = threadIdx.x & 63;
  if (t0 >= tokens) return;
  const int CV = C / 8;
  float v[U][MV][8];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < MV; ++j) {
      const int cv = lane + 64 * j;
      if (cv < CV && t0 + u < tokens) {
        load8f(x + (t0 + u) * C + cv * 8, v[u][j]);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[u][j][i] = 0.f;
      }
    }
  float mean[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < MV; ++j)
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[u][j][i];
    mean[u] = wave_sum(s) / C;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < MV; ++j)
      if (lane + 64 * j < CV)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float d = v[u][j][i] - mean[u];
          q = fmaf(d, d, q);
        }
    const float r = rsqrtf(wave_sum(q) / C + eps);
    if (lane == 0 && t0 + u < tokens) rstd[t0 + u] = r;
  }
}

// The same scale with L lanes per token (64 / L tokens per wave), each lane
// holding NV vectors of 8 (C = 8 L NV): every lane loads, and a token's
// sums take log2(L) exchanges within its lane group.  Used where C / 8
// splits evenly (C = 320, 640, 1280, ...), so that no lane idles as with a
// wave per token at C = 320.
template <typename T, int L, int NV>
__global__ __launch_bounds__(256) void layernorm_rstd_grp_kernel(const T* x, float* rstd, long tokens, float eps) {
  constexpr int C = 8 * L * NV;
  const int lane = threadIdx.x & 63, g = lane % L;
  const long t = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 / L) + lane / L;
  float v[NV][8];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (t < tokens) {
      load8f(x + t * C + (g + L * j) * 8, v[j]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[j][i] = 0.f;
    }
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) s += v[j][i];
#pragma unroll
  for (int o = L / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  const float mean = s / C;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float d = v[j][i] - mean;
      q = fmaf(d, d, q);
    }
#pragma unroll
  for (int o = L / 2; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
  if (g == 0 && t < tokens) rstd[t] = rsqrtf(q / C + eps);
}

template <typename T, int L, int NV>
static void launch_ln_rstd_grp(const void* x, float* rstd, long tokens, float eps, hipStream_t s) {
  constexpr long TPB = 4 * (64 / L);  // tokens per block
  const unsigned blocks = (unsigned)((tokens + TPB - 1) / TPB);
  layernorm_rstd_grp_kernel<T, L, NV><<<blocks, 256, 0, s>>>((const T*)x, rstd, tokens, eps);
}

template <typename T, int MV, int U>
static void launch_ln_rstd(const void* x, float* rstd, long tokens, int C, float eps, hipStream_t s) {
  const unsigned blocks = (unsigned)((tokens + 4 * U - 1) / (4 * U));
  layernorm_rstd_kernel<T, MV, U><<<blocks, 256, 0, s>>>((const T*)x, rstd, tokens, C, eps);
}

// MV = vectors of 8 per lane and token (C / 512 rounded up); U = 4 tokens
// per wave for C <= 512, 2 above (4 loads per lane in flight at C = 640).
template <typename T>
static void launch_ln_rstd_t(const void* x, float* rstd, long tokens, int C, float eps, hipStream_t s) {
  switch (C) {  // the SD / SDXL widths: lane groups of five vectors per lane
    case 320: launch_ln_rstd_grp<T, 8, 5>(x, rstd, tokens, eps, s); return;
    case 640: launch_ln_rstd_grp<T, 16, 5>(x, rstd, tokens, eps, s); return;
    case 1280: launch_ln_rstd_grp<T, 32, 5>(x, rstd, tokens, eps, s); return;
    default: break;
  }
  switch ((C / 8 + 63) / 64) {
    case 1: launch_ln_rstd<T, 1, 4>(x, rstd, tokens, C, eps, s); break;
    case 2: launch_ln_rstd<T, 2, 2>(x, rstd, tokens, C, eps, s); break;
    case 3: launch_ln_rstd<T, 3, 2>(x, rstd, tokens, C, eps, s); break;
    default: launch_ln_rstd<T, 4, 2>(x, rstd, tokens, C, eps, s); break;
  }
}

hipError_t launch_layernorm_rstd(DType dt, const void* x, float* rstd, long tokens, int C, float eps,
                                 hipStream_t s) {
  if (tokens == 0) return hipSuccess;
  if (C % 8 || C > 2048) return hipErrorInvalidValue;
  if (dt == BF16)
    launch_ln_rstd_t<bf16>(x, rstd, tokens, C, eps, s);
  else
    launch_ln_rstd_t<float>(x, rstd, tokens, C, eps, s);
  return hipGetLastError();
}

// ------------------------------------------------------------------ GEGLU
template <typename T>
__global__ void geglu_kernel(const T* x, T* y, long tokens, int half) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;  // one 8-vector
  const int hv = half / 8;
  if (i >= tokens * hv) return;
  const long t = i / hv;
  const int j = (int)(i - t * hv) * 8;
  float a[8], g[8], o[8];
  load8f(x + t * 2 * half + j, a);
  load8f(x + t * 2 * half + half + j, g);
#pragma unroll
  for (int k = 0; k < 8; ++k) o[k] = a[k] * (0.5f * g[k] * (1.0f + erff(g[k] * 0.70710678118654752f)));
  store8f(y + t * half + j, o);
}

hipError_t launch_geglu(DType dt, const void* x, void* y, long tokens, int half, hipStream_t s) {
  const long n = tokens * (half / 8);
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (dt == BF16)
    geglu_kernel<bf16><<<blocks, 256, 0, s>>>((const bf16*)x, (bf16*)y, tokens, half);
  else
    geglu_kernel<float><<<blocks, 256, 0, s>>>((const float*)x, (float*)y, tokens, half);
  return hipGetLastError();
}

// ------------------------------------------------------ CFG combine + DDIM
// eps = cfg ? eps_u + w (eps_c - eps_u) : eps_c;  x' = A x + B eps.
__global__ void cfg_ddim_kernel(const float* eps_rows, const float* lat_in, float* lat_out,
                                float* eps_out, int n_req, int lc, int hw, const int* req_row_u,
                                const float* req_coef) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)n_req * hw) return;
  const int r = (int)(i / hw), p = (int)(i - (long)r * hw);
  const int ru = req_row_u[r];
  const float A = req_coef[3 * r], B = req_coef[3 * r + 1], w = req_coef[3 * r + 2];
  const float* ec = eps_rows + ((long)r * hw + p) * lc;
  const float* eu = ru >= 0 ? eps_rows + ((long)ru * hw + p) * lc : nullptr;
  for (int c = 0; c < lc; ++c) {
    float e = ec[c];
    if (eu) e = eu[c] + w * (e - eu[c]);
    const long o = ((long)r * lc + c) * hw + p;
    const float x = lat_in[o];
    lat_out[o] = A * x + B * e;
    if (eps_out) eps_out[o] = e;
  }
}

hipError_t launch_cfg_ddim(const float* eps_rows, const float* lat_in, float* lat_out,
                           float* eps_out, int n_req, int lc, int hw, const int* req_row_u,
                           const float* req_coef, hipStream_t s) {
  const long n = (long)n_req * hw;
  if (n == 0) return hipSuccess;
  cfg_ddim_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(eps_rows, lat_in, lat_out, eps_out, n_req,
                                                              lc, hw, req_row_u, req_coef);
  return hipGetLastError();
}

}  // namespace sd
