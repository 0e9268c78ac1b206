// Bandwidth-bound steps of the block: dtype conversion, LayerNorm / RMSNorm
// forward and backward (fused with the residual-gradient add), rotary
// embedding, GELU / SwiGLU forward and backward, column sums for bias
// gradients.  All statistics and transcendental math are fp32.
#include <type_traits>

#include "common.h"

namespace {

// ------------------------------------------------------------------ convert
__global__ void convert_kernel(const void* src, int sdt, void* dst, int ddt, size_t n, const float* scale) {
  const float sc = scale ? *scale : 1.f;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    store_from_f(dst, i, ddt, load_as_f(src, i, sdt) * sc);
}

// ------------------------------------------------------------ gradient scale
// out[0] = 2^e with max|x| * 2^e in (8, 16], out[1] = 2^-e.  Multiplying the
// upstream gradient by out[0] keeps every 16-bit gradient operand of the
// backward pass well inside the fp16 normal range (the matrix cores flush
// fp16 subnormal inputs); results are multiplied by out[1], which is exact.
// A workgroup's maximum (256 threads) into the global one: one atomic per workgroup - with one per wavefront
// the eight thousand atomics on one address took 90 of the kernel's 100 us at 4096 x 4096 elements.  Values
// that are not finite are left out (the scale then comes from the finite ones).
__device__ __forceinline__ void block_amax(float m, unsigned* amax_bits) {
  __shared__ float wave_m[4];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) wave_m[threadIdx.x >> 6] = m <= 3.0e38f ? m : 0.f;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmaxf(fmaxf(wave_m[0], wave_m[1]), fmaxf(wave_m[2], wave_m[3]));
    if (__float_as_uint(m) > __hip_atomic_load(amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(amax_bits, __float_as_uint(m));
  }
}
__global__ void amax_kernel(const void* x, int dt, size_t n, unsigned* amax_bits) {
  float m = 0.f;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    m = fmaxf(m, fabsf(load_as_f(x, i, dt)));
  block_amax(m, amax_bits);
}
__global__ void scale_reset_kernel(float* out) { out[2] = 0.f; }
__global__ void scale_finish_kernel(float* out) {
  const float a = out[2];
  float e = 0.f;
  if (a > 0.f && a <= 3.0e38f) e = fminf(fmaxf(floorf(log2f(16.f / a)), -24.f), 40.f);
  out[0] = exp2f(e);
  out[1] = exp2f(-e);
}

// ---------------------------------------------------------------- norm fwd
// one 256-thread workgroup per row; the row is read once and held in registers
constexpr int NF_MAXCOL = 32;  // d <= 256 * 32
__global__ __launch_bounds__(256) void norm_fwd_kernel(int kind, const float* x, int d,
                                                       const void* gamma, const void* beta,
                                                       int pdt, float eps, void* h, int hdt,
                                                       float* mean, float* rstd) {
  __shared__ float red[16];
  const size_t row = blockIdx.x;
  const float* xr = x + row * d;
  float v[NF_MAXCOL];
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NF_MAXCOL; ++c) {
    const int i = threadIdx.x + c * 256;
    v[c] = i < d ? xr[i] : 0.f;
    s += v[c];
  }
  float mu = 0.f;
  if (kind == 0) mu = block_sum(s, red) / d;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < NF_MAXCOL; ++c) {
    const int i = threadIdx.x + c * 256;
    const float t = i < d ? v[c] - mu : 0.f;
    q += t * t;
  }
  const float var = block_sum(q, red) / d;
  const float r = 1.0f / sqrtf(var + eps);
#pragma unroll
  for (int c = 0; c < NF_MAXCOL; ++c) {
    const int i = threadIdx.x + c * 256;
    if (i < d) {
      float o = (v[c] - mu) * r * load_as_f(gamma, i, pdt);
      if (kind == 0 && beta) o += load_as_f(beta, i, pdt);
      store_from_f(h, row * d + i, hdt, o);
    }
  }
  if (threadIdx.x == 0) {
    if (mean && kind == 0) mean[row] = mu;
    if (rstd) rstd[row] = r;
  }
}

// ---------------------------------------------------------------- norm bwd
// Two kernels.  (1) per-row statistics m1 = mean(dh*gamma), m2 = mean(dh*gamma*xhat),
// one wavefront per row.  (2) dx and the column partial sums: a thread owns 8
// consecutive columns (16-byte loads) and walks NB_ROWS rows, so a workgroup
// covers a 2048-column x NB_ROWS-row patch; its dgamma/dbeta partials go to
// partial[row chunk][2][d] and a last kernel sums them in a fixed order.
constexpr int NB_ROWS = 16;

template <class TD> struct Ld8 {
  static __device__ __forceinline__ void load(const TD* p, float (&v)[8]) {
    typedef typename vec8<TD>::type V8;
    const V8 t = *(const V8*)p;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = to_f(t[i]);
  }
  static __device__ __forceinline__ void store(TD* p, const float (&v)[8]) {
    typedef typename vec8<TD>::type V8;
    V8 t;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = from_f<TD>(v[i]);
    *(V8*)p = t;
  }
};
template <> struct Ld8<float> {
  static __device__ __forceinline__ void load(const float* p, float (&v)[8]) {
    const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
  }
  static __device__ __forceinline__ void store(float* p, const float (&v)[8]) {
    *(f32x4*)p = f32x4{v[0], v[1], v[2], v[3]};
    *(f32x4*)(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
  }
};

// conversion of eight consecutive elements per thread (16-byte accesses on the 16-bit side)
template <class TS, class TD>
__global__ void convert8_kernel(const TS* src, TD* dst, size_t n8, const float* scale) {
  const float sc = scale ? *scale : 1.f;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x) {
    float v[8];
    Ld8<TS>::load(src + i * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] *= sc;
    Ld8<TD>::store(dst + i * 8, v);
  }
}

// maximum of |x| over eight consecutive elements per thread
template <class TS>
__global__ void amax8_kernel(const TS* x, size_t n8, unsigned* amax_bits) {
  float m = 0.f;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x) {
    float v[8];
    Ld8<TS>::load(x + i * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) m = fmaxf(m, fabsf(v[k]));
  }
  block_amax(m, amax_bits);
}

// eight consecutive values of a parameter vector whose type is known only at run time
__device__ __forceinline__ void load8_param(const void* p, int c, int dt, float (&v)[8]) {
  if (dt == LS_F32) Ld8<float>::load((const float*)p + c, v);
  else if (dt == LS_BF16) Ld8<bf16_t>::load((const bf16_t*)p + c, v);
  else Ld8<f16_t>::load((const f16_t*)p + c, v);
}

// eight values kept in the form they were loaded in (four registers for a 16-bit type)
template <class TD> struct Raw8 {
  typename vec8<TD>::type t;
  __device__ __forceinline__ void load(const TD* p) { t = *(const typename vec8<TD>::type*)p; }
  __device__ __forceinline__ float get(int i) const { return to_f(t[i]); }
};
template <> struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) { a = *(const f32x4*)p; b = *(const f32x4*)(p + 4); }
  __device__ __forceinline__ float get(int i) const { return i < 4 ? a[i] : b[i - 4]; }
};

// Forward, one wavefront per row (four rows per workgroup): a lane owns eight
// consecutive columns out of every 512, the row stays in registers between the
// statistics and the output, and no LDS or barrier is involved.  Needs
// d % 8 == 0, d <= 512 * NIT and 16-byte aligned rows and parameters.
template <class TH, int NIT>
__global__ __launch_bounds__(256) void norm_fwd_rows_kernel(int kind, const float* x, int T, int d,
                                                            const void* gamma, const void* beta, int pdt,
                                                            float eps, TH* h, float* mean, float* rstd) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= T) return;
  const size_t off = (size_t)row * d;
  float v[NIT][8];
  float s = 0.f;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = lane * 8 + it * 512;
    if (c < d) Ld8<float>::load(x + off + c, v[it]);
    else
#pragma unroll
      for (int i = 0; i < 8; ++i) v[it][i] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += v[it][i];
  }
  const float mu = kind == 0 ? wave_total(s) / d : 0.f;
  float q = 0.f;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
    if (lane * 8 + it * 512 < d)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float t = v[it][i] - mu;
        q += t * t;
      }
  const float r = 1.0f / sqrtf(wave_total(q) / d + eps);
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = lane * 8 + it * 512;
    if (c < d) {
      float gam[8], o[8];
      load8_param(gamma, c, pdt, gam);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = (v[it][i] - mu) * r * gam[i];
      if (kind == 0 && beta) {
        load8_param(beta, c, pdt, gam);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] += gam[i];
      }
      Ld8<TH>::store(h + off + c, o);
    }
  }
  if (lane == 0) {
    if (mean && kind == 0) mean[row] = mu;
    if (rstd) rstd[row] = r;
  }
}

// eight parameters as they are in memory; the type is looked at when they are used, so that the loads of a row are all
// requested before the first of them is waited for
template <bool P32> struct RawParam {
  u32x4 v[P32 ? 2 : 1];
  __device__ __forceinline__ void load(const void* p, int c) {
    const u32x4* q = (const u32x4*)((const char*)p + (size_t)c * (P32 ? 4 : 2));
    v[0] = q[0];
    if constexpr (P32) v[1] = q[1];
  }
  __device__ __forceinline__ void get(int dt, float (&o)[8]) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (P32) {
        const uint32_t bits = v[i / 4][i % 4];
        o[i] = __uint_as_float(bits);
      } else {
        const uint16_t h = (uint16_t)(v[0][i / 2] >> (i % 2 * 16));
        o[i] = dt == LS_BF16 ? to_f(__builtin_bit_cast(bf16_t, h)) : to_f(__builtin_bit_cast(f16_t, h));
      }
    }
  }
};

// Backward in one pass over the data, one wavefront per row and `rows` rows (8 or 16) per
// 512-thread workgroup: the row's dh and xhat stay in registers between the two
// row means and dx, each wave keeps its dgamma / dbeta column sums in registers
// and the eight waves' sums are combined in a fixed order through LDS into
// partial[workgroup][2][d] (RMSNorm leaves the dbeta half unwritten).  Needs d % 8 == 0, d <= 512 * NIT, 16-byte alignment.
// PRE: a row's loads, those of the residual gradient and the parameters among them, are one round trip, none of them
// behind a branch (columns past the end repeat the last eight).  Wider rows have no registers for that.  With
// the finishing launch, 1024 rows of 768: 13.6 -> 10.1 us, 4096 rows 21.3 -> 19.0 (up to four round trips a row before).
template <class TD, int KIND, int NIT, bool PRE, bool P32>
__global__ __launch_bounds__(512) void norm_bwd_rows_kernel(const TD* dh, const float* x, const float* mean,
                                                            const float* rstd, const void* gamma, int pdt,
                                                            int T, int d, int rows, const float* dres, float* dx,
                                                            TD* dx16, float* partial) {
  extern __shared__ float sred[];  // [8][d]
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r0 = blockIdx.x * rows, r1 = min(T, r0 + rows);
  constexpr int NB = KIND == 0 ? NIT : 1;
  float dg[NIT][8], db[NB][8];
#pragma unroll
  for (int it = 0; it < NIT; ++it)
#pragma unroll
    for (int i = 0; i < 8; ++i) dg[it][i] = 0.f;
#pragma unroll
  for (int it = 0; it < NB; ++it)
#pragma unroll
    for (int i = 0; i < 8; ++i) db[it][i] = 0.f;
  for (int row = r0 + w; row < r1; row += 8) {
    const size_t off = (size_t)row * d;
    const float mu = KIND == 0 ? mean[row] : 0.f, r = rstd[row];
    Raw8<TD> g[NIT];
    Raw8<float> dr[PRE ? NIT : 1];
    RawParam<P32> gp[PRE ? NIT : 1];
    float xh[NIT][8];
    float s1 = 0.f, s2 = 0.f;
    if constexpr (PRE) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int c = min(lane * 8 + it * 512, d - 8);
        g[it].load(dh + off + c);
        Ld8<float>::load(x + off + c, xh[it]);
        gp[it].load(gamma, c);
      }
      if (dres)
#pragma unroll
        for (int it = 0; it < NIT; ++it) dr[it].load(dres + off + min(lane * 8 + it * 512, d - 8));
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int c = lane * 8 + it * 512;
      if (c < d) {
        float gam[8];
        if constexpr (PRE) {
          gp[it].get(pdt, gam);
        } else {
          g[it].load(dh + off + c);
          Ld8<float>::load(x + off + c, xh[it]);
          load8_param(gamma, c, pdt, gam);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float dxh = g[it].get(i) * gam[i];
          xh[it][i] = (xh[it][i] - mu) * r;
          s1 += dxh;
          s2 += dxh * xh[it][i];
        }
      }
    }
    const float m1 = KIND == 0 ? wave_total(s1) / d : 0.f;
    const float m2 = wave_total(s2) / d;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int c = lane * 8 + it * 512;
      if (c < d) {
        float gam[8], o[8];
        if constexpr (PRE) {
          gp[it].get(pdt, gam);
#pragma unroll
          for (int i = 0; i < 8; ++i) o[i] = dr[it].get(i);
        } else {
          load8_param(gamma, c, pdt, gam);
          if (dres) Ld8<float>::load(dres + off + c, o);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float gi = g[it].get(i);
          const float val = r * (gi * gam[i] - m1 - xh[it][i] * m2);
          o[i] = dres ? o[i] + val : val;
          dg[it][i] += gi * xh[it][i];
          if (KIND == 0) db[it][i] += gi;
        }
        Ld8<float>::store(dx + off + c, o);
        if (dx16) Ld8<TD>::store(dx16 + off + c, o);
      }
    }
  }
  float* p = partial + (size_t)blockIdx.x * 2 * d;
#pragma unroll
  for (int pass = 0; pass < (KIND == 0 ? 2 : 1); ++pass) {
    if (pass) __syncthreads();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int c = lane * 8 + it * 512;
      if (c < d) Ld8<float>::store(sred + (size_t)w * d + c, pass == 0 ? dg[it] : db[KIND == 0 ? it : 0]);
    }
    __syncthreads();
    for (int c = threadIdx.x * 4; c < d; c += 2048) {
      f32x4 a = *(const f32x4*)(sred + c);
#pragma unroll
      for (int k = 1; k < 8; ++k) a += *(const f32x4*)(sred + (size_t)k * d + c);
      *(f32x4*)(p + pass * d + c) = a;
    }
  }
}

template <class TD>
__global__ __launch_bounds__(256) void norm_bwd_stats_kernel(int kind, const TD* dh, const float* x,
                                                             const float* mean, const float* rstd,
                                                             const void* gamma, int pdt, int T, int d,
                                                             float* stats) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= T) return;
  const size_t off = (size_t)row * d;
  const float mu = kind == 0 ? mean[row] : 0.f, r = rstd[row];
  float s1 = 0.f, s2 = 0.f;
  for (int c = lane * 8; c < d; c += 512) {
    float g[8], xv[8];
    Ld8<TD>::load(dh + off + c, g);
    Ld8<float>::load(x + off + c, xv);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float dxh = g[i] * load_as_f(gamma, c + i, pdt);
      s1 += dxh;
      s2 += dxh * (xv[i] - mu) * r;
    }
  }
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  if (lane == 0) {
    stats[2 * row] = s1 / d;
    stats[2 * row + 1] = s2 / d;
  }
}

template <class TD>
__global__ __launch_bounds__(256) void norm_bwd_apply_kernel(int kind, const TD* dh, const float* x,
                                                             const float* mean, const float* rstd,
                                                             const void* gamma, int pdt, int T, int d,
                                                             const float* stats, const float* dres,
                                                             float* dx, TD* dx16, float* partial) {
  const int c = (blockIdx.x * 256 + threadIdx.x) * 8;
  if (c >= d) return;
  float gam[8], dg[8], db[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    gam[i] = load_as_f(gamma, c + i, pdt);
    dg[i] = db[i] = 0.f;
  }
  const int r0 = blockIdx.y * NB_ROWS, r1 = min(T, r0 + NB_ROWS);
  for (int row = r0; row < r1; ++row) {
    const size_t off = (size_t)row * d + c;
    const float mu = kind == 0 ? mean[row] : 0.f, r = rstd[row];
    const float m1 = kind == 0 ? stats[2 * row] : 0.f, m2 = stats[2 * row + 1];
    float g[8], xv[8], o[8];
    Ld8<TD>::load(dh + off, g);
    Ld8<float>::load(x + off, xv);
    if (dres) Ld8<float>::load(dres + off, o);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float xh = (xv[i] - mu) * r;
      const float v = r * (g[i] * gam[i] - m1 - xh * m2);
      o[i] = dres ? o[i] + v : v;
      dg[i] += g[i] * xh;
      db[i] += g[i];
    }
    Ld8<float>::store(dx + off, o);
    if (dx16) Ld8<TD>::store(dx16 + off, o);
  }
  float* p = partial + (size_t)blockIdx.y * 2 * d + c;
  Ld8<float>::store(p, dg);
  Ld8<float>::store(p + d, db);
}

// The column sums of several norm backwards over the same rows: set i = blockIdx.y has its partial sums at
// partial + i * stride and its results in block i / 2 of the gradient vector, at first (i even) or second.
struct NormSums {
  const float* partial; size_t stride;
  float* grad; size_t per_block;   // elements of a block
  size_t gamma[2], beta[2];        // offsets in a block
  int has_gamma, has_beta;
};

// 32 columns (eight float4 lanes) x 32 row groups per workgroup; the 32 partial sums of a
// column are combined in a fixed order through LDS.  d % 4 == 0.
__global__ __launch_bounds__(256) void norm_bwd_finish_kernel(NormSums s, int nwg, int d, int accumulate, const float* alpha) {
  __shared__ float sg[32][32], sb[32][32];
  const float* partial = s.partial + blockIdx.y * s.stride;
  float* grad = s.grad + (blockIdx.y >> 1) * s.per_block;
  const int cg = threadIdx.x & 7, rg = threadIdx.x >> 3;
  const int i = blockIdx.x * 32 + cg * 4;
  f32x4 g = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
  if (i < d)
    for (int w = rg; w < nwg; w += 32) {
      g += *(const f32x4*)(partial + (size_t)w * 2 * d + i);
      if (s.has_beta) b += *(const f32x4*)(partial + (size_t)w * 2 * d + d + i);
    }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    sg[rg][cg * 4 + k] = g[k];
    sb[rg][cg * 4 + k] = b[k];
  }
  __syncthreads();
  const int col = blockIdx.x * 32 + threadIdx.x;
  if (threadIdx.x >= 32 || col >= d) return;
  float tg = 0.f, tb = 0.f;
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    tg += sg[k][threadIdx.x];
    tb += sb[k][threadIdx.x];
  }
  if (alpha) { tg *= *alpha; tb *= *alpha; }
  float *dgamma = grad + s.gamma[blockIdx.y & 1] + col, *dbeta = grad + s.beta[blockIdx.y & 1] + col;
  if (s.has_gamma) *dgamma = accumulate ? *dgamma + tg : tg;
  if (s.has_beta) *dbeta = accumulate ? *dbeta + tb : tb;
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// Rows per workgroup of the one-pass kernel: one per wavefront while two would leave compute units without a workgroup or
// with half of their registers idle; beyond, two, as every workgroup also sums its rows' columns and writes 2 d of them.
// us with the finishing launch, one row -> two: d 768, 128 rows 7.4, 8.9; 1024 rows 10.1, 10.9; 1500 rows 11.7, 11.7; 2048
// rows 13.4, 12.6; d 4096, 16 rows 14.6, 26.9; 1024 rows 29.5, 44.1; 2048 rows 37.2, 51.8; 3000 rows 61.6, 58.2.
inline int norm_bwd_few_rows(int d) { return d <= 1024 ? 1280 : 2048; }
inline int norm_bwd_rows_per_wg(int T, int d) { return T <= norm_bwd_few_rows(d) ? 8 : 16; }

template <class TD, int KIND, int NIT, bool PRE>
ls_status launch_norm_bwd_rows(const void* dh, const float* x, const float* mean, const float* rstd,
                               const void* gamma, int pdt, int T, int d, const float* dres, float* dx,
                               void* dx16, float* partial, hipStream_t st) {
  const size_t lds = (size_t)8 * d * sizeof(float);
  const int rows = norm_bwd_rows_per_wg(T, d);
  auto go = [&](auto* kern, bool& attr_set) -> ls_status {
    if (!attr_set) {
      LS_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * 512 * NIT * 4));
      attr_set = true;
    }
    kern<<<(T + rows - 1) / rows, 512, lds, st>>>((const TD*)dh, x, mean, rstd, gamma, pdt, T, d, rows, dres, dx,
                                                  (TD*)dx16, partial);
    return LS_OK;
  };
  static bool set16 = false, set32 = false;
  return PRE && pdt == LS_F32 ? go(norm_bwd_rows_kernel<TD, KIND, NIT, PRE, PRE>, set32)
                              : go(norm_bwd_rows_kernel<TD, KIND, NIT, PRE, false>, set16);
}

template <class TD>
ls_status launch_norm_bwd(int kind, const void* dh, const float* x, const float* mean, const float* rstd,
                          const void* gamma, int pdt, int T, int d, const float* dres, float* dx, void* dx16,
                          float* partial, bool rows_ok, hipStream_t st) {
  if (rows_ok) {
#define LS_NB(K, N, P) launch_norm_bwd_rows<TD, K, N, P>(dh, x, mean, rstd, gamma, pdt, T, d, dres, dx, dx16, partial, st)
    if (d <= 1024) return kind == 0 ? LS_NB(0, 2, true) : LS_NB(1, 2, true);
    if (kind == 0) return LS_NB(0, 4, false);
    return d <= 2048 ? LS_NB(1, 4, false) : LS_NB(1, 8, false);
#undef LS_NB
  }
  const int nchunk = (T + NB_ROWS - 1) / NB_ROWS;
  float* stats = partial + (size_t)nchunk * 2 * d;
  norm_bwd_stats_kernel<TD><<<(T + 3) / 4, 256, 0, st>>>(kind, (const TD*)dh, x, mean, rstd, gamma, pdt, T, d, stats);
  norm_bwd_apply_kernel<TD><<<dim3((d + 2047) / 2048, nchunk), 256, 0, st>>>(
      kind, (const TD*)dh, x, mean, rstd, gamma, pdt, T, d, stats, dres, dx, (TD*)dx16, partial);
  return LS_OK;
}

template <class TH>
void launch_norm_fwd_rows(int kind, const float* x, int T, int d, const void* gamma, const void* beta, int pdt,
                          float eps, void* h, float* mean, float* rstd, hipStream_t st) {
  const int grid = (T + 3) / 4;
  if (d <= 2048)
    norm_fwd_rows_kernel<TH, 4><<<grid, 256, 0, st>>>(kind, x, T, d, gamma, beta, pdt, eps, (TH*)h, mean, rstd);
  else if (d <= 4096)
    norm_fwd_rows_kernel<TH, 8><<<grid, 256, 0, st>>>(kind, x, T, d, gamma, beta, pdt, eps, (TH*)h, mean, rstd);
  else
    norm_fwd_rows_kernel<TH, 16><<<grid, 256, 0, st>>>(kind, x, T, d, gamma, beta, pdt, eps, (TH*)h, mean, rstd);
}

// -------------------------------------------------------------------- rope
// one thread per (row, head, pair)
__global__ void rope_kernel(void* qkv, int dt, int T, int h, int dh, const int32_t* pos,
                            const float* table, float sign) {
  const int half = dh / 2;
  const size_t n = (size_t)T * 2 * h * half;
  const int d = h * dh;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int i = idx % half;
    const int hh = (idx / half) % (2 * h);  // q heads then k heads
    const size_t t = idx / ((size_t)half * 2 * h);
    const size_t base = t * 3 * d + (size_t)hh * dh + i;
    const float c = table[((size_t)pos[t] * half + i) * 2];
    const float s = table[((size_t)pos[t] * half + i) * 2 + 1] * sign;
    const float a = load_as_f(qkv, base, dt), b = load_as_f(qkv, base + half, dt);
    store_from_f(qkv, base, dt, a * c - b * s);
    store_from_f(qkv, base + half, dt, b * c + a * s);
  }
}

// ------------------------------------------------------------- activations
__device__ __forceinline__ float gelu_grad_f(float u, int kind) {
  if (kind == LS_ACT_GELU_TANH) {
    const float t = tanhf(kGeluC * (u + 0.044715f * u * u * u));
    return 0.5f * (1.f + t) + 0.5f * u * (1.f - t * t) * kGeluC * (1.f + 3.f * 0.044715f * u * u);
  }
  const float Phi = 0.5f * (1.f + erff(u * 0.70710678118654752f));
  const float phi = 0.3989422804014327f * expf(-0.5f * u * u);
  return Phi + u * phi;
}

__global__ void gelu_fwd_kernel(const void* u, void* g, int dt, size_t n, int kind) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    store_from_f(g, i, dt, gelu_f(load_as_f(u, i, dt), kind));
}
__global__ void gelu_bwd_kernel(const void* dg, const void* u, void* du, int dt, size_t n, int kind) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    store_from_f(du, i, dt, load_as_f(dg, i, dt) * gelu_grad_f(load_as_f(u, i, dt), kind));
}
// 16-bit operands: 8 units per thread with 16-byte accesses, the tanh form written as u sigmoid(2 y), which keeps its
// relative accuracy in the negative tail where 1 + tanh(y) cancels.  The element-per-thread kernels above, with tanhf,
// were bound by instructions (4096 x 3072 units: 29 us a launch on average; the six-layer task of 4 x 1024 tokens, which
// launches twelve, went from 3641 to 3523 us).
template <int KIND> __device__ __forceinline__ float gelu16_f(float u) {
  if (KIND != LS_ACT_GELU_TANH) return gelu_f(u, KIND);
  const float y = kGeluC * (u + 0.044715f * u * u * u);
  return u * __builtin_amdgcn_rcpf(1.f + expf(-2.f * y));
}
template <int KIND> __device__ __forceinline__ float gelu16_grad_f(float u) {
  if (KIND != LS_ACT_GELU_TANH) return gelu_grad_f(u, KIND);
  const float y = kGeluC * (u + 0.044715f * u * u * u);
  const float s = __builtin_amdgcn_rcpf(1.f + expf(-2.f * y));
  return s + 2.f * u * s * (1.f - s) * kGeluC * (1.f + 3.f * 0.044715f * u * u);
}
template <class TD, int KIND>
__global__ void gelu8_fwd_kernel(const TD* u, TD* g, size_t n8) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x) {
    float v[8];
    Ld8<TD>::load(u + i * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = gelu16_f<KIND>(v[k]);
    Ld8<TD>::store(g + i * 8, v);
  }
}
template <class TD, int KIND>
__global__ void gelu8_bwd_kernel(const TD* dg, const TD* u, TD* du, size_t n8) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x) {
    float v[8], g[8];
    Ld8<TD>::load(u + i * 8, v);
    Ld8<TD>::load(dg + i * 8, g);
#pragma unroll
    for (int k = 0; k < 8; ++k) g[k] *= gelu16_grad_f<KIND>(v[k]);
    Ld8<TD>::store(du + i * 8, g);
  }
}
// SwiGLU: a thread owns 8 consecutive hidden units (16-byte loads of gate, up)
template <class TD>
__global__ void swiglu_fwd_kernel(const TD* gu, TD* a, size_t T, int F) {
  const size_t n8 = T * (size_t)(F / 8);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8;
       i += (size_t)gridDim.x * blockDim.x) {
    const size_t t = i / (F / 8), f = (i % (F / 8)) * 8;
    float gt[8], up[8], o[8];
    Ld8<TD>::load(gu + t * 2 * F + f, gt);
    Ld8<TD>::load(gu + t * 2 * F + F + f, up);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = gt[k] / (1.f + __expf(-gt[k])) * up[k];
    Ld8<TD>::store(a + t * F + f, o);
  }
}
template <class TD>
__global__ void swiglu_bwd_kernel(const TD* da, const TD* gu, TD* dgu, size_t T, int F) {
  const size_t n8 = T * (size_t)(F / 8);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8;
       i += (size_t)gridDim.x * blockDim.x) {
    const size_t t = i / (F / 8), f = (i % (F / 8)) * 8;
    float gt[8], up[8], g[8], og[8], ou[8];
    Ld8<TD>::load(gu + t * 2 * F + f, gt);
    Ld8<TD>::load(gu + t * 2 * F + F + f, up);
    Ld8<TD>::load(da + t * F + f, g);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float sg = 1.f / (1.f + __expf(-gt[k]));
      og[k] = g[k] * up[k] * sg * (1.f + gt[k] * (1.f - sg));
      ou[k] = g[k] * gt[k] * sg;
    }
    Ld8<TD>::store(dgu + t * 2 * F + f, og);
    Ld8<TD>::store(dgu + t * 2 * F + F + f, ou);
  }
}

// ------------------------------------------------------------------ colsum
// Two kernels: partial sums over CS_ROWS rows, then the sum of the partials in a fixed order.  A workgroup takes
// 256 columns (32 lanes of eight consecutive ones, 16-byte loads of a 16-bit type) x CS_ROWS rows dealt to eight
// row lanes, so a thread has its eight loads in flight together and a 4096 x 768 matrix gives 192 workgroups.
// One column per thread, 128 rows one after the other (the form kept below for widths or bases that are not
// multiples of eight elements) was a chain of 128 dependent additions: 40 us at 4096 x 768, 39 us at 999 x 768,
// against 4.6 and 4.7 us now, which is what any launch takes here.
constexpr int CS_ROWS = 64;
__global__ __launch_bounds__(256) void colsum_kernel(const void* x, int dt, int T, int N, long ld,
                                                     float* partial) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  const int r0 = blockIdx.y * CS_ROWS;
  if (n >= N) return;
  float s = 0.f;
  const int r1 = min(T, r0 + CS_ROWS);
  for (int r = r0; r < r1; ++r) s += load_as_f(x, (size_t)r * ld + n, dt);
  partial[(size_t)blockIdx.y * N + n] = s;
}

// the eight row lanes' sums of a workgroup's 256 columns, combined in a fixed order; partial row of the workgroup
__device__ __forceinline__ void colsum_combine(const float (&s)[8], int n, int N, float* partial) {
  __shared__ float red[8][32 * 8 + 4];
  const int cl = threadIdx.x & 31, rl = threadIdx.x >> 5;
  Ld8<float>::store(&red[rl][cl * 8], s);
  __syncthreads();
  const int c = threadIdx.x, col = (n - cl * 8) + c;
  if (col >= N) return;
  float t = red[0][c];
#pragma unroll
  for (int k = 1; k < 8; ++k) t += red[k][c];
  partial[(size_t)blockIdx.y * N + col] = t;
}
template <class TD>
__global__ __launch_bounds__(256) void colsum8_kernel(const TD* x, int T, int N, long ld, float* partial) {
  const int n = blockIdx.x * 256 + (threadIdx.x & 31) * 8, r0 = blockIdx.y * CS_ROWS + (threadIdx.x >> 5);
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (n < N) {
    Raw8<TD> v[CS_ROWS / 8];
#pragma unroll
    for (int k = 0; k < CS_ROWS / 8; ++k)   // rows past the end read the last one and are left out of the sum
      v[k].load(x + (size_t)min(r0 + k * 8, T - 1) * ld + n);
#pragma unroll
    for (int k = 0; k < CS_ROWS / 8; ++k)
      if (r0 + k * 8 < T)
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] += v[k].get(i);
  }
  colsum_combine(s, n, N, partial);
}
// 32 columns x 8 chunk lanes per workgroup, for up to four sums over the same rows: a launch of its own for each sum was
// 3 - 5 us of latency, three of them per block more than needed (training pass of two
// micro-batches of 3 x 333 tokens, six blocks: 3590 -> 3491 us)
struct ColsumSet {
  int n, first[kMaxColsums + 1];   // first workgroup of each
  LsColsum sum[kMaxColsums];
};
__global__ __launch_bounds__(256) void colsum_finish_kernel(ColsumSet set, int nchunk, int accumulate,
                                                            const float* alpha) {
  int i = 0;
  while (i + 1 < set.n && (int)blockIdx.x >= set.first[i + 1]) ++i;
  const float* partial = set.sum[i].partial;
  const int N = set.sum[i].N;
  float* out = set.sum[i].out;
  __shared__ float red[8][32];
  const int c = threadIdx.x & 31, k0 = threadIdx.x >> 5, n = ((int)blockIdx.x - set.first[i]) * 32 + c;
  float s = 0.f;
  if (n < N)
#pragma unroll 8
    for (int k = k0; k < nchunk; k += 8) s += partial[(size_t)k * N + n];
  red[k0][c] = s;
  __syncthreads();
  if (threadIdx.x >= 32 || n >= N) return;
  s = red[0][c];
#pragma unroll
  for (int k = 1; k < 8; ++k) s += red[k][c];
  if (alpha) s *= *alpha;
  out[n] = accumulate ? out[n] + s : s;
}

inline int grid_for(size_t n, int block = 256, int cap = 256 * 32) {
  size_t g = (n + block - 1) / block;
  return (int)(g < 1 ? 1 : (g > (size_t)cap ? cap : g));
}
bool ok_dtype(int dt) { return dt == LS_F32 || dt == LS_BF16 || dt == LS_F16; }

}  // namespace

extern "C" {

ls_status lsk_convert_scaled(const void* src, int sdt, void* dst, int ddt, size_t n, const float* scale_dev,
                             void* stream) {
  LS_REQUIRE(src && dst && ok_dtype(sdt) && ok_dtype(ddt), "convert: bad argument");
  if (n == 0) return LS_OK;
  hipStream_t st = (hipStream_t)stream;
  if (n % 8 == 0 && ((uintptr_t)src & 15) == 0 && ((uintptr_t)dst & 15) == 0) {
    const size_t n8 = n / 8;
    const int g = grid_for(n8);
#define LS_CV(TS, TD) convert8_kernel<TS, TD><<<g, 256, 0, st>>>((const TS*)src, (TD*)dst, n8, scale_dev)
    if (sdt == LS_F32) { if (ddt == LS_F32) LS_CV(float, float); else if (ddt == LS_BF16) LS_CV(float, bf16_t); else LS_CV(float, f16_t); }
    else if (sdt == LS_BF16) { if (ddt == LS_F32) LS_CV(bf16_t, float); else if (ddt == LS_BF16) LS_CV(bf16_t, bf16_t); else LS_CV(bf16_t, f16_t); }
    else { if (ddt == LS_F32) LS_CV(f16_t, float); else if (ddt == LS_BF16) LS_CV(f16_t, bf16_t); else LS_CV(f16_t, f16_t); }
#undef LS_CV
  } else {
    convert_kernel<<<grid_for(n), 256, 0, st>>>(src, sdt, dst, ddt, n, scale_dev);
  }
  LS_CHECK_LAUNCH();
  return LS_OK;
}
ls_status lsk_convert(const void* src, int sdt, void* dst, int ddt, size_t n, void* stream) {
  return lsk_convert_scaled(src, sdt, dst, ddt, n, nullptr, stream);
}

ls_status lsk_grad_scale(const void* x, int dt, size_t n, float* out3, void* stream) {
  LS_REQUIRE(x && out3 && ok_dtype(dt) && n > 0, "grad_scale: bad argument");
  hipStream_t st = (hipStream_t)stream;
  scale_reset_kernel<<<1, 1, 0, st>>>(out3);
  if (n % 8 == 0 && ((uintptr_t)x & 15) == 0) {
    const int g = grid_for(n / 8, 256, 2048);
    if (dt == LS_F32) amax8_kernel<float><<<g, 256, 0, st>>>((const float*)x, n / 8, (unsigned*)(out3 + 2));
    else if (dt == LS_BF16) amax8_kernel<bf16_t><<<g, 256, 0, st>>>((const bf16_t*)x, n / 8, (unsigned*)(out3 + 2));
    else amax8_kernel<f16_t><<<g, 256, 0, st>>>((const f16_t*)x, n / 8, (unsigned*)(out3 + 2));
  } else {
    amax_kernel<<<grid_for(n, 256, 2048), 256, 0, st>>>(x, dt, n, (unsigned*)(out3 + 2));
  }
  scale_finish_kernel<<<1, 1, 0, st>>>(out3);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_norm_fwd(int kind, const float* x, int T, int d, const void* gamma, const void* beta,
                       int pdt, float eps, void* h, int hdt, float* mean, float* rstd, void* stream) {
  LS_REQUIRE(x && gamma && h && T > 0 && d > 0, "norm_fwd: bad argument");
  LS_REQUIRE(kind == 0 || kind == 1, "norm_fwd: kind must be 0 (LayerNorm) or 1 (RMSNorm)");
  LS_REQUIRE(d <= 256 * NF_MAXCOL, "norm_fwd: d_model %d exceeds %d", d, 256 * NF_MAXCOL);
  hipStream_t st = (hipStream_t)stream;
  if (d % 8 == 0 && aligned16(x) && aligned16(h) && aligned16(gamma) && (!beta || aligned16(beta))) {
    if (hdt == LS_F32) launch_norm_fwd_rows<float>(kind, x, T, d, gamma, beta, pdt, eps, h, mean, rstd, st);
    else if (hdt == LS_BF16) launch_norm_fwd_rows<bf16_t>(kind, x, T, d, gamma, beta, pdt, eps, h, mean, rstd, st);
    else launch_norm_fwd_rows<f16_t>(kind, x, T, d, gamma, beta, pdt, eps, h, mean, rstd, st);
  } else {
    norm_fwd_kernel<<<T, 256, 0, st>>>(kind, x, d, gamma, beta, pdt, eps, h, hdt, mean, rstd);
  }
  LS_CHECK_LAUNCH();
  return LS_OK;
}

size_t lsk_norm_bwd_partial_floats(int T, int d) {
  // never less for more rows: a workspace sized for T holds every shorter call
  const int few = norm_bwd_few_rows(d), by8 = ((T < few ? T : few) + 7) / 8, by16 = (T + NB_ROWS - 1) / NB_ROWS;
  return (size_t)(by8 > by16 ? by8 : by16) * 2 * d + 2 * (size_t)T;
}

// dx, and the column sums of `chunks` runs of rows in partial, for lsk_norm_bwd_sums
ls_status lsk_norm_bwd_partials(int kind, const void* dh, int dhdt, const float* x, const float* mean, const float* rstd,
                                const void* gamma, int pdt, int T, int d, const float* dres, float* dx, void* dx16,
                                int dx16dt, float* partial, int* chunks, void* stream) {
  LS_REQUIRE(dh && x && rstd && gamma && dx && partial && T > 0 && d > 0, "norm_bwd: bad argument");
  LS_REQUIRE(kind == 1 || mean, "norm_bwd: LayerNorm needs the saved mean");
  LS_REQUIRE(d % 8 == 0, "norm_bwd: d_model must be a multiple of 8");
  LS_REQUIRE(!dx16 || dx16dt == dhdt, "norm_bwd: the 16-bit copy of dx must have the type of dh");
  hipStream_t st = (hipStream_t)stream;
  // LayerNorm's second set of column sums does not fit the register file beyond 2048 columns
  const bool rows_ok = d <= (kind == 0 ? 2048 : 4096) && aligned16(dh) && aligned16(x) && aligned16(gamma) && aligned16(dx) &&
                       aligned16(partial) && (!dres || aligned16(dres)) && (!dx16 || aligned16(dx16));
  if (dhdt == LS_F32) LS_TRY(launch_norm_bwd<float>(kind, dh, x, mean, rstd, gamma, pdt, T, d, dres, dx, dx16, partial, rows_ok, st));
  else if (dhdt == LS_BF16) LS_TRY(launch_norm_bwd<bf16_t>(kind, dh, x, mean, rstd, gamma, pdt, T, d, dres, dx, dx16, partial, rows_ok, st));
  else LS_TRY(launch_norm_bwd<f16_t>(kind, dh, x, mean, rstd, gamma, pdt, T, d, dres, dx, dx16, partial, rows_ok, st));
  LS_CHECK_LAUNCH();
  const int rows = rows_ok ? norm_bwd_rows_per_wg(T, d) : NB_ROWS;
  *chunks = (T + rows - 1) / rows;
  return LS_OK;
}
// The gradients of both norms of n blocks from the partial sums of 2 n calls, in one launch: the sets `stride` floats apart,
// two a block (gamma[0] / beta[0], then gamma[1] / beta[1], elements into a block's part of grad); beta null: none.
ls_status lsk_norm_bwd_sums(const float* partial, size_t stride, int chunks, int d, int n, float* grad, size_t per_block,
                            const size_t* gamma, const size_t* beta, int accumulate, const float* alpha_dev, void* stream) {
  LS_REQUIRE(partial && grad && gamma && chunks > 0 && d > 0 && n > 0, "norm_bwd_sums: bad argument");
  const NormSums s{partial, stride, grad, per_block, {gamma[0], gamma[1]}, {beta ? beta[0] : 0, beta ? beta[1] : 0}, 1,
                   beta != nullptr};
  norm_bwd_finish_kernel<<<dim3((d + 31) / 32, 2 * n), 256, 0, (hipStream_t)stream>>>(s, chunks, d, accumulate, alpha_dev);
  LS_CHECK_LAUNCH();
  return LS_OK;
}
ls_status lsk_norm_bwd_scaled(int kind, const void* dh, int dhdt, const float* x, const float* mean,
                              const float* rstd, const void* gamma, int pdt, int T, int d,
                              const float* dres, float* dx, void* dx16, int dx16dt, float* dgamma,
                              float* dbeta, int accumulate, float* partial, const float* alpha_dev,
                              void* stream) {
  int chunks = 0;
  LS_TRY(lsk_norm_bwd_partials(kind, dh, dhdt, x, mean, rstd, gamma, pdt, T, d, dres, dx, dx16, dx16dt, partial, &chunks,
                               stream));
  if (dgamma || (dbeta && kind == 0)) {
    // offsets from one address, which may be either
    float* base = dgamma ? dgamma : dbeta;
    const size_t off = dgamma && dbeta ? (size_t)(dbeta - dgamma) : 0;
    const NormSums s{partial, 0, base, 0, {0, 0}, {off, off}, dgamma != nullptr, dbeta && kind == 0};
    norm_bwd_finish_kernel<<<(d + 31) / 32, 256, 0, (hipStream_t)stream>>>(s, chunks, d, accumulate, alpha_dev);
    LS_CHECK_LAUNCH();
  }
  return LS_OK;
}
ls_status lsk_norm_bwd(int kind, const void* dh, int dhdt, const float* x, const float* mean,
                       const float* rstd, const void* gamma, int pdt, int T, int d,
                       const float* dres, float* dx, void* dx16, int dx16dt, float* dgamma,
                       float* dbeta, int accumulate, float* partial, void* stream) {
  return lsk_norm_bwd_scaled(kind, dh, dhdt, x, mean, rstd, gamma, pdt, T, d, dres, dx, dx16, dx16dt, dgamma,
                             dbeta, accumulate, partial, nullptr, stream);
}

ls_status lsk_rope(void* qkv, int dt, int T, int h, int dh, const int32_t* pos, const float* table,
                   float sign, void* stream) {
  LS_REQUIRE(qkv && pos && table && T > 0 && h > 0 && dh > 0 && dh % 2 == 0, "rope: bad argument");
  const size_t n = (size_t)T * 2 * h * (dh / 2);
  rope_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(qkv, dt, T, h, dh, pos, table, sign);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_gelu_fwd(const void* u, void* g, int dt, size_t n, int kind, void* stream) {
  LS_REQUIRE(u && g && n > 0, "gelu_fwd: bad argument");
  if (dt != LS_F32 && n % 8 == 0 && (((uintptr_t)u | (uintptr_t)g) & 15) == 0) {
    auto go = [&](auto* p, auto* q) {
      typedef std::remove_pointer_t<decltype(q)> TD;
      const int gr = grid_for(n / 8);
      if (kind == LS_ACT_GELU_TANH) gelu8_fwd_kernel<TD, LS_ACT_GELU_TANH><<<gr, 256, 0, (hipStream_t)stream>>>(p, q, n / 8);
      else gelu8_fwd_kernel<TD, LS_ACT_GELU_ERF><<<gr, 256, 0, (hipStream_t)stream>>>(p, q, n / 8);
    };
    if (dt == LS_BF16) go((const bf16_t*)u, (bf16_t*)g);
    else go((const f16_t*)u, (f16_t*)g);
    LS_CHECK_LAUNCH();
    return LS_OK;
  }
  gelu_fwd_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(u, g, dt, n, kind);
  LS_CHECK_LAUNCH();
  return LS_OK;
}
ls_status lsk_gelu_bwd(const void* dg, const void* u, void* du, int dt, size_t n, int kind, void* stream) {
  LS_REQUIRE(dg && u && du && n > 0, "gelu_bwd: bad argument");
  if (dt != LS_F32 && n % 8 == 0 && (((uintptr_t)dg | (uintptr_t)u | (uintptr_t)du) & 15) == 0) {
    auto go = [&](auto* p, auto* q, auto* r) {
      typedef std::remove_pointer_t<decltype(r)> TD;
      const int gr = grid_for(n / 8);
      if (kind == LS_ACT_GELU_TANH)
        gelu8_bwd_kernel<TD, LS_ACT_GELU_TANH><<<gr, 256, 0, (hipStream_t)stream>>>(p, q, r, n / 8);
      else
        gelu8_bwd_kernel<TD, LS_ACT_GELU_ERF><<<gr, 256, 0, (hipStream_t)stream>>>(p, q, r, n / 8);
    };
    if (dt == LS_BF16) go((const bf16_t*)dg, (const bf16_t*)u, (bf16_t*)du);
    else go((const f16_t*)dg, (const f16_t*)u, (f16_t*)du);
    LS_CHECK_LAUNCH();
    return LS_OK;
  }
  gelu_bwd_kernel<<<grid_for(n), 256, 0, (hipStream_t)stream>>>(dg, u, du, dt, n, kind);
  LS_CHECK_LAUNCH();
  return LS_OK;
}
ls_status lsk_swiglu_fwd(const void* gu, void* a, int dt, int T, int F, void* stream) {
  LS_REQUIRE(gu && a && T > 0 && F > 0, "swiglu_fwd: bad argument");
  LS_REQUIRE(F % 8 == 0, "swiglu_fwd: d_ff must be a multiple of 8");
  const int gr = grid_for((size_t)T * F / 8);
  hipStream_t st = (hipStream_t)stream;
  if (dt == LS_F32) swiglu_fwd_kernel<float><<<gr, 256, 0, st>>>((const float*)gu, (float*)a, T, F);
  else if (dt == LS_BF16) swiglu_fwd_kernel<bf16_t><<<gr, 256, 0, st>>>((const bf16_t*)gu, (bf16_t*)a, T, F);
  else swiglu_fwd_kernel<f16_t><<<gr, 256, 0, st>>>((const f16_t*)gu, (f16_t*)a, T, F);
  LS_CHECK_LAUNCH();
  return LS_OK;
}
ls_status lsk_swiglu_bwd(const void* da, const void* gu, void* dgu, int dt, int T, int F, void* stream) {
  LS_REQUIRE(da && gu && dgu && T > 0 && F > 0, "swiglu_bwd: bad argument");
  LS_REQUIRE(F % 8 == 0, "swiglu_bwd: d_ff must be a multiple of 8");
  const int gr = grid_for((size_t)T * F / 8);
  hipStream_t st = (hipStream_t)stream;
  if (dt == LS_F32) swiglu_bwd_kernel<float><<<gr, 256, 0, st>>>((const float*)da, (const float*)gu, (float*)dgu, T, F);
  else if (dt == LS_BF16) swiglu_bwd_kernel<bf16_t><<<gr, 256, 0, st>>>((const bf16_t*)da, (const bf16_t*)gu, (bf16_t*)dgu, T, F);
  else swiglu_bwd_kernel<f16_t><<<gr, 256, 0, st>>>((const f16_t*)da, (const f16_t*)gu, (f16_t*)dgu, T, F);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

size_t lsk_colsum_partial_floats(int T, int N) { return (size_t)((T + CS_ROWS - 1) / CS_ROWS) * N; }

// the chunks' sums of x [T][N] into partial (lsk_colsum_partial_floats of them), for lsk_colsum_finish
ls_status lsk_colsum_partials(const void* x, int dt, int T, int N, long ld, float* partial, void* stream) {
  LS_REQUIRE(x && partial && T > 0 && N > 0 && ok_dtype(dt), "colsum: bad argument");
  hipStream_t st = (hipStream_t)stream;
  const int nchunk = (T + CS_ROWS - 1) / CS_ROWS;
  const dim3 grid((N + 255) / 256, nchunk);
  if (N % 8 == 0 && ld % 8 == 0 && aligned16(x)) {
    if (dt == LS_F32) colsum8_kernel<float><<<grid, 256, 0, st>>>((const float*)x, T, N, ld, partial);
    else if (dt == LS_BF16) colsum8_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t*)x, T, N, ld, partial);
    else colsum8_kernel<f16_t><<<grid, 256, 0, st>>>((const f16_t*)x, T, N, ld, partial);
  } else {
    colsum_kernel<<<grid, 256, 0, st>>>(x, dt, T, N, ld, partial);
  }
  LS_CHECK_LAUNCH();
  return LS_OK;
}
// out (+)= alpha * sum over the chunks, for n sums over the same T rows
ls_status lsk_colsum_finish(int n, const LsColsum* sums, int T, int accumulate, const float* alpha_dev, void* stream) {
  LS_REQUIRE(n >= 1 && n <= kMaxColsums && sums && T > 0, "colsum_finish: bad argument");
  ColsumSet set{n, {}, {}};
  for (int i = 0; i < n; ++i) {
    LS_REQUIRE(sums[i].partial && sums[i].out && sums[i].N > 0, "colsum_finish: bad argument");
    set.sum[i] = sums[i];
    set.first[i + 1] = set.first[i] + (sums[i].N + 31) / 32;
  }
  colsum_finish_kernel<<<set.first[n], 256, 0, (hipStream_t)stream>>>(set, (T + CS_ROWS - 1) / CS_ROWS, accumulate, alpha_dev);
  LS_CHECK_LAUNCH();
  return LS_OK;
}
ls_status lsk_colsum_scaled(const void* x, int dt, int T, int N, long ld, float* out, int accumulate,
                            float* partial, const float* alpha_dev, void* stream) {
  LS_REQUIRE(x && out && partial && T > 0 && N > 0 && ok_dtype(dt), "colsum: bad argument");
  LS_TRY(lsk_colsum_partials(x, dt, T, N, ld, partial, stream));
  const LsColsum one{partial, N, out};
  return lsk_colsum_finish(1, &one, T, accumulate, alpha_dev, stream);
}
ls_status lsk_colsum(const void* x, int dt, int T, int N, long ld, float* out, int accumulate,
                     float* partial, void* stream) {
  return lsk_colsum_scaled(x, dt, T, N, ld, out, accumulate, partial, nullptr, stream);
}

}  // extern "C"
