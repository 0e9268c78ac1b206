// Serving calls of 5 to 32 rows on a small stage: each projection in one launch on the matrix cores, with the norm before
// it and what follows it inside.
//
// The weights of such a projection (1 - 5 MB) are a microsecond of HBM traffic; what a block takes is the number of its
// launches and of the round trips in each.  So nothing is split across workgroups: a workgroup owns 16 weight rows, its
// eight wavefronts share the contraction (straight into the fragments, up to 256 elements of a wavefront's share in flight at
// once: all of it up to a contraction of 2048), and their partial results are summed in LDS, in the order of the
// wavefronts.  A workgroup that needs the normalised rows normalises them for itself, into LDS, while its weights are on
// their way.  Five launches a block in place of nine: QKV (norm, bias, rotary embedding, page write), attention, output
// projection (bias, residual), FFN-up (norm, bias, activation), FFN-down (bias, residual).  Six where a call of 17 rows or
// more leaves FFN-down to the split products and their sum (block_forward_few).
//
// The 16 weight rows are two runs of eight: a rotary pair's halves, gate and up columns of the same units, or 16 in a row.
// Six blocks of d 768, nine launches a block -> these: 5 rows 262 -> 203 us, 16 rows 278 -> 219, 32 rows 289 -> 260.
#include "common.h"

namespace {

constexpr int NW = 8, NT = NW * 64;
constexpr int U = 4;                 // k chunks of 32 in flight ahead
constexpr int PS = 20;               // floats from one row of partial results to the next: four rows are 16 banks
constexpr int MAX_D = 1024;          // normalised columns: four float4 per lane
constexpr int PAD = 8;               // elements between normalised rows in LDS

enum { EPI_RESID = 0, EPI_ACT = 1, EPI_QKV = 2 };

struct RowsArgs {
  int T, N, K;            // rows, weight rows, contraction
  const void* W;          // [N][K]
  const void* in;         // [T][K] operand type, or null: the input is normalised here
  const float* x;         // [T][K]
  int kind;               // 0 LayerNorm, 1 RMSNorm
  const bf16_t *gamma, *beta;
  float eps;
  const bf16_t* bias;
  const float* resid;     // EPI_RESID: [T][N]
  float* out_f;
  void* out;              // EPI_ACT: [T][F];  EPI_QKV: [T][N]
  int act, F;
  int dh, h;              // EPI_QKV
  const int32_t *pos, *req;
  const float* table;
  void *k_pool, *v_pool;
  const int32_t* block_table;
  int max_pages, page;
};

template <class T> struct MfR;
template <> struct MfR<bf16_t> {
  static __device__ __forceinline__ f32x4 run(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct MfR<f16_t> {
  static __device__ __forceinline__ f32x4 run(f16x8 a, f16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

template <class T, int MB, int EPI, bool NORM>
__global__ __launch_bounds__(NT) void rows_kernel(RowsArgs g) {
  typedef typename vec8<T>::type V8;
  typedef T V4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 15, kg = lane >> 4, K = g.K;
  const bool gated = EPI == EPI_ACT && g.act == LS_ACT_SWIGLU;
  const int half = g.dh / 2, tile = blockIdx.x;
  // the first rows of the two runs of eight
  const int per_part = half / 8, hp = EPI == EPI_QKV ? tile / per_part : 0, i0 = EPI == EPI_QKV ? tile % per_part * 8 : 0;
  const int r0 = EPI == EPI_QKV ? hp * g.dh + i0 : tile * (gated ? 8 : 16);
  const int r1 = r0 + (EPI == EPI_QKV ? half : gated ? g.F : 8);
  const int nch = K / 32, c_lo = wave * nch / NW, c_hi = (wave + 1) * nch / NW;
  const T* w = (const T*)g.W + (long)((r & 8 ? r1 : r0) + (r & 7)) * K + kg * 8;
  auto fetch_w = [&](V8 (&b)[U], int c) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c_hi) b[u] = __builtin_nontemporal_load((const V8*)(w + (long)(c + u) * 32));   // uniform
  };
  V8 b0[U], b1[U];
  fetch_w(b0, c_lo);

  // this thread's results: row m, columns p of both runs; what the epilogue adds is requested now
  const int p = threadIdx.x & 7, m = threadIdx.x >> 3;
  const bool mine = m < g.T;
  float add0 = 0.f, add1 = 0.f, rc = 1.f, rs = 0.f;
  int at = 0, slot = 0;
  if (mine) {
    if (g.bias) { add0 = (float)g.bias[r0 + p]; add1 = (float)g.bias[r1 + p]; }
    if constexpr (EPI == EPI_RESID) {
      add0 += g.resid[(long)m * g.N + r0 + p];
      add1 += g.resid[(long)m * g.N + r1 + p];
    }
    if constexpr (EPI == EPI_QKV) {
      at = g.pos[m];
      slot = g.block_table[(long)g.req[m] * g.max_pages + at / g.page];
      if (g.table && hp / g.h < 2) {
        rc = g.table[((long)at * half + i0 + p) * 2];
        rs = g.table[((long)at * half + i0 + p) * 2 + 1];
      }
    }
  }

  T* hs = (T*)smem;   // NORM: [T][K + PAD]
  if constexpr (NORM) {
    constexpr int NV = MAX_D / 256, RB = MB * 2;   // rows of a wavefront, all requested together
    bf16x4 ga[NV], be[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (lane + i * 64) * 4;
      ga[i] = be[i] = bf16x4{};
      if (c < K) {
        ga[i] = *(const bf16x4*)(g.gamma + c);
        if (g.kind == 0 && g.beta) be[i] = *(const bf16x4*)(g.beta + c);
      }
    }
    for (int row0 = wave; row0 < g.T; row0 += NW * RB) {
      f32x4 v[RB][NV];
      float mu[RB], q[RB];
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const float* x = g.x + (long)min(row0 + j * NW, g.T - 1) * K;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int c = (lane + i * 64) * 4;
          v[j][i] = c < K ? *(const f32x4*)(x + c) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        mu[j] = q[j] = 0.f;
        if (g.kind == 0) {
#pragma unroll
          for (int i = 0; i < NV; ++i) mu[j] += (v[j][i][0] + v[j][i][1]) + (v[j][i][2] + v[j][i][3]);
          mu[j] = wave_total(mu[j]) / K;
        }
      }
#pragma unroll
      for (int j = 0; j < RB; ++j) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
          if ((lane + i * 64) * 4 < K)
#pragma unroll
            for (int e = 0; e < 4; ++e) q[j] += (v[j][i][e] - mu[j]) * (v[j][i][e] - mu[j]);
        q[j] = 1.0f / sqrtf(wave_total(q[j]) / K + g.eps);
      }
#pragma unroll
      for (int j = 0; j < RB; ++j)
        if (row0 + j * NW < g.T)
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            const int c = (lane + i * 64) * 4;
            if (c < K) {
              V4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = from_f<T>((v[j][i][e] - mu[j]) * q[j] * (float)ga[i][e] + (float)be[i][e]);
              *(V4*)(hs + (long)(row0 + j * NW) * (K + PAD) + c) = o;
            }
          }
    }
    __syncthreads();
  }

  // rows past the last repeat it and are not stored
  const T* a_row[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int row = min(i * 16 + r, g.T - 1);
    a_row[i] = (NORM ? hs + (long)row * (K + PAD) : (const T*)g.in + (long)row * K) + kg * 8;
  }
  f32x4 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto fetch_a = [&](V8 (&a)[MB][U], int c) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c_hi)
#pragma unroll
        for (int i = 0; i < MB; ++i) a[i][u] = *(const V8*)(a_row[i] + (long)(c + u) * 32);
  };
  auto multiply = [&](const V8 (&a)[MB][U], const V8 (&b)[U], int c) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c_hi)   // uniform
#pragma unroll
        for (int i = 0; i < MB; ++i) acc[i] = MfR<T>::run(a[i][u], b[u], acc[i]);
  };
  {
    V8 a0[MB][U], a1[MB][U];
    fetch_a(a0, c_lo);
    for (int c = c_lo; c < c_hi; c += 2 * U) {
      if (c + U < c_hi) {
        fetch_w(b1, c + U);
        fetch_a(a1, c + U);
      }
      multiply(a0, b0, c);
      if (c + U < c_hi) {
        if (c + 2 * U < c_hi) {
          fetch_w(b0, c + 2 * U);
          fetch_a(a0, c + 2 * U);
        }
        multiply(a1, b1, c + U);
      }
    }
  }
  if (NORM) __syncthreads();   // the normalised rows make room for the partial results
  float* part = (float*)smem;  // [NW][MB * 16][PS]
  // block i: lane -> column lane & 15, register e -> row 4 (lane >> 4) + e
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) part[(wave * MB * 16 + i * 16 + kg * 4 + e) * PS + r] = acc[i][e];
  __syncthreads();
  if (!mine) return;
  float xa = 0.f, xb = 0.f;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    xa += part[(q * MB * 16 + m) * PS + p];
    xb += part[(q * MB * 16 + m) * PS + p + 8];
  }
  xa += add0;
  xb += add1;
  if constexpr (EPI == EPI_RESID) {
    g.out_f[(long)m * g.N + r0 + p] = xa;
    g.out_f[(long)m * g.N + r1 + p] = xb;
  } else if constexpr (EPI == EPI_ACT) {
    T* out = (T*)g.out + (long)m * g.F + r0 + p;
    if (gated) {
      out[0] = from_f<T>(xa / (1.f + __expf(-xa)) * xb);
    } else {
      out[0] = from_f<T>(gelu_f(xa, g.act));
      out[8] = from_f<T>(gelu_f(xb, g.act));
    }
  } else {
    const int part_of = hp / g.h, head = hp % g.h, i = i0 + p;
    if (g.table && part_of < 2) {
      const float ra = xa * rc - xb * rs, rb = xb * rc + xa * rs;
      xa = ra; xb = rb;
    }
    const T oa = from_f<T>(xa), ob = from_f<T>(xb);
    T* qo = (T*)g.out + (long)m * g.N + (long)hp * g.dh + i;
    qo[0] = oa;
    qo[half] = ob;
    if (part_of > 0) {
      T* dst = (T*)(part_of == 1 ? g.k_pool : g.v_pool) + (((long)slot * g.h + head) * g.page + at % g.page) * g.dh + i;
      dst[0] = oa;
      dst[half] = ob;
    }
  }
}

template <class T, int MB, int EPI, bool NORM>
ls_status launch(const RowsArgs& g, hipStream_t st) {
  const size_t sums = (size_t)NW * MB * 16 * PS * 4, rows = NORM ? (size_t)g.T * (g.K + PAD) * sizeof(T) : 0;
  const size_t lds = sums > rows ? sums : rows;
  static bool attr_set = false;
  if (!attr_set) {
    LS_CHECK_HIP(hipFuncSetAttribute((const void*)rows_kernel<T, MB, EPI, NORM>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     160 * 1024));
    attr_set = true;
  }
  rows_kernel<T, MB, EPI, NORM><<<(unsigned)(g.N / 16), NT, lds, st>>>(g);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

template <int EPI, bool NORM>
ls_status run(const RowsArgs& g, int dt, hipStream_t st) {
  auto go = [&](auto t) {
    typedef decltype(t) T;
    if (g.T <= 16) return launch<T, 1, EPI, NORM>(g, st);
    return launch<T, 2, EPI, NORM>(g, st);
  };
  return dt == LS_BF16 ? go(bf16_t{}) : go(f16_t{});
}

bool common_ok(int dt, int T, int N, int K, const void* W) {
  return (dt == LS_BF16 || dt == LS_F16) && T >= 1 && T <= 32 && N > 0 && N % 16 == 0 && K >= 32 && K % 32 == 0 && W &&
         (uintptr_t)W % 16 == 0;
}
bool norm_ok(int K, const float* x, const void* gamma, const void* beta) {
  return K <= MAX_D && x && gamma && (uintptr_t)x % 16 == 0 && (uintptr_t)gamma % 8 == 0 && (uintptr_t)beta % 8 == 0;
}

}  // namespace

// Whether the kernels below cover a block's projections and are the better ones for it: while a workgroup's rows are few
// (QKV of d 768: 5.6 us at 5 rows, 8.0 at 32, 14.9 at 64 against 5.7 + 3.6 for a split product and its sum) and the weights
// few enough to be latency.  Four blocks over short contexts, nine launches a block -> these, us at 5 and 32 rows: d 256 143 ->
// 81, 149 -> 114; d 512 161 -> 98, 165 -> 124; d 1024 172 -> 125, 181 -> 157; gated, d 1024 over 4096 166 -> 127, 176 -> 175.
bool decode_rows_covers(int dt, int param_dtype, int T, int d, int F, int dh) {
  return (dt == LS_BF16 || dt == LS_F16) && param_dtype == LS_BF16 && T >= 1 && T <= 32 && d % 32 == 0 && d <= MAX_D &&
         F % 32 == 0 && F <= 4 * MAX_D && dh % 16 == 0;
}

extern "C" {

// qkv[T, 3 d] = rope(norm(x) Wqkv^T + bias); the rows of k and v also go to their page slots
ls_status lsk_rows_norm_qkv(int dt, int T, int h, int dh, const float* x, int kind, const void* gamma, const void* beta,
                            float eps, const void* W, const void* bias, const int32_t* pos, const int32_t* req,
                            const float* table, void* qkv, void* k_pool, void* v_pool, const int32_t* block_table,
                            int max_pages, int page, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  const int d = h * dh;
  LS_REQUIRE(common_ok(dt, T, 3 * d, d, W) && norm_ok(d, x, gamma, beta) && dh % 16 == 0 && pos && req && qkv && k_pool &&
                 v_pool && block_table && max_pages > 0 && page > 0 && (uintptr_t)k_pool % 8 == 0 && (uintptr_t)v_pool % 8 == 0,
             "rows_norm_qkv: bad argument");
  RowsArgs g{};
  g.T = T; g.N = 3 * d; g.K = d; g.W = W; g.x = x; g.kind = kind;
  g.gamma = (const bf16_t*)gamma; g.beta = (const bf16_t*)beta; g.eps = eps; g.bias = (const bf16_t*)bias;
  g.out = qkv; g.dh = dh; g.h = h; g.pos = pos; g.req = req; g.table = table;
  g.k_pool = k_pool; g.v_pool = v_pool; g.block_table = block_table; g.max_pages = max_pages; g.page = page;
  return run<EPI_QKV, true>(g, dt, (hipStream_t)stream);
}

// out[T, F] = act(norm(x) Wup^T + bias)
ls_status lsk_rows_norm_act(int dt, int T, int d, int F, int act, const float* x, int kind, const void* gamma,
                            const void* beta, float eps, const void* W, const void* bias, void* out, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  const int N = act == LS_ACT_SWIGLU ? 2 * F : F;
  LS_REQUIRE(common_ok(dt, T, N, d, W) && norm_ok(d, x, gamma, beta) && out && F % 8 == 0, "rows_norm_act: bad argument");
  RowsArgs g{};
  g.T = T; g.N = N; g.K = d; g.W = W; g.x = x; g.kind = kind;
  g.gamma = (const bf16_t*)gamma; g.beta = (const bf16_t*)beta; g.eps = eps; g.bias = (const bf16_t*)bias;
  g.out = out; g.act = act; g.F = F; g.dh = 16; g.h = 1;
  return run<EPI_ACT, true>(g, dt, (hipStream_t)stream);
}

// out[T, N] (fp32) = resid + in W^T + bias
ls_status lsk_rows_resid(int dt, int T, int N, int K, const void* in, const void* W, const void* bias, const float* resid,
                         float* out, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  LS_REQUIRE(common_ok(dt, T, N, K, W) && in && resid && out && (uintptr_t)in % 16 == 0, "rows_resid: bad argument");
  RowsArgs g{};
  g.T = T; g.N = N; g.K = K; g.W = W; g.in = in; g.bias = (const bf16_t*)bias; g.resid = resid; g.out_f = out;
  g.dh = 16; g.h = 1;
  return run<EPI_RESID, false>(g, dt, (hipStream_t)stream);
}

}  // extern "C"
