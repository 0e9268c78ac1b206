// Serving calls of one to four rows: the projections as matrix-vector products on the vector units.
//
// Such a call reads every weight once for a handful of rows, so it is bound by HBM (large stages) or by the number
// of launches (small ones).  The matrix-core kernels pad the rows to a 64-row tile, have to split the contraction to
// fill the chip and need a kernel after each product that sums the partial results.  Here a wavefront owns four
// weight rows and a share of the contraction: all of its loads are whole 1 KB lines, the whole weight matrix is in
// flight over the chip at once, and nothing is left to sum across workgroups, so what precedes and follows a
// projection runs in the same kernel:
//   QKV:      normalisation of the input, bias, rotary embedding of q and k, K/V page write
//   output:   bias, residual                       FFN-down: the same
//   FFN-up:   normalisation of the input, bias, GELU or SwiGLU
// Every workgroup of a normalising kernel normalises the rows for itself (they are in L2), after it has issued its
// first weight loads.  Sums are fp32, in an order that depends on the sizes alone.
//
// Per decode step of one row, matrix-core kernels -> these: six blocks of d 768 309 -> 148 us; eight of d 4096 with
// 1537 cached tokens 1028 -> 749 us (180 MB of FFN-up weights in 34 us, 5.3 TB/s).
#include "common.h"

namespace {

constexpr int NT = 512, NW = NT / 64;   // threads, wavefronts
constexpr int R = 4;                    // weight rows per wavefront
constexpr int CHUNK = 512;              // elements of a weight row per load (64 lanes x 16 bytes)
constexpr int NV = 4;                   // float4 per thread and row in the normalisation: d <= NT * 4 * NV = 8192

enum { EPI_RESID = 0, EPI_ACT = 1, EPI_QKV = 2 };

struct GemvArgs {
  int T, N, K;            // rows, weight rows, contraction
  int wk;                 // wavefronts that share a unit of four weight rows (1, 2, 4, 8)
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

template <class T, int M, int EPI, bool NORM>
__global__ __launch_bounds__(NT) void gemv_kernel(GemvArgs g) {
  typedef typename vec8<T>::type V8;
  typedef T V4 __attribute__((ext_vector_type(4)));
  extern __shared__ __attribute__((aligned(16))) char smem[];
  T* hs = (T*)smem;                      // NORM: [M][K]
  __shared__ float red[NW][R * M];
  __shared__ float nred[M][NW];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int K = g.K, wk = g.wk, per_wg = NW / wk, units = g.N / R, groups = (units + per_wg - 1) / per_wg;
  const int kw = wave % wk;
  const int half = g.dh / 2, per_head = half / 2;
  const bool gated = EPI == EPI_ACT && g.act == LS_ACT_SWIGLU;
  const int nc = (K + CHUNK - 1) / CHUNK;

  V8 wv[2][R];
  const T* w[R];
  auto fetch = [&](int b, int c) {
    const int k = min(c * CHUNK + lane * 8, K - 8);
#pragma unroll
    for (int j = 0; j < R; ++j) wv[b][j] = __builtin_nontemporal_load((const V8*)(w[j] + k));
  };
  // the first loads of a group.  A unit's rows: r0, r0 + 1 and the two that belong to them (the other half of the
  // rotary pairs, the up column of a gate column, the next two).  The last group's units may not exist: they repeat
  // the last one and store nothing.
  auto start = [&](int group) {
    const int unit = min(group * per_wg + wave / wk, units - 1);
    const long r0 = EPI == EPI_QKV ? (long)(unit / per_head) * g.dh + unit % per_head * 2 : (long)unit * (gated ? 2 : R);
    const long r1 = r0 + (EPI == EPI_QKV ? half : gated ? g.F : 2);
    w[0] = (const T*)g.W + r0 * K;
    w[1] = w[0] + K;
    w[2] = (const T*)g.W + r1 * K;
    w[3] = w[2] + K;
    if (kw < nc) fetch(0, kw);
    if (kw + wk < nc) fetch(1, kw + wk);
  };
  int group = blockIdx.x;
  start(group);

  if constexpr (NORM) {
    f32x4 v[M][NV];
    float s[M], q[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const float* x = g.x + (long)min(m, g.T - 1) * K;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = (threadIdx.x + i * NT) * 4;
        v[m][i] = c < K ? *(const f32x4*)(x + c) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    bf16x4 ga[NV], be[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (threadIdx.x + i * NT) * 4;
      ga[i] = be[i] = bf16x4{};
      if (c < K) {
        ga[i] = *(const bf16x4*)(g.gamma + c);
        if (g.kind == 0 && g.beta) be[i] = *(const bf16x4*)(g.beta + c);
      }
    }
    // sums over the workgroup, of all rows between one pair of barriers
    auto sums = [&](float (&t)[M]) {
#pragma unroll
      for (int m = 0; m < M; ++m) t[m] = wave_total(t[m]);
      __syncthreads();
      if (lane == 0)
#pragma unroll
        for (int m = 0; m < M; ++m) nred[m][wave] = t[m];
      __syncthreads();
#pragma unroll
      for (int m = 0; m < M; ++m) {
        t[m] = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) t[m] += nred[m][i];
      }
    };
#pragma unroll
    for (int m = 0; m < M; ++m) s[m] = 0.f;
    if (g.kind == 0) {
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int i = 0; i < NV; ++i) s[m] += (v[m][i][0] + v[m][i][1]) + (v[m][i][2] + v[m][i][3]);
      sums(s);
#pragma unroll
      for (int m = 0; m < M; ++m) s[m] /= K;
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      q[m] = 0.f;
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if ((int)(threadIdx.x + i * NT) * 4 < K)
#pragma unroll
          for (int e = 0; e < 4; ++e) q[m] += (v[m][i][e] - s[m]) * (v[m][i][e] - s[m]);
    }
    sums(q);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const float r = 1.0f / sqrtf(q[m] / K + g.eps);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = (threadIdx.x + i * NT) * 4;
        if (c < K) {
          V4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = from_f<T>((v[m][i][e] - s[m]) * r * (float)ga[i][e] + (float)be[i][e]);
          *(V4*)(hs + m * K + c) = o;
        }
      }
    }
    __syncthreads();
  }

  // results of a group: local unit lu, row m, and a single column or a pair of them
  const bool paired = EPI == EPI_QKV || gated;
  const int ncol = paired ? 2 : R;
  const int p = threadIdx.x % ncol, m_out = threadIdx.x / ncol % M, lu = threadIdx.x / (ncol * M);

  for (; group < groups; group += gridDim.x) {
    float acc[R * M];   // [j][m]
#pragma unroll
    for (int i = 0; i < R * M; ++i) acc[i] = 0.f;
    auto multiply = [&](int b, int c) {
      const int k = c * CHUNK + lane * 8;
      // lanes past the end of the contraction hold zeros on both sides
      V8 xv[M];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const T* src = NORM ? hs + m * K : (const T*)g.in + (long)min(m, g.T - 1) * K;
        xv[m] = *(const V8*)(src + min(k, K - 8));
        if (k >= K) xv[m] = V8{};
      }
#pragma unroll
      for (int j = 0; j < R; ++j) {
        if (k >= K) wv[b][j] = V8{};
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int m = 0; m < M; ++m) acc[j * M + m] = fmaf((float)wv[b][j][e], (float)xv[m][e], acc[j * M + m]);
      }
    };
    for (int c = kw; c < nc; c += 2 * wk) {
      multiply(0, c);
      if (c + 2 * wk < nc) fetch(0, c + 2 * wk);
      if (c + wk < nc) multiply(1, c + wk);
      if (c + 3 * wk < nc) fetch(1, c + 3 * wk);
    }
    if (group + (int)gridDim.x < groups) start(group + gridDim.x);
    // sum over the lanes: each step halves the values a lane holds and sends it the other lane's half, until lane l
    // has the value l / LPV of all of them, in part
    constexpr int LPV = 64 / (R * M);
#pragma unroll
    for (int n = R * M / 2, o = 32; n >= 1; n /= 2, o /= 2)
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const bool up = lane & o;
        const float keep = up ? acc[i + n] : acc[i], give = up ? acc[i] : acc[i + n];
        acc[i] = keep + __shfl_xor(give, o, 64);
      }
#pragma unroll
    for (int o = LPV / 2; o >= 1; o /= 2) acc[0] += __shfl_xor(acc[0], o, 64);
    if (lane % LPV == 0) red[wave][lane / LPV] = acc[0];
    __syncthreads();

    const int u = group * per_wg + lu, m = m_out;
    if (lu < per_wg && u < units && m < g.T) {
      auto total = [&](int j) {
        float v = 0.f;
        for (int q = 0; q < wk; ++q) v += red[lu * wk + q][j * M + m];
        return v;
      };
      if constexpr (EPI == EPI_RESID) {
        const long n = (long)u * R + p, i = (long)m * g.N + n;
        float v = total(p);
        if (g.bias) v += (float)g.bias[n];
        g.out_f[i] = v + g.resid[i];
      } else if constexpr (EPI == EPI_ACT) {
        const int f = u * (gated ? 2 : R) + p;
        float a = total(p), o;
        if (g.bias) a += (float)g.bias[f];
        if (gated) {
          float up = total(p + 2);
          if (g.bias) up += (float)g.bias[g.F + f];
          o = a / (1.f + __expf(-a)) * up;
        } else {
          o = gelu_f(a, g.act);
        }
        ((T*)g.out)[(long)m * g.F + f] = from_f<T>(o);
      } else {
        const int hp = u / per_head, i = u % per_head * 2 + p, part = hp / g.h, head = hp % g.h;
        float xa = total(p), xb = total(p + 2);
        if (g.bias) {
          xa += (float)g.bias[(long)hp * g.dh + i];
          xb += (float)g.bias[(long)hp * g.dh + i + half];
        }
        const int at = g.pos[m];
        if (g.table && part < 2) {
          const float c = g.table[((long)at * half + i) * 2], sn = g.table[((long)at * half + i) * 2 + 1];
          const float ra = xa * c - xb * sn, rb = xb * c + xa * sn;
          xa = ra; xb = rb;
        }
        const T oa = from_f<T>(xa), ob = from_f<T>(xb);
        T* qo = (T*)g.out + (long)m * g.N + (long)hp * g.dh + i;
        qo[0] = oa;
        qo[half] = ob;
        if (part > 0) {
          const int pg = g.block_table[(long)g.req[m] * g.max_pages + at / g.page];
          T* dst = (T*)(part == 1 ? g.k_pool : g.v_pool) + (((long)pg * g.h + head) * g.page + at % g.page) * g.dh + i;
          dst[0] = oa;
          dst[half] = ob;
        }
      }
    }
    __syncthreads();   // the partial sums are read before the next group's
  }
}

template <class T, int M, int EPI, bool NORM>
ls_status launch(const GemvArgs& g, hipStream_t st) {
  const int per_wg = NW / g.wk, units = g.N / R, groups = (units + per_wg - 1) / per_wg;
  // a normalising workgroup takes several groups of units, so that the chip normalises the rows 768 times at most
  // and not once per group; every workgroup the same number
  const int each = NORM ? (groups + 767) / 768 : 1;
  const size_t lds = NORM ? (size_t)M * g.K * sizeof(T) : 0;
  gemv_kernel<T, M, EPI, NORM><<<(unsigned)((groups + each - 1) / each), NT, lds, st>>>(g);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

template <int EPI, bool NORM>
ls_status run(GemvArgs g, int dt, hipStream_t st) {
  // One to four loads of a row for each of the wavefronts that share it.  More of them (two loads each) for rows of
  // 4097 - 8192 elements is slower, as a workgroup then covers half as many rows between two barriers: four blocks of d
  // 5120 510 -> 539 us for one row and 550 -> 609 for two, two blocks of d 6144 247 -> 268, of d 8192 299 -> 302.
  const int nc = (g.K + CHUNK - 1) / CHUNK;
  g.wk = nc <= 1 ? 1 : nc <= 4 ? 2 : nc <= 16 ? 4 : 8;
  auto go = [&](auto t) {
    typedef decltype(t) T;
    if (g.T == 1) return launch<T, 1, EPI, NORM>(g, st);
    if (g.T == 2) return launch<T, 2, EPI, NORM>(g, st);
    return launch<T, 4, EPI, NORM>(g, st);
  };
  return dt == LS_BF16 ? go(bf16_t{}) : go(f16_t{});
}

bool common_ok(int dt, int T, int N, int K, const void* W) {
  return (dt == LS_BF16 || dt == LS_F16) && T >= 1 && T <= 4 && N > 0 && N % R == 0 && K >= 8 && K % 8 == 0 && W &&
         (uintptr_t)W % 16 == 0;
}

}  // namespace

// Whether the kernels below cover a block and are the better ones for it.  One and two rows: always (per step of four
// large blocks, d 4096, matrix-core kernels -> these: 1 row 493 -> 369 us, 2 rows 508 -> 410; d 5120: 660 -> 514, 683 ->
// 576).  Three and four: where the launches count and not the weights (six blocks of d 768: 335 -> 219 us); at d 4096 the
// conversions and multiplications of the vector units take longer than the weights (513 -> 570 us); at d 2048
// (four blocks) 309 -> 267 us.
bool decode_gemv_covers(int dt, int param_dtype, int T, int d, int F, int dh) {
  return (dt == LS_BF16 || dt == LS_F16) && param_dtype == LS_BF16 && T >= 1 && T <= (d <= 2048 ? 4 : 2) && d % 8 == 0 &&
         F % 8 == 0 && dh % 8 == 0 && d <= NT * 4 * NV;
}

extern "C" {

// qkv[T, 3 d] = rope(norm(x) Wqkv^T + bias); the rows of k and v also go to their page slots
ls_status lsk_gemv_norm_qkv(int dt, int T, int h, int dh, const float* x, int kind, const void* gamma, const void* beta,
                            float eps, const void* W, const void* bias, const int32_t* pos, const int32_t* req,
                            const float* table, void* qkv, void* k_pool, void* v_pool, const int32_t* block_table,
                            int max_pages, int page, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  const int d = h * dh;
  LS_REQUIRE(common_ok(dt, T, 3 * d, d, W) && decode_gemv_covers(dt, LS_BF16, T, d, 8, dh) && x && gamma && pos && req && qkv &&
                 k_pool && v_pool && block_table && max_pages > 0 && page > 0 && (uintptr_t)x % 16 == 0 &&
                 (uintptr_t)gamma % 8 == 0 && (uintptr_t)beta % 8 == 0,
             "gemv_norm_qkv: bad argument");
  GemvArgs g{};
  g.T = T; g.N = 3 * d; g.K = d; g.W = W; g.x = x; g.kind = kind;
  g.gamma = (const bf16_t*)gamma; g.beta = (const bf16_t*)beta; g.eps = eps; g.bias = (const bf16_t*)bias;
  g.out = qkv; g.dh = dh; g.h = h; g.pos = pos; g.req = req; g.table = table;
  g.k_pool = k_pool; g.v_pool = v_pool; g.block_table = block_table; g.max_pages = max_pages; g.page = page;
  return run<EPI_QKV, true>(g, dt, (hipStream_t)stream);
}

// out[T, F] = act(norm(x) Wup^T + bias)
ls_status lsk_gemv_norm_act(int dt, int T, int d, int F, int act, const float* x, int kind, const void* gamma,
                            const void* beta, float eps, const void* W, const void* bias, void* out, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  const int N = act == LS_ACT_SWIGLU ? 2 * F : F;
  LS_REQUIRE(common_ok(dt, T, N, d, W) && decode_gemv_covers(dt, LS_BF16, T, d, F, 8) && x && gamma && out && (uintptr_t)x % 16 == 0 &&
                 (uintptr_t)gamma % 8 == 0 && (uintptr_t)beta % 8 == 0,
             "gemv_norm_act: bad argument");
  GemvArgs g{};
  g.T = T; g.N = N; g.K = d; g.W = W; g.x = x; g.kind = kind;
  g.gamma = (const bf16_t*)gamma; g.beta = (const bf16_t*)beta; g.eps = eps; g.bias = (const bf16_t*)bias;
  g.out = out; g.act = act; g.F = F; g.dh = 8; g.h = 1;
  return run<EPI_ACT, true>(g, dt, (hipStream_t)stream);
}

// out[T, N] (fp32) = resid + in W^T + bias
ls_status lsk_gemv_resid(int dt, int T, int N, int K, const void* in, const void* W, const void* bias, const float* resid,
                         float* out, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  LS_REQUIRE(common_ok(dt, T, N, K, W) && in && resid && out && (uintptr_t)in % 16 == 0, "gemv_resid: bad argument");
  GemvArgs g{};
  g.T = T; g.N = N; g.K = K; g.W = W; g.in = in; g.bias = (const bf16_t*)bias; g.resid = resid; g.out_f = out;
  g.dh = 8; g.h = 1;
  return run<EPI_RESID, false>(g, dt, (hipStream_t)stream);
}

}  // extern "C"
