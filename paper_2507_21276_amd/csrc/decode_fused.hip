// Decode batches (at most 128 rows) and serving calls of a few hundred rows: the split-K projections leave fp32 partial
// products; the kernels here sum them in a fixed order and apply, in the same
// pass, the step that follows the projection in the block:
//   QKV projection   -> bias, rotary embedding of q and k, K/V page write
//   output / FFN-down -> bias, residual add, and the normalisation that comes next
//   FFN-up           -> bias, GELU or SwiGLU
// so that a decode step launches one small kernel per projection instead of a
// reduce kernel plus the elementwise kernel after it.
#include <type_traits>

#include "common.h"

ls_status gemm_dma_skinny_partials(int, int, int, int, const void*, long, const void*, long, float*, size_t, int*,
                                   hipStream_t);

namespace {

// N partial products at C columns, all of them requested before the first is added.  p is the same for the whole wavefront
// and `at`, in bytes, unsigned: a scalar address for each part and one register for a column's offset.  (The empty
// statement keeps the compiler from forming the addresses of all counts ahead of the switch below, in two vector
// registers each.)
template <int N, int C>
__device__ __forceinline__ void add_parts(f32x4 (&v)[C], const float* p, long stride, const uint32_t (&at)[C]) {
  f32x4 t[N][C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    uint32_t a = at[c];
    asm("" : "+v"(a));
#pragma unroll
    for (int i = 0; i < N; ++i) t[i][c] = *(const f32x4*)((const char*)(p + i * stride) + a);
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int i = 0; i < N; ++i) v[c] += t[i][c];
}
// Sums over the parts in ascending order, at one column or at two of the same row: eight loads at a time, and then the
// rest at once, so one or two round trips to memory for up to 16 parts at one column or eight at two.  A loop over a
// run-time count, unrolled by eight, fetched the rest (all of up to eight parts) one load and one wait after the other.
template <int C>
__device__ __forceinline__ void sum_partials(f32x4 (&v)[C], const float* row, int splits, long stride, const int (&col)[C]) {
  constexpr int G = 8 / C;
  uint32_t at[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    v[c] = f32x4{-0.f, -0.f, -0.f, -0.f};   // -0 + x is x, for every x
    at[c] = (uint32_t)col[c] * 4u;
  }
  for (; splits > G; splits -= G, row += G * stride) add_parts<G>(v, row, stride, at);
  if constexpr (C == 1) {
    switch (splits) {
      case 8: add_parts<8>(v, row, stride, at); return;
      case 7: add_parts<7>(v, row, stride, at); return;
      case 6: add_parts<6>(v, row, stride, at); return;
      case 5: add_parts<5>(v, row, stride, at); return;
    }
  }
  switch (splits) {
    case 4: add_parts<4>(v, row, stride, at); break;
    case 3: add_parts<3>(v, row, stride, at); break;
    case 2: add_parts<2>(v, row, stride, at); break;
    default: add_parts<1>(v, row, stride, at); break;
  }
}
__device__ __forceinline__ f32x4 sum_partials(const float* row, int splits, long stride, int col) {
  f32x4 v[1];
  sum_partials(v, row, splits, stride, {col});
  return v[0];
}

template <class TH> __device__ __forceinline__ void store4(TH* p, f32x4 v) {
  typedef TH V4 __attribute__((ext_vector_type(4)));
  V4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = from_f<TH>(v[e]);
  *(V4*)p = o;
}
template <> __device__ __forceinline__ void store4<float>(float* p, f32x4 v) { *(f32x4*)p = v; }

// four consecutive parameters: one load where they are bf16 and 8-byte aligned (c a multiple of 4)
__device__ __forceinline__ f32x4 load4_param(const void* p, int c, int dt) {
  f32x4 v;
  if (dt == LS_BF16 && ((uintptr_t)p & 7) == 0) {
    const bf16x4 b = *(const bf16x4*)((const bf16_t*)p + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (float)b[e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = load_as_f(p, c + e, dt);
  }
  return v;
}

// one workgroup of up to 1024 threads per row (a decode batch has few rows, so the parallelism has to
// come from the columns): x_out = sum of partials + bias + resid; h = norm(x_out) (kind 0 LayerNorm,
// 1 RMSNorm, < 0 none).  d % 4 == 0, d <= 8192 = 1024 threads x FN_MAX float4; FN float4 per thread.
// VEC: the parameters are bf16 and 8-byte aligned.  Their bits are requested before the partial sums and converted where
// they are used, so that they arrive under the sums; converted where they are loaded, the compiler waits for each of them
// first.  With FN = 2 the gain and shift are requested after the sums, for want of registers.
// At most 64 registers: two workgroups of 1024 threads on a compute unit.  As one kernel of 66 registers for both FN it
// held one of them, which cost calls of more rows than compute units and, more, calls beside a training task: decode of 64
// rows on eight blocks of d 4096 next to a forward and backward of 2048 tokens 5.27 ms, now 5.01; alone 2.605 -> 2.564;
// 32 rows on six blocks of d 768 347 -> 327 us.
constexpr int FN_MAX = 2;
template <class TH, bool VEC, int FN>
__global__ __launch_bounds__(1024, 8) void finish_resid_norm_kernel(const float* partial, int splits, int T, int d,
                                                                   const void* bias, const float* resid, float* x_out,
                                                                   int kind, const void* gamma, const void* beta,
                                                                   int pdt, float eps, TH* h) {
  __shared__ float red[16];
  const long row = blockIdx.x, stride = (long)T * d;
  const float* part = partial + row * d;
  f32x4 v[FN];
  bf16x4 ga[FN], be[FN];
  // a parameter that does not exist: bits of the partial sums in its place, not used (behind a branch on its pointer the
  // compiler waits for what is in flight)
  auto raw = [&](const void* p, int c) { return VEC ? *(const bf16x4*)((const bf16_t*)(p ? p : partial) + c) : bf16x4{}; };
  auto value = [&](const void* p, int c, bf16x4 bits) {
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = VEC ? (float)bits[e] : load_as_f(p, c + e, pdt);
    return r;
  };
  auto ask = [&] {
#pragma unroll
    for (int i = 0; i < FN; ++i) {
      const int c = (threadIdx.x + i * (int)blockDim.x) * 4;
      if (c < d) {
        ga[i] = raw(gamma, c);
        be[i] = raw(beta, c);
      }
    }
  };
  if constexpr (FN == 1) ask();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < FN; ++i) {
    const int c = (threadIdx.x + i * (int)blockDim.x) * 4;
    v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (c < d) {
      const bf16x4 bi = raw(bias, c);
      const f32x4 re = *(const f32x4*)((resid ? resid : partial) + row * d + c);
      v[i] = sum_partials(part, splits, stride, c);
      if (bias) v[i] += value(bias, c, bi);
      if (resid) v[i] += re;
      *(f32x4*)(x_out + row * d + c) = v[i];
      s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
    }
  }
  if (kind < 0) return;
  if constexpr (FN > 1) ask();   // under the block sums only: there are no registers for more
  const float mu = kind == 0 ? block_sum(s, red) / d : 0.f;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < FN; ++i)
    if ((threadIdx.x + i * (int)blockDim.x) * 4 < d)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = v[i][e] - mu;
        q += t * t;
      }
  const float r = 1.0f / sqrtf(block_sum(q, red) / d + eps);
#pragma unroll
  for (int i = 0; i < FN; ++i) {
    const int c = (threadIdx.x + i * (int)blockDim.x) * 4;
    if (c < d) {
      const f32x4 gv = value(gamma, c, ga[i]);
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (v[i][e] - mu) * r * gv[e];
      if (kind == 0 && beta) o += value(beta, c, be[i]);
      store4<TH>(h + row * d + c, o);
    }
  }
}

// The two kernels below: a workgroup takes a piece of one row, so that its addresses are scalar, and both columns of a
// pair are asked for at once.  With row and column divided out of one running index and a sum after the other they took 72
// registers (46 and 52 now); d 4096, 64 rows, two parts: gate and up 3.6 -> 3.2 us, q, k and v 4.3 -> 3.6 us.

// four hidden units per thread.  act LS_ACT_SWIGLU: the projection has 2F columns (gate, then up).
template <class TH>
__global__ __launch_bounds__(256) void finish_act_kernel(const float* partial, int splits, int T, int t0, int F, int pieces, int act,
                                                         const void* bias, int pdt, TH* out) {
  const int cols = act == LS_ACT_SWIGLU ? 2 * F : F;
  const long stride = (long)T * cols;
  const int f = (int)(blockIdx.x % pieces * blockDim.x + threadIdx.x) * 4;
  if (f >= F) return;
  const long t = t0 + blockIdx.x / pieces;
  const float* row = partial + t * cols;
  f32x4 o;
  if (act == LS_ACT_SWIGLU) {
    f32x4 v[2];
    sum_partials(v, row, splits, stride, {f, F + f});
    f32x4 a = v[0], u = v[1];
    if (bias) {
      a += load4_param(bias, f, pdt);
      u += load4_param(bias, F + f, pdt);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = a[e] / (1.f + __expf(-a[e])) * u[e];
  } else {
    f32x4 a = sum_partials(row, splits, stride, f);
    if (bias) a += load4_param(bias, f, pdt);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = gelu_f(a[e], act);
  }
  store4<TH>(out + t * F + f, o);
}

// one thread per (row, q / k / v, head, four pairs i .. i + 3 < dh / 2); rotation of q and k by
// pos[row] when a table is given; the values go to the qkv buffer and those of k and v also to
// the request's page slot.  dh % 8 == 0.
template <class TH>
__global__ __launch_bounds__(512) void finish_qkv_kernel(const float* partial, int splits, int T, int t0, int h, int dh, int pieces,
                                                         const void* bias, int pdt, const int32_t* pos, const int32_t* req,
                                                         const float* table, TH* qkv, TH* k_pool, TH* v_pool,
                                                         const int32_t* block_table, int max_pages, int page) {
  const int half = dh / 2, d = h * dh, q4 = half / 4;
  const long stride = (long)T * 3 * d;
  const int idx = (int)(blockIdx.x % pieces * blockDim.x + threadIdx.x);
  if (idx >= 3 * h * q4) return;
  const int i = idx % q4 * 4, hp = idx / q4;   // hp = part * h + head
  const int part = hp / h, head = hp % h;
  const int col = hp * dh + i;
  const long t = t0 + blockIdx.x / pieces;
  const float* row = partial + t * 3 * d;
  const int p = pos[t], rq = req[t];   // asked for ahead of the sums: the page and the rotation wait for them
  f32x4 v[2];
  sum_partials(v, row, splits, stride, {col, col + half});
  f32x4 xa = v[0], xb = v[1];
  if (bias) {
    xa += load4_param(bias, col, pdt);
    xb += load4_param(bias, col + half, pdt);
  }
  if (table && part < 2) {
    const float* tb = table + ((long)p * half + i) * 2;   // (cos, sin) pairs
    const f32x4 cs0 = *(const f32x4*)tb, cs1 = *(const f32x4*)(tb + 4);
    const f32x4 c = {cs0[0], cs0[2], cs1[0], cs1[2]}, sn = {cs0[1], cs0[3], cs1[1], cs1[3]};
    const f32x4 ra = xa * c - xb * sn, rb = xb * c + xa * sn;
    xa = ra; xb = rb;
  }
  typedef TH V4 __attribute__((ext_vector_type(4)));
  V4 oa, ob;
#pragma unroll
  for (int e = 0; e < 4; ++e) { oa[e] = from_f<TH>(xa[e]); ob[e] = from_f<TH>(xb[e]); }
  TH* to = qkv + t * 3 * d + col;
  *(V4*)to = oa;
  *(V4*)(to + half) = ob;
  if (part > 0) {
    TH* pool = part == 1 ? k_pool : v_pool;
    const int pg = block_table[(long)rq * max_pages + p / page];
    const long dst = (((long)pg * h + head) * page + p % page) * dh + i;
    *(V4*)(pool + dst) = oa;
    *(V4*)(pool + dst + half) = ob;
  }
}

// launches of the two kernels above for T rows of n threads each, in pieces of 256 to `widest` threads, of which those that
// leave the fewest lanes idle: go(first row, pieces of a row, workgroups, threads of one)
template <class Go>
void for_rows(int T, int n, int widest, Go go) {
  int pieces = 0, threads = 0;
  for (int p = (n + widest - 1) / widest; p <= (n + 255) / 256; ++p) {
    const int nt = ((n + p - 1) / p + 63) / 64 * 64;
    if (!pieces || (long)p * nt < (long)pieces * threads) { pieces = p; threads = nt; }
  }
  const int most = (1 << 22) / pieces > 0 ? (1 << 22) / pieces : 1;   // rows of a launch: fewer than 2^32 threads
  for (long t = 0; t < T; t += most) go((int)t, pieces, (unsigned)(T - t < most ? T - t : most) * (unsigned)pieces, threads);
}
inline bool half_type(int dt) { return dt == LS_BF16 || dt == LS_F16; }

}  // namespace

extern "C" {

ls_status lsk_gemm_partials(int op_dtype, int M, int N, int K, const void* X, long ldx, const void* W, long ldw,
                            float* partial, size_t partial_floats, int* splits, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_GEMM, stream);
  LS_REQUIRE(X && W && partial && splits, "gemm_partials: null argument");
  LS_REQUIRE(half_type(op_dtype), "gemm_partials: 16-bit operands only");
  LS_REQUIRE(M >= 1 && M <= 128 && N >= 64 && N % 4 == 0 && K >= 64 && K % 64 == 0,
             "gemm_partials: need 1 <= M <= 128, N >= 64 and a multiple of 4, K a multiple of 64 (M=%d N=%d K=%d)", M, N, K);
  LS_REQUIRE(ldx % 8 == 0 && ldw % 8 == 0 && (uintptr_t)X % 16 == 0 && (uintptr_t)W % 16 == 0 &&
                 (uintptr_t)partial % 16 == 0,
             "gemm_partials: operands must be 16-byte aligned with leading dimensions that are multiples of 8");
  LS_REQUIRE(partial_floats >= (size_t)M * N, "gemm_partials: the partial buffer holds %zu floats, one M x N result needs %zu",
             partial_floats, (size_t)M * N);
  const ls_status r = gemm_dma_skinny_partials(op_dtype, M, N, K, X, ldx, W, ldw, partial, partial_floats, splits,
                                               (hipStream_t)stream);
  LS_REQUIRE(r != LS_ESTATE, "gemm_partials: shape not covered (M=%d N=%d K=%d)", M, N, K);
  return r;
}

ls_status lsk_finish_resid_norm(const float* partial, int splits, int T, int d, const void* bias, const float* resid,
                                float* x_out, int kind, const void* gamma, const void* beta, int pdt, float eps,
                                void* h, int hdt, void* stream) {
  LsTimed timed(LSK_TIMED_FINISH, stream);
  LS_REQUIRE(partial && x_out && splits >= 1 && T > 0 && d > 0, "finish_resid_norm: bad argument");
  LS_REQUIRE(d % 4 == 0 && d <= 4096 * FN_MAX, "finish_resid_norm: d_model %d must be a multiple of 4, at most %d", d,
             4096 * FN_MAX);
  LS_REQUIRE(kind < 0 || (kind <= 1 && gamma && h), "finish_resid_norm: the normalisation needs gamma and an output");
  LS_REQUIRE((uintptr_t)partial % 16 == 0 && (uintptr_t)x_out % 16 == 0 && (!resid || (uintptr_t)resid % 16 == 0) &&
                 (!h || (uintptr_t)h % 16 == 0),
             "finish_resid_norm: buffers must be 16-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  int nt = (d / 4 + 63) / 64 * 64;   // one float4 per thread up to 4096 columns, two beyond
  if (nt > 1024) nt = 1024;
  const bool vec = pdt == LS_BF16 && (((uintptr_t)bias | (uintptr_t)gamma | (uintptr_t)beta) & 7) == 0;
  auto go = [&](auto* out) {
    typedef std::remove_pointer_t<decltype(out)> TH;
    auto run = [&](auto kernel) {
      kernel<<<T, nt, 0, st>>>(partial, splits, T, d, bias, resid, x_out, kind, gamma, beta, pdt, eps, out);
    };
    if (d <= 4096) vec ? run(finish_resid_norm_kernel<TH, true, 1>) : run(finish_resid_norm_kernel<TH, false, 1>);
    else vec ? run(finish_resid_norm_kernel<TH, true, FN_MAX>) : run(finish_resid_norm_kernel<TH, false, FN_MAX>);
  };
  if (hdt == LS_F32) go((float*)h);
  else if (hdt == LS_BF16) go((bf16_t*)h);
  else go((f16_t*)h);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_finish_act(const float* partial, int splits, int T, int F, int act, const void* bias, int pdt, void* out,
                         int odt, void* stream) {
  LsTimed timed(LSK_TIMED_FINISH, stream);
  LS_REQUIRE(partial && out && splits >= 1 && T > 0 && F > 0, "finish_act: bad argument");
  LS_REQUIRE(F % 4 == 0, "finish_act: d_ff must be a multiple of 4");
  LS_REQUIRE(act == LS_ACT_GELU_TANH || act == LS_ACT_GELU_ERF || act == LS_ACT_SWIGLU, "finish_act: unknown activation %d", act);
  LS_REQUIRE((uintptr_t)partial % 16 == 0 && (uintptr_t)out % 16 == 0, "finish_act: buffers must be 16-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  for_rows(T, F / 4, 256, [&](int t0, int pieces, unsigned wgs, int nt) {
    if (odt == LS_F32)
      finish_act_kernel<float><<<wgs, nt, 0, st>>>(partial, splits, T, t0, F, pieces, act, bias, pdt, (float*)out);
    else if (odt == LS_BF16)
      finish_act_kernel<bf16_t><<<wgs, nt, 0, st>>>(partial, splits, T, t0, F, pieces, act, bias, pdt, (bf16_t*)out);
    else
      finish_act_kernel<f16_t><<<wgs, nt, 0, st>>>(partial, splits, T, t0, F, pieces, act, bias, pdt, (f16_t*)out);
  });
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_finish_qkv(const float* partial, int splits, int T, int h, int dh, const void* bias, int pdt,
                         const int32_t* pos, const int32_t* req, const float* table, void* qkv, int dt, void* k_pool,
                         void* v_pool, const int32_t* block_table, int max_pages, int page, void* stream) {
  LsTimed timed(LSK_TIMED_FINISH, stream);
  LS_REQUIRE(partial && pos && req && qkv && k_pool && v_pool && block_table, "finish_qkv: null argument");
  LS_REQUIRE(splits >= 1 && T > 0 && h > 0 && dh > 0 && dh % 8 == 0 && max_pages > 0 && page > 0,
             "finish_qkv: bad size (head_dim must be a multiple of 8)");
  LS_REQUIRE((uintptr_t)partial % 16 == 0 && (uintptr_t)qkv % 8 == 0 && (uintptr_t)k_pool % 8 == 0 &&
                 (uintptr_t)v_pool % 8 == 0 && (!table || (uintptr_t)table % 16 == 0),
             "finish_qkv: buffers must be aligned to their vector accesses");
  LS_REQUIRE(half_type(dt), "finish_qkv: 16-bit q, k, v only");
  hipStream_t st = (hipStream_t)stream;
  for_rows(T, 3 * h * (dh / 8), 512, [&](int t0, int pieces, unsigned wgs, int nt) {
    if (dt == LS_BF16)
      finish_qkv_kernel<bf16_t><<<wgs, nt, 0, st>>>(partial, splits, T, t0, h, dh, pieces, bias, pdt, pos, req, table,
                                                   (bf16_t*)qkv, (bf16_t*)k_pool, (bf16_t*)v_pool, block_table, max_pages,
                                                   page);
    else
      finish_qkv_kernel<f16_t><<<wgs, nt, 0, st>>>(partial, splits, T, t0, h, dh, pieces, bias, pdt, pos, req, table,
                                                  (f16_t*)qkv, (f16_t*)k_pool, (f16_t*)v_pool, block_table, max_pages, page);
  });
  LS_CHECK_LAUNCH();
  return LS_OK;
}

}  // extern "C"
