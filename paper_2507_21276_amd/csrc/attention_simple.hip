// Plain (no matrix core) attention kernels: forward over contiguous sequences
// or over the paged pool, and the training backward.  One wavefront owns one
// (query row, head) pair - or one (key row, head) pair in the dK/dV kernel -
// and works in two passes: lanes over keys for the scores (kept in LDS), then
// lanes over head dimensions for the weighted sums.  Deterministic: no atomics.
// These kernels serve the fp32 stage mode and any shape the MFMA kernels do
// not cover.
#include <initializer_list>

#include "common.h"

namespace {

struct KvView {
  // contiguous: keys of the row's sequence live in qkv rows seq0 .. seq0+pos
  // paged: keys live in the pool, found through the request's block table
  const void* qkv;
  const void* k_pool;
  const void* v_pool;
  const int32_t* block_table;
  int paged, dt, h, dh, d, max_pages, page;
};

__device__ __forceinline__ size_t k_index(const KvView& kv, int seq0, int req, int j, int head) {
  if (!kv.paged) return (size_t)(seq0 + j) * 3 * kv.d + kv.d + (size_t)head * kv.dh;
  const int pg = kv.block_table[(size_t)req * kv.max_pages + j / kv.page];
  return (((size_t)pg * kv.h + head) * kv.page + j % kv.page) * kv.dh;
}
__device__ __forceinline__ size_t v_index(const KvView& kv, int seq0, int req, int j, int head) {
  if (!kv.paged) return (size_t)(seq0 + j) * 3 * kv.d + 2 * kv.d + (size_t)head * kv.dh;
  return k_index(kv, seq0, req, j, head);
}

// grid: (ceil(T*h / 4)), block 256 (4 wavefronts), dynamic LDS: 4 * (max_ctx + dh) floats
__global__ __launch_bounds__(256) void attn_fwd_simple_kernel(KvView kv, int T, int L,
                                                              const int32_t* pos_arr,
                                                              const int32_t* req_arr, int max_ctx,
                                                              void* o, float* lse) {
  extern __shared__ float smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long item = (long)blockIdx.x * 4 + wave;
  if (item >= (long)T * kv.h) return;
  const int t = item / kv.h, head = item % kv.h;
  float* sc = smem + (size_t)wave * (max_ctx + kv.dh);
  float* qs = sc + max_ctx;
  int pos, req = 0, seq0 = 0;
  if (kv.paged) { pos = pos_arr[t]; req = req_arr[t]; }
  else { pos = t % L; seq0 = t - pos; }
  const int nkeys = pos + 1;
  const float scale = 1.0f / sqrtf((float)kv.dh);
  const void* kbase = kv.paged ? kv.k_pool : kv.qkv;
  const void* vbase = kv.paged ? kv.v_pool : kv.qkv;
  for (int c = lane; c < kv.dh; c += 64)
    qs[c] = load_as_f(kv.qkv, (size_t)t * 3 * kv.d + (size_t)head * kv.dh + c, kv.dt);
  __builtin_amdgcn_wave_barrier();
  float m = -INFINITY;
  for (int j = lane; j < nkeys; j += 64) {
    const size_t ki = k_index(kv, seq0, req, j, head);
    float s = 0.f;
    for (int c = 0; c < kv.dh; ++c) s = fmaf(qs[c], load_as_f(kbase, ki + c, kv.dt), s);
    s *= scale;
    sc[j] = s;
    m = fmaxf(m, s);
  }
  m = wave_max(m);
  float l = 0.f;
  for (int j = lane; j < nkeys; j += 64) {
    const float p = expf(sc[j] - m);
    sc[j] = p;
    l += p;
  }
  l = wave_sum(l);
  __builtin_amdgcn_wave_barrier();
  const float inv = 1.0f / l;
  for (int c = lane; c < kv.dh; c += 64) {
    float acc = 0.f;
    for (int j = 0; j < nkeys; ++j)
      acc = fmaf(sc[j], load_as_f(vbase, v_index(kv, seq0, req, j, head) + c, kv.dt), acc);
    store_from_f(o, (size_t)t * kv.d + (size_t)head * kv.dh + c, kv.dt, acc * inv);
  }
  if (lse && lane == 0) lse[(size_t)t * kv.h + head] = m + logf(l);
}

// D[t, head] = sum_c dO * O
__global__ void attn_dvec_kernel(const void* o, const void* dO, int dt, long n_items, int dh, float* dvec) {
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (item >= n_items) return;
  float s = 0.f;
  for (int c = lane; c < dh; c += 64)
    s += load_as_f(o, item * dh + c, dt) * load_as_f(dO, item * dh + c, dt);
  s = wave_sum(s);
  if (lane == 0) dvec[item] = s;
}

// dQ: one wavefront per (query row, head)
__global__ __launch_bounds__(256) void attn_bwd_dq_simple_kernel(const void* qkv, const void* dO,
                                                                 const float* lse, const float* dvec,
                                                                 int dt, int T, int L, int h, int dh,
                                                                 void* dqkv) {
  extern __shared__ float smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long item = (long)blockIdx.x * 4 + wave;
  if (item >= (long)T * h) return;
  const int t = item / h, head = item % h, d = h * dh;
  float* ds = smem + (size_t)wave * (L + 2 * dh);
  float* qs = ds + L;
  float* gs = qs + dh;
  const int pos = t % L, seq0 = t - pos;
  const float scale = 1.0f / sqrtf((float)dh);
  for (int c = lane; c < dh; c += 64) {
    qs[c] = load_as_f(qkv, (size_t)t * 3 * d + (size_t)head * dh + c, dt);
    gs[c] = load_as_f(dO, (size_t)t * d + (size_t)head * dh + c, dt);
  }
  __builtin_amdgcn_wave_barrier();
  const float ls = lse[item], dv = dvec[item];
  for (int j = lane; j <= pos; j += 64) {
    const size_t ki = (size_t)(seq0 + j) * 3 * d + d + (size_t)head * dh;
    float s = 0.f, dp = 0.f;
    for (int c = 0; c < dh; ++c) {
      s = fmaf(qs[c], load_as_f(qkv, ki + c, dt), s);
      dp = fmaf(gs[c], load_as_f(qkv, ki + d + c, dt), dp);
    }
    ds[j] = expf(s * scale - ls) * (dp - dv);
  }
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < dh; c += 64) {
    float acc = 0.f;
    for (int j = 0; j <= pos; ++j)
      acc = fmaf(ds[j], load_as_f(qkv, (size_t)(seq0 + j) * 3 * d + d + (size_t)head * dh + c, dt), acc);
    store_from_f(dqkv, (size_t)t * 3 * d + (size_t)head * dh + c, dt, acc * scale);
  }
}

// dK, dV: one wavefront per (key row, head); queries i >= j of the same sequence
__global__ __launch_bounds__(256) void attn_bwd_dkv_simple_kernel(const void* qkv, const void* dO,
                                                                  const float* lse, const float* dvec,
                                                                  int dt, int T, int L, int h, int dh,
                                                                  void* dqkv) {
  extern __shared__ float smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long item = (long)blockIdx.x * 4 + wave;
  if (item >= (long)T * h) return;
  const int t = item / h, head = item % h, d = h * dh;
  float* ps = smem + (size_t)wave * (2 * L + 2 * dh);
  float* ds = ps + L;
  float* ks = ds + L;
  float* vs = ks + dh;
  const int pos = t % L, seq0 = t - pos;
  const float scale = 1.0f / sqrtf((float)dh);
  for (int c = lane; c < dh; c += 64) {
    ks[c] = load_as_f(qkv, (size_t)t * 3 * d + d + (size_t)head * dh + c, dt);
    vs[c] = load_as_f(qkv, (size_t)t * 3 * d + 2 * d + (size_t)head * dh + c, dt);
  }
  __builtin_amdgcn_wave_barrier();
  for (int i = pos + lane; i < L; i += 64) {
    const size_t qi = (size_t)(seq0 + i) * 3 * d + (size_t)head * dh;
    const size_t gi = (size_t)(seq0 + i) * d + (size_t)head * dh;
    float s = 0.f, dp = 0.f;
    for (int c = 0; c < dh; ++c) {
      s = fmaf(ks[c], load_as_f(qkv, qi + c, dt), s);
      dp = fmaf(vs[c], load_as_f(dO, gi + c, dt), dp);
    }
    const long it = (long)(seq0 + i) * h + head;
    const float p = expf(s * scale - lse[it]);
    ps[i] = p;
    ds[i] = p * (dp - dvec[it]);
  }
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < dh; c += 64) {
    float ak = 0.f, av = 0.f;
    for (int i = pos; i < L; ++i) {
      ak = fmaf(ds[i], load_as_f(qkv, (size_t)(seq0 + i) * 3 * d + (size_t)head * dh + c, dt), ak);
      av = fmaf(ps[i], load_as_f(dO, (size_t)(seq0 + i) * d + (size_t)head * dh + c, dt), av);
    }
    store_from_f(dqkv, (size_t)t * 3 * d + d + (size_t)head * dh + c, dt, ak * scale);
    store_from_f(dqkv, (size_t)t * 3 * d + 2 * d + (size_t)head * dh + c, dt, av);
  }
}

// ---- fp32, head_dim 32 / 64 / 128 --------------------------------------------------------------------------------
// A workgroup of four wavefronts owns one (query row, head) pair - or one (key row, head) pair - and the wavefronts share
// its keys (its queries) in batches of 16.  A lane holds four consecutive head dimensions of one token, so a load is 16
// bytes a lane and covers whole rows, a batch's loads are all in flight together, and what has been loaded serves both the
// scores and the weighted sums (the kernels above read a row of K four bytes a lane, one lane per key, and walk the
// keys one after the other for the sums: a chain of up to 2 L load latencies).  Parts are merged in the order of the
// wavefronts: deterministic.  2 x 64 tokens, 4 heads of 32: forward 26.8 -> 4.0 us, backward 45.2 + a launch for
// rowsum(dO * O) -> 4.6; 2048 tokens, 12 heads of 64: 4508 -> 485, 29992 -> 1490; 64 requests of 4000 over pages, 16 heads of 128:
// 6002 -> 701.
template <int DH> struct F32Lanes {
  static constexpr int LPT = DH / 4, TPL = 64 / LPT, UN = 16 / TPL;   // lanes per token, tokens per load, loads per batch
  static __device__ __forceinline__ float dot(f32x4 a, f32x4 b) {
    float v = fmaf(a[3], b[3], fmaf(a[2], b[2], fmaf(a[1], b[1], a[0] * b[0])));
#pragma unroll
    for (int off = 1; off < LPT; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
  }
  static __device__ __forceinline__ f32x4 over_tokens(f32x4 v) {   // sum over the token groups of the wavefront
#pragma unroll
    for (int off = LPT; off < 64; off <<= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], off, 64);
    return v;
  }
};

template <int DH, bool PAGED>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(KvView kv, int L, const int32_t* pos_arr, const int32_t* req_arr,
                                                           float* o, float* lse) {
  typedef F32Lanes<DH> Ln;
  constexpr int LPT = Ln::LPT, TPL = Ln::TPL, UN = Ln::UN;
  __shared__ float s_m[4], s_l[4], s_o[4][DH];
  const int t = blockIdx.x / kv.h, head = blockIdx.x % kv.h;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane % LPT, tg = lane / LPT;
  const int d = kv.d;
  const float* qkv = (const float*)kv.qkv;
  const int pos = PAGED ? pos_arr[t] : t % L, req = PAGED ? req_arr[t] : 0, seq0 = PAGED ? 0 : t - pos;
  const int nkeys = pos + 1;
  const float scale = 1.0f / sqrtf((float)DH);
  const f32x4 q = *(const f32x4*)(qkv + (size_t)t * 3 * d + (size_t)head * DH + sub * 4);
  float m = -INFINITY, l = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int j0 = wave * 16; j0 < nkeys; j0 += 64) {
    f32x4 kx[UN], vx[UN];
    float s[UN], mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int j = min(j0 + u * TPL + tg, nkeys - 1);   // slots past the context are never touched
      if (PAGED) {
        const size_t at = k_index(kv, 0, req, j, head) + sub * 4;
        kx[u] = *(const f32x4*)((const float*)kv.k_pool + at);
        vx[u] = *(const f32x4*)((const float*)kv.v_pool + at);
      } else {
        const float* p = qkv + (size_t)(seq0 + j) * 3 * d + d + (size_t)head * DH + sub * 4;
        kx[u] = *(const f32x4*)p;
        vx[u] = *(const f32x4*)(p + d);
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      s[u] = Ln::dot(q, kx[u]) * scale;
      if (j0 + u * TPL + tg >= nkeys) s[u] = -INFINITY;
      mx = fmaxf(mx, s[u]);
    }
#pragma unroll
    for (int off = LPT; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    const float m_new = fmaxf(m, mx);
    // a batch whose scores have all overflowed to -inf counts for nothing beside a finite score, before it or after it
    const float ref = m_new == -INFINITY ? 0.f : m_new, alpha = expf(m - ref);
    l *= alpha;
    acc *= alpha;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const bool in = j0 + u * TPL + tg < nkeys;
      const float p = in ? expf(s[u] - ref) : 0.f;
      l += p;
      // what stands in for a token past the end may be infinite: 0 times it must not reach the sum
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(p, in ? vx[u][e] : 0.f, acc[e]);
    }
    m = m_new;
  }
#pragma unroll
  for (int off = LPT; off < 64; off <<= 1) l += __shfl_xor(l, off, 64);
  acc = Ln::over_tokens(acc);
  if (tg == 0) *(f32x4*)&s_o[wave][sub * 4] = acc;
  if (lane == 0) { s_m[wave] = m; s_l[wave] = l; }
  __syncthreads();
  if (threadIdx.x < DH) {
    const float mm = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
    float ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (w * 16 >= nkeys) break;   // a wavefront that saw no key
      const float f = expf(s_m[w] - mm);
      ll += s_l[w] * f;
      oo += s_o[w][threadIdx.x] * f;
    }
    o[(size_t)t * d + (size_t)head * DH + threadIdx.x] = oo * (1.0f / ll);
    if (lse && threadIdx.x == 0) lse[(size_t)t * kv.h + head] = mm + logf(ll);
  }
}

// blockIdx.y 0: dQ of a query row;  1: dK and dV of a key row.  D = rowsum(dO * O) is taken where it is needed.
template <int DH>
__global__ __launch_bounds__(256) void attn_bwd_f32_kernel(const float* qkv, const float* o, const float* dO,
                                                           const float* lse, int L, int h, float* dqkv) {
  typedef F32Lanes<DH> Ln;
  constexpr int LPT = Ln::LPT, TPL = Ln::TPL, UN = Ln::UN;
  __shared__ float s_a[4][DH], s_b[4][DH];
  const int t = blockIdx.x / h, head = blockIdx.x % h, d = h * DH;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane % LPT, tg = lane / LPT;
  const int pos = t % L, seq0 = t - pos;
  const float scale = 1.0f / sqrtf((float)DH);
  const size_t hc = (size_t)head * DH + sub * 4;
  const float *qp = qkv + hc, *op = o + hc, *gp = dO + hc;   // row r at r * 3 d, r * d, r * d
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
  if (blockIdx.y == 0) {
    const f32x4 q = *(const f32x4*)(qp + (size_t)t * 3 * d), g = *(const f32x4*)(gp + (size_t)t * d);
    const float dv = Ln::dot(g, *(const f32x4*)(op + (size_t)t * d)), ls = lse[(size_t)t * h + head];
    for (int j0 = wave * 16; j0 <= pos; j0 += 64) {
      f32x4 kx[UN], vx[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const float* p = qp + (size_t)(seq0 + min(j0 + u * TPL + tg, pos)) * 3 * d + d;
        kx[u] = *(const f32x4*)p;
        vx[u] = *(const f32x4*)(p + d);
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const float s = Ln::dot(q, kx[u]), dp = Ln::dot(g, vx[u]);
        const float ds = j0 + u * TPL + tg <= pos ? expf(s * scale - ls) * (dp - dv) : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = fmaf(ds, kx[u][e], a[e]);
      }
    }
  } else {
    const f32x4 k = *(const f32x4*)(qp + (size_t)t * 3 * d + d), v = *(const f32x4*)(qp + (size_t)t * 3 * d + 2 * d);
    for (int i0 = pos + wave * 16; i0 < L; i0 += 64) {
      f32x4 qx[UN], gx[UN], ox[UN];
      float ls[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const size_t r = seq0 + min(i0 + u * TPL + tg, L - 1);
        qx[u] = *(const f32x4*)(qp + r * 3 * d);
        gx[u] = *(const f32x4*)(gp + r * d);
        ox[u] = *(const f32x4*)(op + r * d);
        ls[u] = lse[r * h + head];
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const float s = Ln::dot(k, qx[u]), dp = Ln::dot(v, gx[u]), dv = Ln::dot(gx[u], ox[u]);
        const bool in = i0 + u * TPL + tg < L;
        const float p = in ? expf(s * scale - ls[u]) : 0.f, ds = in ? p * (dp - dv) : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = fmaf(ds, in ? qx[u][e] : 0.f, a[e]);
          b[e] = fmaf(p, in ? gx[u][e] : 0.f, b[e]);
        }
      }
    }
  }
  a = Ln::over_tokens(a);
  if (blockIdx.y == 1) b = Ln::over_tokens(b);
  if (tg == 0) {
    *(f32x4*)&s_a[wave][sub * 4] = a;
    *(f32x4*)&s_b[wave][sub * 4] = b;
  }
  __syncthreads();
  const int c = threadIdx.x;
  if (c < DH) {
    float* out = dqkv + (size_t)t * 3 * d + (size_t)head * DH + c;
    const float sa = (s_a[0][c] + s_a[1][c]) + (s_a[2][c] + s_a[3][c]);
    if (blockIdx.y == 0) {
      out[0] = sa * scale;
    } else {
      out[d] = sa * scale;
      out[2 * d] = (s_b[0][c] + s_b[1][c]) + (s_b[2][c] + s_b[3][c]);
    }
  }
}

bool f32_covers(int dt, int dh, long items, std::initializer_list<const void*> p) {
  if (dt != LS_F32 || (dh != 32 && dh != 64 && dh != 128) || items > (1 << 22)) return false;   // a launch has 2^32 threads at most
  for (const void* q : p)
    if ((uintptr_t)q % 16 != 0) return false;
  return true;
}

template <bool PAGED>
ls_status launch_fwd_f32(const KvView& kv, int T, int L, const int32_t* pos, const int32_t* req, float* o, float* lse,
                         hipStream_t st) {
  const dim3 grid((unsigned)((size_t)T * kv.h));
  if (kv.dh == 32) attn_fwd_f32_kernel<32, PAGED><<<grid, 256, 0, st>>>(kv, L, pos, req, o, lse);
  else if (kv.dh == 64) attn_fwd_f32_kernel<64, PAGED><<<grid, 256, 0, st>>>(kv, L, pos, req, o, lse);
  else attn_fwd_f32_kernel<128, PAGED><<<grid, 256, 0, st>>>(kv, L, pos, req, o, lse);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

// scatter the new K/V rows into their pages: one thread per (row, head, 8-lane of dh)
__global__ void kv_write_kernel(const void* qkv, int dt, int T, int h, int dh, const int32_t* pos,
                                const int32_t* req, void* k_pool, void* v_pool,
                                const int32_t* block_table, int max_pages, int page) {
  const size_t n = (size_t)T * h * dh;
  const int d = h * dh;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int c = idx % dh, head = (idx / dh) % h;
    const size_t t = idx / ((size_t)dh * h);
    const int p = pos[t];
    const int pg = block_table[(size_t)req[t] * max_pages + p / page];
    const size_t dst = (((size_t)pg * h + head) * page + p % page) * dh + c;
    const size_t src = t * 3 * d + d + (size_t)head * dh + c;
    if (dt == LS_F32) {
      ((float*)k_pool)[dst] = ((const float*)qkv)[src];
      ((float*)v_pool)[dst] = ((const float*)qkv)[src + d];
    } else {
      ((uint16_t*)k_pool)[dst] = ((const uint16_t*)qkv)[src];
      ((uint16_t*)v_pool)[dst] = ((const uint16_t*)qkv)[src + d];
    }
  }
}

// serving: rotary embedding of q and k (optional) fused with the K/V page write;
// one thread per (row, head, pair i < dh/2)
__global__ void rope_kv_kernel(void* qkv, int dt, int T, int h, int dh, const int32_t* pos,
                               const int32_t* req, const float* table, void* k_pool, void* v_pool,
                               const int32_t* block_table, int max_pages, int page) {
  const int half = dh / 2, d = h * dh;
  const size_t n = (size_t)T * h * half;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int i = idx % half, head = (idx / half) % h;
    const size_t t = idx / ((size_t)half * h);
    const int p = pos[t];
    const size_t qi = t * 3 * d + (size_t)head * dh + i;
    float ka = load_as_f(qkv, qi + d, dt), kb = load_as_f(qkv, qi + d + half, dt);
    if (table) {
      const float c = table[((size_t)p * half + i) * 2], s = table[((size_t)p * half + i) * 2 + 1];
      const float qa = load_as_f(qkv, qi, dt), qb = load_as_f(qkv, qi + half, dt);
      store_from_f(qkv, qi, dt, qa * c - qb * s);
      store_from_f(qkv, qi + half, dt, qb * c + qa * s);
      const float ra = ka * c - kb * s, rb = kb * c + ka * s;
      ka = ra; kb = rb;
      store_from_f(qkv, qi + d, dt, ka);
      store_from_f(qkv, qi + d + half, dt, kb);
    }
    const int pg = block_table[(size_t)req[t] * max_pages + p / page];
    const size_t dst = (((size_t)pg * h + head) * page + p % page) * dh + i;
    store_from_f(k_pool, dst, dt, ka);
    store_from_f(k_pool, dst + half, dt, kb);
    if (dt == LS_F32) {
      ((float*)v_pool)[dst] = ((const float*)qkv)[qi + 2 * d];
      ((float*)v_pool)[dst + half] = ((const float*)qkv)[qi + 2 * d + half];
    } else {
      ((uint16_t*)v_pool)[dst] = ((const uint16_t*)qkv)[qi + 2 * d];
      ((uint16_t*)v_pool)[dst + half] = ((const uint16_t*)qkv)[qi + 2 * d + half];
    }
  }
}

// The same for 16-bit data, head_dim % 8 == 0: one thread per (row, q / k / v, head, four pairs
// i .. i + 3 < dh / 2), 8-byte accesses.  v and (without a table) q are not rewritten in place.
template <class TH>
__global__ void rope_kv_vec_kernel(TH* qkv, int T, int h, int dh, const int32_t* pos, const int32_t* req,
                                   const float* table, TH* k_pool, TH* v_pool, const int32_t* block_table,
                                   int max_pages, int page) {
  typedef TH V4 __attribute__((ext_vector_type(4)));
  const int half = dh / 2, d = h * dh, q4 = half / 4;
  const size_t n = (size_t)T * 3 * h * q4;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx % q4) * 4, hp = (int)((idx / q4) % (3 * h));   // hp = part * h + head
    const int part = hp / h, head = hp % h;
    const size_t t = idx / ((size_t)q4 * 3 * h);
    if (part == 0 && !table) continue;
    const size_t qi = t * 3 * d + (size_t)hp * dh + i;
    V4 a = *(const V4*)(qkv + qi), b = *(const V4*)(qkv + qi + half);
    const int p = pos[t];
    if (table && part < 2) {
      const float* tb = table + ((size_t)p * half + i) * 2;   // (cos, sin) pairs
      const f32x4 cs0 = *(const f32x4*)tb, cs1 = *(const f32x4*)(tb + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float c = e < 2 ? cs0[2 * e] : cs1[2 * (e - 2)], sn = e < 2 ? cs0[2 * e + 1] : cs1[2 * (e - 2) + 1];
        const float xa = to_f(a[e]), xb = to_f(b[e]);
        a[e] = from_f<TH>(xa * c - xb * sn);
        b[e] = from_f<TH>(xb * c + xa * sn);
      }
      *(V4*)(qkv + qi) = a;
      *(V4*)(qkv + qi + half) = b;
    }
    if (part > 0) {
      TH* pool = part == 1 ? k_pool : v_pool;
      const int pg = block_table[(size_t)req[t] * max_pages + p / page];
      const size_t dst = (((size_t)pg * h + head) * page + p % page) * dh + i;
      *(V4*)(pool + dst) = a;
      *(V4*)(pool + dst + half) = b;
    }
  }
}

// The longest context that the entry points take: one whose scores the kernels of any type and head_dim hold in LDS
ls_status context_fits(size_t bytes) {
  LS_REQUIRE(bytes <= 160 * 1024, "attention: context too long for the plain kernel (%zu bytes of LDS)", bytes);
  return LS_OK;
}
ls_status set_lds(const void* fn, size_t bytes) {
  LS_TRY(context_fits(bytes));
  if (bytes > 48 * 1024)
    LS_CHECK_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  return LS_OK;
}

}  // namespace

extern "C" {

ls_status lsk_attn_fwd_simple(const void* qkv, int dt, int B, int L, int h, int dh, void* o,
                              float* lse, void* stream) {
  LS_REQUIRE(qkv && o && B > 0 && L > 0 && h > 0 && dh > 0, "attn_fwd: bad argument");
  KvView kv{qkv, nullptr, nullptr, nullptr, 0, dt, h, dh, h * dh, 0, 1};
  const int T = B * L;
  const size_t lds = 4 * (size_t)(L + dh) * sizeof(float);
  LS_TRY(context_fits(lds));
  const long items = (long)T * h;
  if (f32_covers(dt, dh, items, {qkv}))
    return launch_fwd_f32<false>(kv, T, L, nullptr, nullptr, (float*)o, lse, (hipStream_t)stream);
  LS_TRY(set_lds((const void*)attn_fwd_simple_kernel, lds));
  attn_fwd_simple_kernel<<<(unsigned)((items + 3) / 4), 256, lds, (hipStream_t)stream>>>(
      kv, T, L, nullptr, nullptr, L, o, lse);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_attn_bwd_simple(const void* qkv, const void* o, const void* dO, const float* lse,
                              int dt, int B, int L, int h, int dh, void* dqkv, float* dvec,
                              void* stream) {
  LS_REQUIRE(qkv && o && dO && lse && dqkv && dvec && B > 0 && L > 0, "attn_bwd: bad argument");
  const int T = B * L;
  const long items = (long)T * h;
  hipStream_t st = (hipStream_t)stream;
  if (f32_covers(dt, dh, items, {qkv, o, dO})) {
    LS_TRY(context_fits(4 * (size_t)(2 * L + 2 * dh) * sizeof(float)));
    const dim3 grid((unsigned)items, 2);
    if (dh == 32) attn_bwd_f32_kernel<32><<<grid, 256, 0, st>>>((const float*)qkv, (const float*)o, (const float*)dO, lse, L, h, (float*)dqkv);
    else if (dh == 64) attn_bwd_f32_kernel<64><<<grid, 256, 0, st>>>((const float*)qkv, (const float*)o, (const float*)dO, lse, L, h, (float*)dqkv);
    else attn_bwd_f32_kernel<128><<<grid, 256, 0, st>>>((const float*)qkv, (const float*)o, (const float*)dO, lse, L, h, (float*)dqkv);
    LS_CHECK_LAUNCH();
    return LS_OK;
  }
  attn_dvec_kernel<<<(unsigned)((items + 3) / 4), 256, 0, st>>>(o, dO, dt, items, dh, dvec);
  LS_CHECK_LAUNCH();
  size_t lds = 4 * (size_t)(L + 2 * dh) * sizeof(float);
  LS_TRY(set_lds((const void*)attn_bwd_dq_simple_kernel, lds));
  attn_bwd_dq_simple_kernel<<<(unsigned)((items + 3) / 4), 256, lds, st>>>(qkv, dO, lse, dvec, dt, T, L, h,
                                                                          dh, dqkv);
  LS_CHECK_LAUNCH();
  lds = 4 * (size_t)(2 * L + 2 * dh) * sizeof(float);
  LS_TRY(set_lds((const void*)attn_bwd_dkv_simple_kernel, lds));
  attn_bwd_dkv_simple_kernel<<<(unsigned)((items + 3) / 4), 256, lds, st>>>(qkv, dO, lse, dvec, dt, T, L, h,
                                                                           dh, dqkv);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_kv_write(const void* qkv, int dt, int T, int h, int dh, const int32_t* pos,
                       const int32_t* req, void* k_pool, void* v_pool, const int32_t* block_table,
                       int max_pages, int page, void* stream) {
  LS_REQUIRE(qkv && pos && req && k_pool && v_pool && block_table && T > 0, "kv_write: bad argument");
  const size_t n = (size_t)T * h * dh;
  size_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  kv_write_kernel<<<(unsigned)g, 256, 0, (hipStream_t)stream>>>(qkv, dt, T, h, dh, pos, req, k_pool, v_pool,
                                                                block_table, max_pages, page);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_rope_kv_write(void* qkv, int dt, int T, int h, int dh, const int32_t* pos, const int32_t* req,
                            const float* table, void* k_pool, void* v_pool, const int32_t* block_table,
                            int max_pages, int page, void* stream) {
  LS_REQUIRE(qkv && pos && req && k_pool && v_pool && block_table && T > 0 && dh % 2 == 0,
             "rope_kv_write: bad argument");
  if (dt != LS_F32 && dh % 8 == 0 && ((uintptr_t)qkv | (uintptr_t)k_pool | (uintptr_t)v_pool) % 8 == 0 &&
      (!table || (uintptr_t)table % 16 == 0)) {
    const size_t nv = (size_t)T * 3 * h * (dh / 8);
    size_t gv = (nv + 255) / 256;
    if (gv > 8192) gv = 8192;
    if (dt == LS_BF16)
      rope_kv_vec_kernel<bf16_t><<<(unsigned)gv, 256, 0, (hipStream_t)stream>>>(
          (bf16_t*)qkv, T, h, dh, pos, req, table, (bf16_t*)k_pool, (bf16_t*)v_pool, block_table, max_pages, page);
    else
      rope_kv_vec_kernel<f16_t><<<(unsigned)gv, 256, 0, (hipStream_t)stream>>>(
          (f16_t*)qkv, T, h, dh, pos, req, table, (f16_t*)k_pool, (f16_t*)v_pool, block_table, max_pages, page);
    LS_CHECK_LAUNCH();
    return LS_OK;
  }
  const size_t n = (size_t)T * h * (dh / 2);
  size_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  rope_kv_kernel<<<(unsigned)g, 256, 0, (hipStream_t)stream>>>(qkv, dt, T, h, dh, pos, req, table, k_pool,
                                                               v_pool, block_table, max_pages, page);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status lsk_attn_paged_simple(const void* qkv, int dt, int T, int h, int dh, const int32_t* pos,
                                const int32_t* req, const void* k_pool, const void* v_pool,
                                const int32_t* block_table, int max_pages, int page, int max_ctx,
                                void* o, void* stream) {
  LS_REQUIRE(qkv && pos && req && k_pool && v_pool && block_table && o && T > 0 && max_ctx > 0,
             "attn_paged: bad argument");
  KvView kv{qkv, k_pool, v_pool, block_table, 1, dt, h, dh, h * dh, max_pages, page};
  const size_t lds = 4 * (size_t)(max_ctx + dh) * sizeof(float);
  LS_TRY(context_fits(lds));
  const long items = (long)T * h;
  if (f32_covers(dt, dh, items, {qkv, k_pool, v_pool}))
    return launch_fwd_f32<true>(kv, T, 0, pos, req, (float*)o, nullptr, (hipStream_t)stream);
  LS_TRY(set_lds((const void*)attn_fwd_simple_kernel, lds));
  attn_fwd_simple_kernel<<<(unsigned)((items + 3) / 4), 256, lds, (hipStream_t)stream>>>(
      kv, T, 0, pos, req, max_ctx, o, nullptr);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

}  // extern "C"
