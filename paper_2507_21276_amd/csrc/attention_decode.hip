// Ragged paged decode attention: one query row per request, keys gathered page
// by page from the pool.  Bandwidth-bound: every K and V byte is read once, in
// 16-byte-per-lane loads that cover whole pages contiguously (a page of one
// head is page_size * head_dim 16-bit elements, 4 KB for 16 x 128).
//
// Work split: a workgroup of 4, 8 or 16 wavefronts owns one (row, head, split); the
// split's tokens are dealt to the wavefronts in groups of eight loads (4 KB of K, 4 KB of V).  A lane holds 8
// consecutive head-dimension elements of one token; the q.k dot product is
// finished with a butterfly over the head_dim/8 lanes that share a token.
// A wavefront has the loads of two groups in flight, and the block table is read a group further ahead: with one group, and
// its pages looked up when it is its turn, a wavefront waited for a table entry and then for the keys, and a chip full of
// them reached 6.2 TB/s.  us, one group in flight and the plan of then -> now: 32 requests of 512 tokens, 12 heads of 64:
// 15.6 -> 13.2; 64 of up to 2048, 32 heads of 128: 191 -> 173 (6.5 TB/s); 128 of up to 4096, 40 heads: 992 -> 902 (6.6).
// Softmax is online per wavefront; the wavefronts' partial (max, sum, output) triples
// are merged in LDS, and when the context was split across workgroups a second
// kernel merges the per-split partials (deterministic, no atomics).
#include <mutex>

#include "common.h"

namespace {

// Scratch of the entry point that allocates nothing (lsk_attn_paged_noalloc): the per-split partial results
// (output, maximum, sum; head_dim + 2 floats) of contexts split over workgroups.  8 MiB hold 16 131 (row, head,
// split) items at head_dim 128: every launch below 2048 (row, head) pairs (fewer than 4096 items), and e.g. 64
// rows x 32 heads with contexts up to 3584 tokens.  One copy per GPU, held until the process ends; every call
// on a GPU shares it.
constexpr size_t kStaticScratchFloats = (size_t)2 << 20;   // 8 MiB
static __device__ __align__(256) float scratch[kStaticScratchFloats];

template <class T, int DH, int NW>
__global__ __launch_bounds__(NW * 64) void decode_attn_kernel(
    const T* __restrict__ qkv, const int32_t* __restrict__ pos_arr, const int32_t* __restrict__ req_arr,
    const T* __restrict__ k_pool, const T* __restrict__ v_pool, const int32_t* __restrict__ block_table,
    int max_pages, int page, int h, int nsplit, int chunk_pages, float scale_log2, T* __restrict__ o,
    float* __restrict__ partial) {
  constexpr int LPT = DH / 8;        // lanes per token
  constexpr int TPL = 64 / LPT;      // tokens per wave-wide load (1 KB)
  constexpr int G = 4;               // loads of K, and of V, per group
  typedef typename vec8<T>::type V8;
  __shared__ float s_m[NW], s_l[NW];
  __shared__ float s_o[NW][DH];

  const int t = blockIdx.x / h, head = blockIdx.x % h, split = blockIdx.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int sub = lane % LPT;        // which 8-element chunk of the head dimension
  const int tok_in = lane / LPT;     // token within a load
  const int d = h * DH;
  const int nkeys = pos_arr[t] + 1;
  const int req = req_arr[t];
  const V8 qv = *(const V8*)(qkv + (long)t * 3 * d + (long)head * DH + sub * 8);
  const int npages = (nkeys + page - 1) / page;
  // chunk_pages > 0: every split covers that many pages whatever the request's length (splits past its end
  // are empty), so that the work items of a ragged batch are all about the same size; otherwise the
  // request's own pages are divided evenly over the splits
  const int per = chunk_pages > 0 ? chunk_pages : (npages + nsplit - 1) / nsplit;
  const int p_lo = split * per, p_hi = min(npages, p_lo + per);
  if (p_lo >= p_hi && nsplit > 1) {   // an empty split: only its marker is read by the merge
    if (threadIdx.x == 0) {
      float* pp = partial + (((long)t * h + head) * nsplit + split) * (DH + 2);
      pp[DH] = -INFINITY;
      pp[DH + 1] = 0.f;
    }
    return;
  }
  // The split's tokens in units of one load (1 KB of K, 1 KB of V); every unit has a token of the context.  Groups of G
  // units are dealt to the wavefronts; a group may span pages (two of 16 tokens of 64 elements) or be part of one.
  const int lpp = page / TPL, sh = (lpp & (lpp - 1)) == 0 ? __ffs(lpp) - 1 : -1;
  const int u_lo = p_lo * lpp, u_hi = min(p_hi * lpp, (nkeys + TPL - 1) / TPL);
  const int ng = (u_hi - u_lo + G - 1) / G;
  const int32_t* bt = block_table + (long)req * max_pages;
  auto page_of = [&](int u) { return sh >= 0 ? u >> sh : u / lpp; };
  // where a group's units lie in the pools; the block table is read a group ahead of the loads that need it
  auto find = [&](int g, long (&at)[G]) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const int u = min(u_lo + g * G + i, u_hi - 1), p = page_of(u);
      at[i] = (((long)bt[p] * h + head) * page) * DH + (u - p * lpp) * 512;
    }
  };
  auto fetch = [&](const long (&at)[G], V8 (&k)[G], V8 (&v)[G]) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      k[i] = __builtin_nontemporal_load((const V8*)(k_pool + at[i] + lane * 8));
      v[i] = __builtin_nontemporal_load((const V8*)(v_pool + at[i] + lane * 8));
    }
  };

  float q[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) q[i] = to_f(qv[i]) * scale_log2;
  float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  auto attend = [&](int g, const V8 (&kv)[G], V8 (&vv)[G]) {
    float s[G], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      float a = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) a = fmaf(q[c], to_f(kv[i][c]), a);
#pragma unroll
      for (int off = 1; off < LPT; off <<= 1) a += __shfl_xor(a, off, 64);
      const int u = u_lo + g * G + i;
      s[i] = u < u_hi && u * TPL + tok_in < nkeys ? a : -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
#pragma unroll
    for (int off = LPT; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    const float m_new = fmaxf(m, mx);
    // a group whose scores have all overflowed to -inf (bf16 operands reach that) counts for nothing beside a finite score
    const float ref = m_new == -INFINITY ? 0.f : m_new, alpha = __builtin_amdgcn_exp2f(m - ref);
    l *= alpha;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] *= alpha;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const float pr = __builtin_amdgcn_exp2f(s[i] - ref);
      l += pr;
      // slots of the last page beyond the context were never written: whatever bit patterns they hold
      // (NaN, infinity) must not reach the sum through 0 * x
      if (s[i] == -INFINITY) vv[i] = V8{};
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] = fmaf(pr, to_f(vv[i][c]), acc[c]);
    }
    m = m_new;
  };
  int g = wave;
  if (g < ng) {
    long at[G];
    V8 k0[G], v0[G], k1[G], v1[G];
    find(g, at);
    fetch(at, k0, v0);
    if (g + NW < ng) find(g + NW, at);
    for (; g < ng; g += 2 * NW) {
      if (g + NW < ng) {
        fetch(at, k1, v1);
        if (g + 2 * NW < ng) find(g + 2 * NW, at);
      }
      attend(g, k0, v0);
      if (g + NW < ng) {
        if (g + 2 * NW < ng) {
          fetch(at, k0, v0);
          if (g + 3 * NW < ng) find(g + 3 * NW, at);
        }
        attend(g + NW, k1, v1);
      }
    }
  }
  // sum over the token groups of the wavefront (lanes with equal `sub`)
#pragma unroll
  for (int off = LPT; off < 64; off <<= 1) {
    l += __shfl_xor(l, off, 64);
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] += __shfl_xor(acc[c], off, 64);
  }
  if (lane < LPT) {
#pragma unroll
    for (int c = 0; c < 8; ++c) s_o[wave][lane * 8 + c] = acc[c];
  }
  if (lane == 0) { s_m[wave] = m; s_l[wave] = l; }
  __syncthreads();
  if (threadIdx.x < DH) {
    float mm = s_m[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, s_m[w]);
    float ll = 0.f, oo = 0.f;
    if (mm != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_m[w] - mm);   // 0 for a wavefront that saw no group
        ll += s_l[w] * f;
        oo += s_o[w][threadIdx.x] * f;
      }
    }
    if (nsplit == 1) {
      o[(long)t * d + (long)head * DH + threadIdx.x] = from_f<T>(oo / ll);
    } else {
      float* pp = partial + (((long)t * h + head) * nsplit + split) * (DH + 2);
      pp[threadIdx.x] = oo;
      if (threadIdx.x == 0) { pp[DH] = mm; pp[DH + 1] = ll; }
    }
  }
}

// A wavefront's lanes hold the splits' maxima and sums (nsplit <= 32), and the partial outputs are read eight at a
// time: the launch is one load after the other otherwise (12 splits of one row: 8.4 us, now 4.6).
template <class T, int DH>
__global__ void decode_merge_kernel(const float* __restrict__ partial, int nsplit, int h, T* __restrict__ o) {
  const long item = blockIdx.x;   // t * h + head
  const float* pp = partial + item * nsplit * (DH + 2);
  const int lane = threadIdx.x & 63;
  const float ms = lane < nsplit ? pp[lane * (DH + 2) + DH] : -INFINITY;
  const float ls = lane < nsplit ? pp[lane * (DH + 2) + DH + 1] : 0.f;
  const float mm = wave_max(ms);
  // 0 for an empty split, whose output was never written and is not used either
  const float f = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - mm);
  const float ll = wave_sum(ls * f);
  float oo = 0.f;
  for (int s0 = 0; s0 < nsplit; s0 += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = pp[min(s0 + i, nsplit - 1) * (DH + 2) + threadIdx.x];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float fs = __shfl(f, s0 + i, 64);   // 0 past the last split
      const float mi = __shfl(ms, s0 + i, 64);
      if (mi != -INFINITY) oo += v[i] * fs;
    }
  }
  const long t = item / h, head = item % h;
  o[t * (long)h * DH + head * DH + threadIdx.x] = from_f<T>(oo / ll);
}

// The most splits that a launch uses: what the scratch of the entry points is sized for.
int most_splits(long items, int max_ctx, int page) {
  const int max_pages = (max_ctx + page - 1) / page;
  if (items >= 2048) {
    const int cp = 512 / page > 0 ? 512 / page : 1;
    if (max_pages <= cp + cp / 2) return 1;
    const int ns = (max_pages + cp - 1) / cp;
    return ns > 32 ? 1 : ns;
  }
  int ns = (int)((2048 + items - 1) / items);
  const int cap = max_pages / 8 > 1 ? max_pages / 8 : 1;
  if (ns > cap) ns = cap;
  if (ns > 32) ns = 32;
  return ns < 1 ? 1 : ns;
}

struct Plan { int splits, chunk_pages, waves; };

// Workgroups and wavefronts for `items` (row, head) pairs with contexts of at most max_ctx tokens.  How far the others fall
// short of the longest is not known here, so a rule has to hold for equal contexts and for one long one among short ones.
// ng: groups of loads in the longest context.  us, splits / wavefronts: equal contexts | 64 tokens to the longest | one of the
// longest and the others up to a sixteenth of it; 128 elements unless said:
//   Fewer than 1024 pairs: contexts of few groups whole (64 pairs of 512 1/16 9.0 | 7.5 | 7.9, 2/8 10.3 | 9.9 | 10.2), longer
//   ones split into about 2048 workgroups in all, which shares out the one long context as well (288 of 2048 1/16 64 | 29 |
//   24, 8/8 50 | 28 | 17; 480 of 16384 1/16 603 | 363 | 170, 5/16 602 | 324 | 84; 512 of 4096 1/16 166 | 85 | 45, 4/8 163 |
//   73 | 31), with more wavefronts for more groups (192 of 8192 in 11 or 12, 4: 125 | 47 | 35, 8: 126 | 44 | 33).
//   From 1024 pairs on whole contexts, as a split costs a launch and the partial results, with more wavefronts for longer
//   ones (1536 of 1000 x 64 elements 1/8 60.6, 1/4 63.9, 1/16 71.5; 2048 of 2048 1/16 326 | 163 | 33, 1/4 324 | 180 | 42), but
//   four where the pairs are many and the longest context short: a short one leaves the others without a group (5120 of
//   300 1/4 121 | 78 | 21, 1/8 120 | 74 | 34).
//   Beyond 6144 tokens chunks, so that one long request is not the last workgroup's for itself: of 4096, or more where the
//   scratch holds no more parts (1024 of 16384 whole 1271 | 668 | 177, chunks 1252 | 636 | 130), from 2048 pairs on of an eighth
//   (2048 of 8192 chunks of 4096 1278 | 687 | 102, of 1024 1302 | 692 | 85).
Plan plan(long items, int max_ctx, int page, int dh, bool may_split) {
  const int per_group = 2048 / dh;   // tokens
  const int ng = (max_ctx + per_group - 1) / per_group, most = may_split ? most_splits(items, max_ctx, page) : 1;
  if (items < 1024) {
    const int ns = most < ng / 8 ? most : ng / 8;   // a group for each wavefront
    if (ns > 1 && ng > (items < 384 ? 32 : 64))
      return Plan{ns, 0, ng / ns >= 128 ? 16 : ng / ns >= 32 || items * ns < 1024 ? 8 : 4};
    if (items < 512) return Plan{1, 0, ng <= 8 ? 4 : items <= 256 ? 16 : 8};
  } else if (max_ctx > 6144 && most > 1) {
    const bool many = items >= 2048;
    const int max_pages = (max_ctx + page - 1) / page, parts = many ? 8 : most, floor = (many ? 1024 : 4096) / page;
    const int even = (max_pages + parts - 1) / parts, cp = even > floor ? even : floor;
    return Plan{(max_pages + cp - 1) / cp, cp, many ? 8 : 16};
  }
  if (ng <= 8 || (items >= 2048 && ng <= 24) || (items >= 4096 && ng <= 48)) return Plan{1, 0, 4};
  return Plan{1, 0, ng <= 64 || (items > 2048 && ng <= 128) ? 8 : 16};
}

template <class T, int DH>
ls_status launch(const void* qkv, int T_, int h, const int32_t* pos, const int32_t* req, const void* kp,
                 const void* vp, const int32_t* bt, int max_pages, int page, int max_ctx, void* o,
                 float* scratch, hipStream_t st) {
  const long items = (long)T_ * h;
  const Plan p = plan(items, max_ctx, page, DH, scratch != nullptr);
  const int ns = p.splits;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
  auto go = [&](auto* kern) {
    kern<<<dim3((unsigned)items, ns), p.waves * 64, 0, st>>>((const T*)qkv, pos, req, (const T*)kp, (const T*)vp, bt,
                                                             max_pages, page, h, ns, p.chunk_pages, scale_log2, (T*)o,
                                                             scratch);
  };
  if (p.waves == 16) go(decode_attn_kernel<T, DH, 16>);
  else if (p.waves == 8) go(decode_attn_kernel<T, DH, 8>);
  else go(decode_attn_kernel<T, DH, 4>);
  LS_CHECK_LAUNCH();
  if (ns > 1) {
    decode_merge_kernel<T, DH><<<(unsigned)items, DH, 0, st>>>(scratch, ns, h, (T*)o);
    LS_CHECK_LAUNCH();
  }
  return LS_OK;
}

// Device address of `scratch` on the current GPU.  The array's name is a host-side stand-in, not a device
// address: the address comes from hipGetSymbolAddress, once per device with that device current (each GPU has
// its own copy at its own address), and only that pointer is handed to kernels.
ls_status static_scratch(float** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static float* ptrs[kMaxDevices] = {};
  int dev = -1;
  LS_CHECK_HIP(hipGetDevice(&dev));
  LS_REQUIRE(dev >= 0 && dev < kMaxDevices, "attn_paged_noalloc: device index %d outside 0..%d", dev, kMaxDevices - 1);
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[dev]) {
    float* p = nullptr;
    LS_CHECK_HIP(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
    LS_REQUIRE(p != nullptr, "attn_paged_noalloc: the scratch array has no device address");
    ptrs[dev] = p;
  }
  *out = ptrs[dev];
  return LS_OK;
}

}  // namespace

extern "C" {

size_t lsk_attn_decode_scratch_floats(int T, int h, int dh, int max_ctx, int page) {
  const int ns = most_splits((long)T * h, max_ctx, page);
  return ns > 1 ? (size_t)T * h * ns * (dh + 2) : 0;
}

ls_status lsk_attn_decode(const void* qkv, int dt, int T, int h, int dh, const int32_t* pos,
                          const int32_t* req, const void* k_pool, const void* v_pool,
                          const int32_t* block_table, int max_pages, int page, int max_ctx, void* o,
                          float* scratch, void* stream) {
  LsTimed timed(LSK_TIMED_DECODE_ATTN, stream);
  LS_REQUIRE(qkv && pos && req && k_pool && v_pool && block_table && o && T > 0 && max_ctx > 0,
             "attn_decode: bad argument");
  LS_REQUIRE(dt == LS_BF16 || dt == LS_F16, "attn_decode: 16-bit pools only");
  LS_REQUIRE(dh == 64 || dh == 128, "attn_decode: head_dim must be 64 or 128");
  LS_REQUIRE(page * dh % 512 == 0, "attn_decode: a page of one head must be a multiple of 1 KB");
  LS_REQUIRE((long)T * h <= 0x7fffffffL, "attn_decode: too many (row, head) pairs");
  hipStream_t st = (hipStream_t)stream;
  if (dt == LS_BF16)
    return dh == 64 ? launch<bf16_t, 64>(qkv, T, h, pos, req, k_pool, v_pool, block_table, max_pages, page, max_ctx, o, scratch, st)
                    : launch<bf16_t, 128>(qkv, T, h, pos, req, k_pool, v_pool, block_table, max_pages, page, max_ctx, o, scratch, st);
  return dh == 64 ? launch<f16_t, 64>(qkv, T, h, pos, req, k_pool, v_pool, block_table, max_pages, page, max_ctx, o, scratch, st)
                  : launch<f16_t, 128>(qkv, T, h, pos, req, k_pool, v_pool, block_table, max_pages, page, max_ctx, o, scratch, st);
}

// lsk_attn_paged with impl 1 for callers that cannot allocate: the split partials go to the library's static
// per-GPU scratch instead of a caller buffer.  No allocation of any kind happens in this call.
ls_status lsk_attn_paged_noalloc(const void* qkv, int dt, int T, int h, int dh, const int32_t* pos, const int32_t* req,
                                 const void* k_pool, const void* v_pool, const int32_t* block_table, int max_pages,
                                 int page, int max_ctx, void* o, void* stream) {
  LS_REQUIRE(T > 0 && h > 0 && max_ctx > 0 && page > 0, "attn_paged_noalloc: non-positive size");
  LS_REQUIRE(dh == 64 || dh == 128, "attn_paged_noalloc: head_dim must be 64 or 128");
  const size_t need = lsk_attn_decode_scratch_floats(T, h, dh, max_ctx, page);
  LS_REQUIRE(need <= kStaticScratchFloats,
             "attn_paged_noalloc: this launch needs %zu scratch floats, the static scratch holds %zu", need,
             kStaticScratchFloats);
  float* sp = nullptr;
  LS_TRY(static_scratch(&sp));
  return lsk_attn_decode(qkv, dt, T, h, dh, pos, req, k_pool, v_pool, block_table, max_pages, page, max_ctx, o, sp,
                         stream);
}

}  // extern "C"
