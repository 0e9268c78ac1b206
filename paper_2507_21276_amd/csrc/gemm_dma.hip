// Large-tile MFMA GEMM whose operand tiles go from global memory straight into
// LDS (16-byte direct-to-LDS loads, no register staging, no LDS store
// instructions).  256 x 256 x 64 tiles (4 wavefronts of 128 x 128) or 128 x 128 x 64
// tiles (4 wavefronts of 64 x 64) for problems with few tiles, or 64 x 128 ones for decode batches; 32x32x16 MFMA; two
// LDS buffers, or a ring of four for the smaller tiles where a compute unit has one workgroup (see launch()).  Used when
// the contraction length is a multiple of 64, or of any length from 64 on when both operands are k-strided (KTAIL:
// weight gradients over any number of tokens); the register-staged kernel in gemm.hip covers everything else.
//
// LDS layouts (a direct-to-LDS wave load writes 1 KB: lane i -> bytes 16 i):
//   k-major operand  (element (r,k) at r*ld + k): [256 rows][64 k], 128 B per
//     row, the eight 16-byte chunks of a row XOR-permuted with (row >> 1) & 7,
//     so that the 16-byte fragment reads of 16 consecutive rows hit 16
//     different bank groups.  Fragments: one 16-byte LDS read per 8 k.
//   k-strided operand (element (r,k) at k*ld + r): [64 k][256 rows], 512 B per
//     k, chunk index XOR-permuted with 4 * (k & 3).  Fragments are read with the
//     transposing LDS load (4 k x 16 rows per 16 lanes), two per 8 k.
// The permutations are applied by choosing which global chunk each lane fetches.
//
// With one wavefront per SIMD nothing hides a stalled wavefront, so the k loop is
// software-pipelined by hand: the next tile's loads are issued a few at a time
// between the MFMAs of the first half of a tile (a burst of 16 loads blocks the
// wavefront on the address path for about as long as the tile's MFMAs take), the
// LDS reads of the next fragments run under the current MFMAs, and the single
// workgroup barrier per tile sits before the last quarter of the MFMAs.
#include "gemm_dma_common.h"

#include <math.h>

#include <type_traits>

namespace {

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <class T> struct Mf;
template <> struct Mf<bf16_t> {
  typedef bf16x8 V8;
  typedef bf16x4 V4;
  static __device__ __forceinline__ f32x16 run(V8 a, V8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ V4 tr(const void* p) {
    return __builtin_bit_cast(V4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
  }
};
template <> struct Mf<f16_t> {
  typedef f16x8 V8;
  typedef f16x4 V4;
  static __device__ __forceinline__ f32x16 run(V8 a, V8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ V4 tr(const void* p) {
    return __builtin_bit_cast(V4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
  }
};

// One operand fragment: 8 k for 32 rows of an operand tile.
//  - k-major tiles: one ordinary 16-byte LDS load, tracked by the compiler.
//  - k-strided tiles: two transposing LDS loads.  These are issued from inline assembly: before
//    the builtin form the compiler waits for every direct-to-LDS load in flight (it cannot tell
//    that the tile being filled is another one), which serialises loads and arithmetic.  The
//    assembly form is invisible to the compiler's wait-count bookkeeping, so wait_frags() must
//    run between the reads and the first use; it redefines the registers, which pins the order.
template <class T, bool KMAJOR> struct Frag { typename Mf<T>::V8 v; };
template <class T> struct Frag<T, false> { s16x4 lo, hi; };

template <class T, bool KMAJOR, int ROWS>
__device__ __forceinline__ void read_frag(Frag<T, KMAJOR>& f, const char* lds_tile, int r0, int ks, int lane) {
  typedef typename Mf<T>::V8 V8;
  const int hf = lane >> 5;
  if constexpr (KMAJOR) {
    const int r = r0 + (lane & 31);
    const int kc = (ks * 2 + hf) ^ ((r >> 1) & 7);
    f.v = *(const V8*)(lds_tile + r * 128 + kc * 16);
  } else {
    constexpr int KROW = ROWS * 2;  // bytes per k row
    const int i16 = lane & 15, a = i16 >> 2, j4 = i16 & 3;
    const int nb = r0 + 16 * ((lane >> 4) & 1) + 4 * j4;  // first of the 4 rows this lane addresses
    const int kb = ks * 16 + 8 * hf;
    const int phys = (nb >> 3) ^ (4 * a);
    const char* p0 = lds_tile + (kb + a) * KROW + phys * 16 + ((nb >> 2) & 1) * 8;
    const uint32_t addr = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p0;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(f.lo) : "v"(addr) : "memory");
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.hi) : "v"(addr), "n"(4 * KROW) : "memory");
  }
}

template <class T, bool KMAJOR, int N>
__device__ __forceinline__ void wait_frags(Frag<T, KMAJOR> (&f)[N]) {
  static_assert(KMAJOR || N == 2 || N == 4, "fragment count");
  if constexpr (!KMAJOR) {
    if constexpr (N == 4)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(f[0].lo), "+v"(f[0].hi), "+v"(f[1].lo), "+v"(f[1].hi), "+v"(f[2].lo), "+v"(f[2].hi),
                     "+v"(f[3].lo), "+v"(f[3].hi));
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0].lo), "+v"(f[0].hi), "+v"(f[1].lo), "+v"(f[1].hi));
  }
}

template <class T, bool KMAJOR>
__device__ __forceinline__ typename Mf<T>::V8 frag_value(const Frag<T, KMAJOR>& f) {
  if constexpr (KMAJOR) {
    return f.v;
  } else {
    const s16x8 w = __builtin_shufflevector(f.lo, f.hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(typename Mf<T>::V8, w);
  }
}

// MODE 0: C (16-bit) = acc + bias;  1: C (fp32) = resid + acc + bias;  2: C (fp32) = acc;  4: C (fp32) += acc;
// The tile `bid` of the launch's order, over part `part` of `parts` of the contraction.
template <class T, int BM, int BN, bool AK, bool BK, int MODE, int ST, bool KTAIL>
__device__ __forceinline__ void gemm_dma_tile(const DmaArgs& g, char* smem, int bid, int part, int parts) {
  typedef typename Mf<T>::V8 V8;
  static_assert(!KTAIL || (!AK && !BK), "only a k-strided operand has a row per k to clear");
  constexpr int TM = BM, TN = BN;
  constexpr int WM = BM / 2, WN = BN / 2;       // wavefront tile
  constexpr int TI = WM / 32, TJ = WN / 32;     // 32x32 MFMA tiles per wavefront
  constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, BUF_BYTES = A_BYTES + B_BYTES;
  // buffer b: A tile at smem + b BUF_BYTES, B tile A_BYTES after it

  // workgroups that run at the same time share operand tiles through L2:
  // walk M fastest inside bands of 8 N tiles
  // (consecutive workgroup ids are dealt round-robin to the 8 XCDs, each with its
  // own L2: give every XCD a contiguous run of the tile order instead)
  const int total = g.tiles_m * g.tiles_n, per_xcd = total / 8;
  if (bid < per_xcd * 8) bid = (bid % 8) * per_xcd + bid / 8;
  const int band = 8;
  const int per_band = band * g.tiles_m;
  const int b0 = (bid / per_band) * band;
  const int bw = min(band, g.tiles_n - b0);
  const int rem = bid % per_band;
  const int tn = b0 + rem % bw, tm = rem / bw;
  const int m0 = tm * TM, n0 = tn * TN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN;
  // uniform tile bases (bytes) and their advance per k step
  const char* a_base = (const char*)g.A + (AK ? (long)m0 * g.lda : (long)m0) * 2;
  const char* b_base = (const char*)g.B + (BK ? (long)n0 * g.ldb : (long)n0) * 2;
  const long a_step = (AK ? (long)TK : (long)TK * g.lda) * 2;
  const long b_step = (BK ? (long)TK : (long)TK * g.ldb) * 2;
  uint32_t a_off[BM / 32], b_off[BN / 32];
  tile_offsets<AK, BM>(a_off, g.lda, m0, g.M, wave, lane);
  tile_offsets<BK, BN>(b_off, g.ldb, n0, g.N, wave, lane);

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // parts > 1: split-K, this workgroup contracts over its share of the k tiles
  const int nk_all = KTAIL ? (g.K + TK - 1) / TK : g.K / TK;
  const int kt0 = (int)((long)part * nk_all / parts);
  const int nk = (int)((long)(part + 1) * nk_all / parts) - kt0;
  a_base += kt0 * a_step;
  b_base += kt0 * b_step;
  // A contraction length that is not a multiple of TK (weight gradients: any number of tokens): the last tile
  // starts `shift` rows early, so that every load is in bounds, and the rows it shares with the tile before it
  // are cleared in LDS, by the lanes that loaded them, before the barrier that publishes the tile.
  const int shift = KTAIL ? nk_all * TK - g.K : 0;
  const int t_last = nk_all - 1 - kt0;   // index of the last tile in this workgroup's count
  auto tile_of = [&](const char* base, long step, int t) {
    return base + t * step - (KTAIL && t == t_last ? shift * (step / TK) : 0);
  };
  auto clear_shared_rows = [&](char* ta, char* tb) {
    constexpr int NA = BM / 32, NB = BN / 32, KA = 512 / BM, KB = 512 / BN;   // wave loads, k rows per wave load
#pragma unroll
    for (int j = 0; j < NA; ++j)
      if ((wave * NA + j) * KA + lane / (BM / 8) < shift)
        *(f32x4_a*)(ta + (wave * NA + j) * 1024 + lane * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if ((wave * NB + j) * KB + lane / (BN / 8) < shift)
        *(f32x4_a*)(tb + (wave * NB + j) * 1024 + lane * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
  };

  // Software pipeline of one k tile (4 sub-steps of 16 k): while the MFMAs of a sub-step run, the
  // fragments of the next one are read from LDS, and during LDKS sub-steps direct-to-LDS loads are
  // issued, at most one memory instruction between two MFMAs (a burst would stall the wavefront,
  // and with it the matrix pipe, on the address path).  The workgroup barrier sits
  // before the last sub-step: by then every wavefront holds its last fragments of the current
  // tile in registers, so the fragments read during the last sub-step come from the next tile.
  // Every MFMA and what follows it are fenced with scheduling barriers: the source order below is the issue order.
  constexpr int NM = TI * TJ;            // MFMAs per k sub-step
  constexpr int NF = TI + TJ;            // fragments per k sub-step
  constexpr int NLD = (BM + BN) / 32;    // direct-to-LDS loads per tile and wavefront
  constexpr int LDKS = 2;                // k sub-steps over which they are issued
  constexpr int LD_FIRST = 3;            // the first of them: sub-step 3 is the first after the barrier that frees a buffer
  constexpr int LPK = NLD / LDKS;        // loads per sub-step
  static_assert(NLD % LDKS == 0, "loads per sub-step");
  constexpr GapPlan<NM, NF, LPK> plan{};
  // tiles 0 .. ST - 2, and what sub-steps LD_FIRST .. 3 of the tile before the first would have issued of the next
#pragma unroll
  for (int t = 0; t < ST - 1; ++t) {
    const int tc = min(t, nk - 1);
    issue_tile<BM>(tile_of(a_base, a_step, tc), a_off, smem + t * BUF_BYTES, wave);
    issue_tile<BN>(tile_of(b_base, b_step, tc), b_off, smem + t * BUF_BYTES + A_BYTES, wave);
  }
  constexpr int NFIRST = (4 - LD_FIRST) * NLD / LDKS;
  {
    const int tc = min(ST - 1, nk - 1);
#pragma unroll
    for (int l = 0; l < NFIRST; ++l)
      issue_one<BM, BN>(l, tile_of(a_base, a_step, tc), a_off, tile_of(b_base, b_step, tc), b_off,
                        smem + (ST - 1) * BUF_BYTES, smem + (ST - 1) * BUF_BYTES + A_BYTES, wave);
  }
  wait_loads<(ST - 2) * NLD + NFIRST>();   // tile 0 has landed
  if (KTAIL && shift && t_last == 0) clear_shared_rows(smem, smem + A_BYTES);
  wait_lds_and_barrier();
  Frag<T, AK> fa[2][TI];
  Frag<T, BK> fb[2][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i) read_frag<T, AK, BM>(fa[0][i], smem, wm + i * 32, 0, lane);
#pragma unroll
  for (int j = 0; j < TJ; ++j) read_frag<T, BK, BN>(fb[0][j], smem + A_BYTES, wn + j * 32, 0, lane);

  // Sums of A over k (the bias gradient beside a weight gradient): the first column of tiles has all of A in its
  // fragments, so the wavefronts on its left add them up under the matrix instructions.  One sum per k sub-step and row
  // block keeps the chains short.
  constexpr bool SUMS = !AK && !BK && BM == 128;
  const bool sums = SUMS && g.row_sums && n0 == 0 && wn == 0;
  float rs[SUMS ? TI : 1][4];
  if constexpr (SUMS)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) rs[i][ks] = 0.f;

  int cur = 0;   // buffer of tile kt
  for (int kt = 0; kt < nk; ++kt) {
    const int nxt = cur + 1 == ST ? 0 : cur + 1, prv = cur == 0 ? ST - 1 : cur - 1;
    char* la = smem + cur * BUF_BYTES;
    char* lb = la + A_BYTES;
    char* na = smem + nxt * BUF_BYTES;   // the next tile's
    char* nb = na + A_BYTES;
    char* pa = smem + prv * BUF_BYTES;   // the one this tile's first sub-steps fill up (ST = 2: the next tile's)
    char* pb = pa + A_BYTES;
    cur = nxt;
    // tiles after the last are the last again: fetched, never multiplied
    const int t1 = min(kt + ST - 1, nk - 1), t2 = min(kt + ST, nk - 1);
    const char* ga1 = tile_of(a_base, a_step, t1);
    const char* gb1 = tile_of(b_base, b_step, t1);
    const char* ga2 = tile_of(a_base, a_step, t2);
    const char* gb2 = tile_of(b_base, b_step, t2);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int c = ks & 1;
      wait_frags<T, AK, TI>(fa[c]);
      wait_frags<T, BK, TJ>(fb[c]);
      if (ks == 3) {
        wait_loads<(ST - 2) * NLD>();    // this wavefront's share of the next tile has landed
        if (KTAIL && shift && kt + 1 == t_last) clear_shared_rows(na, nb);
        wait_lds_and_barrier();
      }
      V8 va[TI], vb[TJ];
#pragma unroll
      for (int i = 0; i < TI; ++i) va[i] = frag_value<T, AK>(fa[c][i]);
#pragma unroll
      for (int j = 0; j < TJ; ++j) vb[j] = frag_value<T, BK>(fb[c][j]);
      const char* ra = ks < 3 ? la : na;
      const char* rb = ks < 3 ? lb : nb;
      const int kn = (ks + 1) & 3;
      __builtin_amdgcn_sched_barrier(0);
      // sub-steps LD_FIRST .. 3 come after this tile's barrier: the buffer being vacated takes the tile
      // after the next; sub-steps before LD_FIRST complete the next tile in the other buffer
      const int ph = (ks - LD_FIRST) & 3;
      const bool ahead = LD_FIRST > 0 && ks >= LD_FIRST;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        // the wavefront's 32 x 32 tiles in boustrophedon order: consecutive MFMAs share an operand (0.4 %)
        const int ti = m / TJ, tj = (ti & 1) ? TJ - 1 - m % TJ : m % TJ;
        acc[ti][tj] = Mf<T>::run(vb[tj], va[ti], acc[ti][tj]);
        __builtin_amdgcn_sched_barrier(0);   // the MFMA first: what follows issues in its shadow
#pragma unroll
        for (int r = 0; r < NF; ++r) {
          if (plan.read_gap[r] != m) continue;
          if (r < TI) read_frag<T, AK, BM>(fa[c ^ 1][r], ra, wm + r * 32, kn, lane);
          else read_frag<T, BK, BN>(fb[c ^ 1][r - TI], rb, wn + (r - TI) * 32, kn, lane);
        }
        if (ph < LDKS) {
#pragma unroll
          for (int l = 0; l < LPK; ++l) {
            if (plan.load_gap[l] != m) continue;
            issue_one<BM, BN>(ph * LPK + l, ahead ? ga2 : ga1, a_off, ahead ? gb2 : gb1, b_off, ahead ? la : pa,
                              ahead ? lb : pb, wave);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (SUMS)
        if (sums)
#pragma unroll
          for (int i = 0; i < TI; ++i) {
            float t[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = to_f(va[i][e]);
            rs[i][ks] += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
          }
    }
  }
  // The last iteration read the fragments of a tile that does not exist.  Their registers must
  // stay allocated until the reads have returned: the compiler does not know that the
  // transposing reads issued from assembly are still in flight and would hand the registers to
  // the epilogue, where the late LDS data would overwrite live values.
  wait_frags<T, AK, TI>(fa[0]);
  wait_frags<T, BK, TJ>(fb[0]);
  __builtin_amdgcn_s_waitcnt(0);

  // Epilogue.  The MFMAs ran with the operands swapped, so the accumulators hold C^T tiles:
  // lane -> row m (lane & 31), register 4 q + e -> column 8 q + 4 (lane >> 5) + e.  Storing
  // from that layout touches 32 rows per instruction, 16 bytes in each, which the memory
  // pipeline takes far longer over than over the same bytes as whole cache lines.  So each
  // wavefront stages its tile in its quarter of the (now idle) LDS, row-major with the 16-byte
  // chunks of a row XOR-permuted by the row number, and writes it out as full rows; residual
  // and accumulation operands are read with the same coalesced pattern.
  typedef typename Mf<T>::V4 V4;
  constexpr int ESZ = MODE == 0 ? 2 : 4;
  constexpr int REGION = (BM + BN) * 128 * 2 / 4;   // bytes of LDS per wavefront
  constexpr int ROWB = WN * ESZ;                    // bytes of a staged row
  constexpr int CPR = ROWB / 16;                    // 16-byte chunks per row
  constexpr int NPASS = (WM * ROWB + REGION - 1) / REGION;
  constexpr int TIP = TI / NPASS;                   // 32-row MFMA tiles per pass
  constexpr int ROWS_P = TIP * 32;
  const int row_in = lane & 31, hf = lane >> 5;
  const float alpha = g.alpha ? *g.alpha : 1.f;
  __syncthreads();   // every wavefront is done with the operand tiles
  char* stg = smem + wave * REGION;
  if constexpr (SUMS)
    if (sums)
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        float v = (rs[i][0] + rs[i][1]) + (rs[i][2] + rs[i][3]);
        v = (v + __shfl_xor(v, 32, 64)) * alpha;   // the other eight k of every sixteen
        const int m = m0 + wm + i * 32 + row_in;
        if (hf == 0 && m < g.M) {
          float* out = g.row_sums + (long)part * g.M + m;
          *out = MODE == 4 ? *out + v : v;
        }
      }
  // A lane's columns are the same for all of its rows: its bias values are fetched once, outside the
  // staging loops (a fetch with a type switch inside them, once per element, made the epilogue some
  // thousands of instructions long and cost 3 - 6 us per launch even without a bias).
  float bv[TJ][4][4];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) bv[j][q][e] = 0.f;
  if ((MODE == 0 || MODE == 1) && g.bias) {
    const int nb = n0 + wn + 4 * hf;
    auto fetch = [&](auto* b) {
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int n = nb + j * 32 + 8 * q + e;
            bv[j][q][e] = (float)b[n < g.N ? n : g.N - 1];
          }
    };
    if (g.bias_dtype == LS_F32) fetch((const float*)g.bias);
    else if (g.bias_dtype == LS_BF16) fetch((const bf16_t*)g.bias);
    else fetch((const f16_t*)g.bias);
  }
#pragma unroll
  for (int pass = 0; pass < NPASS; ++pass) {
    // results added to a buffer (the residual stream, or the output itself): what the pass adds to is fetched
    // first, all of it at once, and arrives while the accumulators are staged (a load per store, each behind its
    // own branch and wait, made an accumulating launch a sixth longer)
    constexpr int NOUT = ROWS_P * CPR / 64;
    constexpr bool ADDS = MODE == 1 || MODE == 4;
    f32x4 c_old[ADDS ? NOUT : 1];
    if constexpr (ADDS) {
      const float* src = MODE == 1 ? g.resid : (const float*)g.C + part * g.split_stride;
      const long ld_src = MODE == 1 ? g.ldr : g.ldc;
#pragma unroll
      for (int it = 0; it < NOUT; ++it) {
        const int idx = it * 64 + lane;
        const int m = m0 + wm + pass * ROWS_P + idx / CPR;
        const int n = n0 + wn + (idx % CPR) * (16 / ESZ);
        c_old[it] = m < g.M && n < g.N ? *(const f32x4*)(src + (long)m * ld_src + n) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int ii = 0; ii < TIP; ++ii) {
      const int i = pass * TIP + ii;
      const int r = ii * 32 + row_in;
      char* srow = stg + r * ROWB;
      const int sw = r & (CPR - 1);
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * q + e] * alpha;
          if constexpr (MODE == 0 || MODE == 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += bv[j][q][e];
          }
          if constexpr (ESZ == 2) {
            V4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = from_f<T>(v[e]);
            *(u32x2_a*)(srow + (((j * 4 + q) ^ sw) * 16) + hf * 8) = __builtin_bit_cast(u32x2_t, o);
          } else {
            *(f32x4_a*)(srow + (((j * 8 + 2 * q + hf) ^ sw) * 16)) = v;
          }
        }
    }
    // full rows out: 64 / CPR rows per instruction, 16 bytes per lane
    constexpr int NIT = ROWS_P * CPR / 64, GRP = NIT % 8 == 0 ? 8 : NIT;
    auto put = [&](int it, int m, int n, const f32x4& v) {
      if constexpr (ESZ == 2) {
        *(f32x4_a*)((T*)g.C + (long)m * g.ldc + n) = v;
      } else if constexpr (MODE == 1) {
        *(f32x4*)((float*)g.C + (long)m * g.ldc + n) = v + c_old[it];
      } else {
        *(f32x4*)((float*)g.C + part * g.split_stride + (long)m * g.ldc + n) = MODE == 4 ? c_old[it] + v : v;
      }
    };
    if (m0 + wm + pass * ROWS_P + ROWS_P <= g.M && n0 + wn + WN <= g.N) {
      // uniform: every row and column of the pass exists, so nothing depends on the lane and a group of staged
      // pieces is read before it is stored (under the per-lane bounds check below the compiler moves each read to
      // its store and waits for it there: one LDS round trip after the other)
#pragma unroll
      for (int it0 = 0; it0 < NIT; it0 += GRP) {
        f32x4 v[GRP];
#pragma unroll
        for (int u = 0; u < GRP; ++u) {
          const int idx = (it0 + u) * 64 + lane;
          const int r = idx / CPR, c = idx % CPR;
          v[u] = *(const f32x4_a*)(stg + r * ROWB + ((c ^ (r & (CPR - 1))) * 16));
        }
#pragma unroll
        for (int u = 0; u < GRP; ++u) {
          const int idx = (it0 + u) * 64 + lane;
          put(it0 + u, m0 + wm + pass * ROWS_P + idx / CPR, n0 + wn + (idx % CPR) * (16 / ESZ), v[u]);
        }
      }
    } else {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int idx = it * 64 + lane;
        const int r = idx / CPR, c = idx % CPR;
        const int m = m0 + wm + pass * ROWS_P + r;
        const int n = n0 + wn + c * (16 / ESZ);
        if (m >= g.M || n >= g.N) continue;
        put(it, m, n, *(const f32x4_a*)(stg + r * ROWB + ((c ^ (r & (CPR - 1))) * 16)));
      }
    }
  }
}

template <class T, int BM, int BN, bool AK, bool BK, int MODE, int ST, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_dma_kernel(DmaArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_dma_tile<T, BM, BN, AK, BK, MODE, ST, KTAIL>(g, smem, blockIdx.x, blockIdx.y, gridDim.y);
}

template <class T, int BM, int BN, bool AK, bool BK, int MODE, int ST, bool KTAIL>
ls_status launch_st(DmaArgs g, hipStream_t st, int splits) {
  static bool attr_set = false;
  const int lds = ST * (BM + BN) * 128;
  if (!attr_set) {
    LS_CHECK_HIP(hipFuncSetAttribute((const void*)gemm_dma_kernel<T, BM, BN, AK, BK, MODE, ST, KTAIL>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (g.N + BN - 1) / BN;
  gemm_dma_kernel<T, BM, BN, AK, BK, MODE, ST, KTAIL><<<dim3(g.tiles_m * g.tiles_n, splits), 256, lds, st>>>(g);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

template <class T, int BM, int BN, bool AK, bool BK, int MODE, int ST>
ls_status launch_tail(const DmaArgs& g, hipStream_t st, int splits) {
  if constexpr (!AK && !BK)
    if (g.K % TK != 0) return launch_st<T, BM, BN, AK, BK, MODE, ST, true>(g, st, splits);
  return launch_st<T, BM, BN, AK, BK, MODE, ST, false>(g, st, splits);
}

template <class T, int BM, int BN, bool AK, bool BK, int MODE>
ls_status launch(const DmaArgs& g, hipStream_t st, int splits = 1) {
  // four LDS buffers where a compute unit has one workgroup at most: what hides a load's latency is then the ring alone
  // (64 x 128 tiles of a decode batch on a stage of d 768, 6 - 12 k tiles: 6.9 -> 5.6 us; 128 x 128 tiles: 0.87 -> 0.60 us
  // per k tile).  With two or three workgroups a unit the smaller footprint of two buffers is the better one.
  if constexpr (BM <= 128 && BN == 128) {
    const long wgs = (long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * splits;
    if (wgs <= 256) return launch_tail<T, BM, BN, AK, BK, MODE, 4>(g, st, splits);
  }
  return launch_tail<T, BM, BN, AK, BK, MODE, 2>(g, st, splits);
}

// the combinations a decoder block uses: forward (k-major x k-major, 16-bit or
// residual output), input gradient (k-major x k-strided, 16-bit output), weight
// gradient (k-strided x k-strided, fp32 output)
template <class T, int BM, int BN>
ls_status dispatch_layout(const DmaArgs& g, hipStream_t st) {
  if (g.rope_table) return LS_ESTATE;
  const int mode = g.c_dtype != LS_F32 ? 0 : (g.resid ? 1 : (g.accumulate ? 4 : 2));
  if (mode >= 2 && g.bias) return LS_ESTATE;
  if (mode == 1 && g.accumulate) return LS_ESTATE;
  if constexpr (BM == 128) {
    if (g.a_kmajor && g.b_kmajor && mode == 0) return launch<T, BM, BN, true, true, 0>(g, st);
    if (g.a_kmajor && g.b_kmajor && mode == 1) return launch<T, BM, BN, true, true, 1>(g, st);
    if (g.a_kmajor && g.b_kmajor && mode == 2) return launch<T, BM, BN, true, true, 2>(g, st);
    if (g.a_kmajor && g.b_kmajor && mode == 4) return launch<T, BM, BN, true, true, 4>(g, st);
    if (g.a_kmajor && !g.b_kmajor && mode == 0) return launch<T, BM, BN, true, false, 0>(g, st);
    if (g.a_kmajor && !g.b_kmajor && mode == 2) return launch<T, BM, BN, true, false, 2>(g, st);
    if (g.a_kmajor && !g.b_kmajor && mode == 4) return launch<T, BM, BN, true, false, 4>(g, st);
  }
  if (!g.a_kmajor && !g.b_kmajor && mode == 2) return launch<T, BM, BN, false, false, 2>(g, st);
  if (!g.a_kmajor && !g.b_kmajor && mode == 4) return launch<T, BM, BN, false, false, 4>(g, st);
  return LS_ESTATE;
}

// Weight gradients: 256 x 256 tiles when they still give most compute units a workgroup, else 128 x 128.  The other
// layouts come here where the 16x16x32 kernel leaves them to the 128 x 128 tiles.
template <class T>
ls_status dispatch(const DmaArgs& g, hipStream_t st) {
  const long big = (long)((g.M + 255) / 256) * ((g.N + 255) / 256);
  if (!g.a_kmajor && big >= 160) return dispatch_layout<T, 256, 256>(g, st);
  return dispatch_layout<T, 128, 128>(g, st);
}

}  // namespace

namespace {

// C = sum over the splits (in order) of the fp32 partial results, + bias + residual
template <class T>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* partial, int splits, long MN, int N,
                                                            void* C, long ldc, int c_dtype, const void* bias,
                                                            int bias_dtype, const float* resid, long ldr) {
  const long i4 = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 >= MN) return;
  f32x4 v = *(const f32x4*)(partial + i4);
  for (int s = 1; s < splits; ++s) v += *(const f32x4*)(partial + s * MN + i4);
  const long m = i4 / N;
  const int n = (int)(i4 % N);
  if (bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += load_as_f(bias, n + e, bias_dtype);
  }
  if (resid) v += *(const f32x4*)(resid + m * ldr + n);
  if (c_dtype == LS_F32) {
    *(f32x4*)((float*)C + m * ldc + n) = v;
  } else {
    typename Mf<T>::V4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = from_f<T>(v[e]);
    *(typename Mf<T>::V4*)((T*)C + m * ldc + n) = o;
  }
}

template <class T, int BM = 128>
ls_status run_splitk(DmaArgs g, int splits, float* scratch, void* C, long ldc, int c_dtype, const void* bias,
                     int bias_dtype, const float* resid, long ldr, hipStream_t st) {
  const long MN = (long)g.M * g.N;
  g.C = scratch; g.ldc = g.N; g.c_dtype = LS_F32; g.bias = nullptr; g.resid = nullptr; g.accumulate = 0;
  g.split_stride = MN;
  LS_TRY((launch<T, BM, 128, true, true, 2>(g, st, splits)));
  splitk_reduce_kernel<T><<<(unsigned)((MN / 4 + 255) / 256), 256, 0, st>>>(scratch, splits, MN, g.N, C, ldc, c_dtype,
                                                                          bias, bias_dtype, resid, ldr);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

}  // namespace

// Forward-layout GEMM (both operands k-major) for problems with too few output tiles to fill
// the chip: the contraction is split over `splits` workgroups per tile, partial results go to
// `scratch` (fp32, splits * M * N) and are summed in a fixed order (deterministic).  Returns
// LS_ESTATE when the shape does not call for it or the scratch is too small.
ls_status gemm_dma_splitk_try(int op_dtype, int M, int N, int K, const void* A, long lda, const void* B, long ldb,
                              void* C, long ldc, int c_dtype, const void* bias, int bias_dtype,
                              const float* resid, long ldr, float* scratch, size_t scratch_floats,
                              hipStream_t st) {
  if (!scratch || K % TK != 0 || M < 64 || N < 64 || N % 4 != 0) return LS_ESTATE;
  const int per16 = c_dtype == LS_F32 ? 4 : 8;
  if (ldc % per16 != 0 || (uintptr_t)C % 16 != 0 || (uintptr_t)scratch % 16 != 0) return LS_ESTATE;
  if (resid && (ldr % 4 != 0 || (uintptr_t)resid % 16 != 0)) return LS_ESTATE;
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  const int nk = K / TK;
  if (tiles >= 200 || nk < 32) return LS_ESTATE;
  int splits = (int)(512 / tiles);
  if (splits > 8) splits = 8;
  while (splits > 1 && nk / splits < 8) --splits;
  while (splits > 1 && (size_t)splits * M * N > scratch_floats) --splits;
  if (splits < 2) return LS_ESTATE;
  DmaArgs g{M, N, K, A, lda, 1, B, ldb, 1, nullptr, 0, LS_F32, nullptr, 0, nullptr, 0, 0, nullptr, 0, 0, 0, nullptr,
            nullptr, 0};
  if (op_dtype == LS_BF16)
    return run_splitk<bf16_t>(g, splits, scratch, C, ldc, c_dtype, bias, bias_dtype, resid, ldr, st);
  if (op_dtype == LS_F16)
    return run_splitk<f16_t>(g, splits, scratch, C, ldc, c_dtype, bias, bias_dtype, resid, ldr, st);
  return LS_ESTATE;
}

ls_status gemm_dma16_partials(int, int, int, int, const void*, long, const void*, long, float*, int, int, hipStream_t);

namespace {
// Parts in which 128 x 256 tiles (three LDS buffers, one workgroup a compute unit) take a product of up to 256 rows, or 0
// where the smaller tiles in `parts` parts are the better way.  A workgroup has twice the weights in flight of two that share
// a unit with two buffers each, and fewer parts are to be written and summed.  More workgroups than about 200 gain nothing
// while a part is short.  us with the sum (parts), weights from HBM, smaller tiles -> these: 128 rows, 12288 columns over
// 4096 35.6 (5) -> 32.0 (4), 22016 over 4096 59.7 (2) -> 55.8 (2); 64 rows, 12288 over 4096 32.3 (8) -> 28.6 (4); 256 rows,
// 4096 over 4096 30.0 (8) -> 28.0 (6).
// Where half of the chip has no workgroup it is the other way round (64 rows, 22016 over 4096 without the sum 41.1 (4), 47.4
// (2)), and also:
//   up to 64 rows, where half of a tile is empty, unless a fifth of the parts is saved (4096 over 11008 29.0 (16), 29.8 (13)),
//     and with more than 216 workgroups of long parts (28672 over 4096 55.1 (3), 62.2 (2); 8192 over 32768 122 (12), 136 (8); but
//     20480 over 5120 53.2 (4) -> 47.5 (3)); at 48 rows with more than 240 of any (16384 over 3072 29.2 (6), 30.6 (4));
//   up to 128 rows, where no part is saved that matters: sixteen are the most of either (96 rows, 3072 over 8192 22.6, 23.3), and
//     parts of less than eight k tiles gain nothing when there are as many (128 rows, 7680 over 2560 24.7, 23.8, but in cached
//     weights 21.3, 22.0);
//   beyond, where parts are short or the chip is full (130 rows, 8192 over 2048 22.9 (4), 26.7 (4), 10240 over 2560 27.7 (3), 32.4
//     (3), 8192 over 22016 125 (4), 141 (4); 200 rows, 6144 over 2048 22.2 (4), 23.2 (4)); but a full chip is the better one
//     with many parts and nearly all rows of the second tile (248 rows, 5120 over 13824 66.2 (6) -> 60.3 (6), 4096 over 11008 48.6
//     (8) -> 47.4 (8); 200 rows 43.5 (8), 44.9 (8); 248 rows, 8192 over 22016 148 (4), 154 (4)).
int parts_of_128x256(int M, int N, int nk, int parts) {
  const int tiles = (M + 127) / 128 * ((N + 255) / 256);
  int s = 256 / tiles < 16 ? 256 / tiles : 16;
  while (s > 4 && s * tiles > 208 && nk / s < 16) --s;
  while (s > 1 && nk / s < 6) --s;
  const int wgs = s * tiles, per = s > 0 ? nk / s : 0;
  if (wgs < (M <= 64 ? 190 : 160) || s > parts) return 0;
  bool better;
  if (M <= 64) better = 10 * s <= 8 * parts && (wgs <= 216 || (per < 32 && wgs <= (M < 56 ? 240 : 256)));
  else if (M <= 128) better = s < parts || (s < 16 && per >= 8);
  else better = wgs <= 216 ? per >= 10 : M > 224 && s >= 6;
  return better ? s : 0;
}
}  // namespace

// The first half of gemm_dma_splitk_try: the partial products stay in `scratch` as [splits][M][N] for a
// caller that sums them together with its next step.  LS_ESTATE when the shape does not call for a split.
ls_status gemm_dma_splitk_partials(int op_dtype, int M, int N, int K, const void* A, long lda, const void* B, long ldb,
                                   float* scratch, size_t scratch_floats, int* splits_out, hipStream_t st) {
  if (!scratch || K % TK != 0 || M <= 128 || N < 64 || N % 4 != 0 || (uintptr_t)scratch % 16 != 0) return LS_ESTATE;
  if (lda % 8 != 0 || ldb % 8 != 0 || (uintptr_t)A % 16 != 0 || (uintptr_t)B % 16 != 0) return LS_ESTATE;
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128), MN = (long)M * N;
  const int nk = K / TK;
  if (nk < 32) return LS_ESTATE;
  // Where 128 x 128 tiles are too many to split: 256 x 256 tiles in as many parts as fill the chip once, at 1.8 us per k
  // tile of four times the arithmetic and 8 us to write a tile of partial sums, against 0.62 us for a 128 x 128 tile
  // alone on its compute unit and 1.4 us for two sharing one.  The sum of the parts (a launch, and its traffic at about
  // 4 TB/s) takes another kernel's place (9 us).  Eight blocks of d 4096: 48 decode rows and a 200-token prompt 3652 ->
  // 3495 us (FFN-up in two parts 66 us, was 80), 890 prompt rows 4051 -> 3934 us (FFN-down in four 90 us, was 110).
  // Fewer tiles stay with the split 128 x 128 ones: at 576 and 640 rows the large tiles made the whole call 4 % longer.
  const long tiles256 = (long)((M + 255) / 256) * ((N + 255) / 256);
  const int s256 = (int)(256 / tiles256 < 8 ? 256 / tiles256 : 8);
  const float us128 = (float)nk * (tiles <= 256 ? 0.62f : 1.4f * (float)((tiles + 511) / 512)) + 9.f;
  const float us256 = (float)nk / (float)(s256 > 0 ? s256 : 1) * 1.8f + 12.f + (float)MN * 4.f * (s256 + 1) / 4e6f;
  const bool wide = tiles >= 200 && N >= 256 && s256 >= 2 && nk / s256 >= 8 && (size_t)(s256 * MN) <= scratch_floats &&
                    us256 < 0.95f * us128;
  // counted here, behind the decision: a caller that is refused runs another entry point, which counts itself
  const int kind = M >= 256 ? LSK_TIMED_GEMM : LSK_TIMED_DECODE_GEMM;
  if (wide) {
    LsTimed timed(kind, st);
    LS_TRY(gemm_dma16_partials(op_dtype, M, N, K, A, lda, B, ldb, scratch, s256, 256, st));
    *splits_out = s256;
    return LS_OK;
  }
  if (tiles >= 200) return LS_ESTATE;
  int splits = (int)(512 / tiles);
  if (splits > 8) splits = 8;
  while (splits > 1 && nk / splits < 8) --splits;
  while (splits > 1 && (size_t)splits * M * N > scratch_floats) --splits;
  if (splits < 2) return LS_ESTATE;
  LsTimed timed(kind, st);
  const int fewer = M <= 256 ? parts_of_128x256(M, N, nk, splits) : 0;
  if (fewer >= 2) {
    LS_TRY(gemm_dma16_partials(op_dtype, M, N, K, A, lda, B, ldb, scratch, fewer, 128, st));
    *splits_out = fewer;
    return LS_OK;
  }
  DmaArgs g{M, N, K, A, lda, 1, B, ldb, 1, scratch, N, LS_F32, nullptr, 0, nullptr, 0, 0, nullptr, 0, 0, 0, nullptr,
            nullptr, 0};
  g.split_stride = (long)M * N;
  if (op_dtype == LS_BF16) LS_TRY((launch<bf16_t, 128, 128, true, true, 2>(g, st, splits)));
  else if (op_dtype == LS_F16) LS_TRY((launch<f16_t, 128, 128, true, true, 2>(g, st, splits)));
  else return LS_ESTATE;
  *splits_out = splits;
  return LS_OK;
}

namespace {

// C = (C +) alpha * sum over the splits, in order
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* partial, int splits, long MN, int N, float* C,
                                                           long ldc, int accumulate, const float* alpha_dev) {
  const long i4 = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i4 >= MN) return;
  float* c = C + i4 / N * ldc + i4 % N;
  f32x4 v = *(const f32x4*)(partial + i4);
#pragma unroll 4
  for (int s = 1; s < splits; ++s) v += *(const f32x4*)(partial + s * MN + i4);
  v *= alpha_dev ? *alpha_dev : 1.f;
  *(f32x4*)c = accumulate ? *(const f32x4*)c + v : v;
}

// Parts into which a product of `tiles` 128 x 128 tiles over nk k tiles is split so that the chip is full once.  A
// workgroup alone on its compute unit takes 0.65 us per k tile (two share one at 1.4 us: nothing is gained beyond 256
// workgroups); the sum of the parts is a launch of 4 us and moves MN (parts + 1) floats at about 4 TB/s.
// Weight gradients over 4096 tokens, alone, one part -> split: 768 x 768 (6 parts) 33 -> 18 us, 2304 x 768 (2) 34 -> 28,
// 256 x 256 (8) 33 -> 11.5; 3072 x 768 (144 tiles) stays whole (39 us in a task; in three parts, two workgroups a compute
// unit, 39 us as well).  A further part has to gain 10 % over the last one taken: the estimate is no better than that.
// The forward splits above go by an older rule (512 workgroups, from 32 k tiles on) that these figures do not cover.
int splits_to_fill(long tiles, int nk, long MN) {
  int best = 1;
  float best_us = 1e30f;
  for (int s = 1; s <= 8 && s * tiles <= 256 && nk / s >= 4; ++s) {
    const float us = (float)((nk + s - 1) / s) * 0.65f + (s > 1 ? 4.f + (float)MN * 4.f * (s + 1) / 4e6f : 0.f);
    if (us < 0.9f * best_us) { best = s; best_us = us; }
  }
  return best;
}

}  // namespace

// Floats of scratch that the gradient of an M x N weight matrix may use, whatever the token count
size_t gemm_dma_wgrad_scratch_floats(long M, long N) {
  const long tiles = ((M + 127) / 128) * ((N + 127) / 128);
  if (tiles > 128) return 0;
  const long most = 256 / tiles < 8 ? 256 / tiles : 8;
  return (size_t)(most * M * N);
}

namespace {

// The two gradients of a linear map as one launch of 128 x 128 tiles: the weight gradient's workgroups (w, WMODE 2 or 4)
// and the input gradient's (d, DMODE 0 or 2), the longer ones first.  Either alone leaves part of the chip without work
// in a task of a few thousand tokens on a small stage (192 and 144 tiles on 256 compute units), and its ramp and drain
// are a third of it.
template <class T, int WMODE, int DMODE, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_grads_kernel(DmaArgs w, int wparts, DmaArgs d, int dparts, int d_first) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tw = w.tiles_m * w.tiles_n, td = d.tiles_m * d.tiles_n;
  const int id = blockIdx.x - (d_first ? td * dparts : 0);
  if (d_first ? id >= 0 : id < tw * wparts) {
    gemm_dma_tile<T, 128, 128, false, false, WMODE, 4, KTAIL>(w, smem, id % tw, id / tw, wparts);
  } else {
    const int i = d_first ? blockIdx.x : id - tw * wparts;
    gemm_dma_tile<T, 128, 128, true, false, DMODE, 4, false>(d, smem, i % td, i / td, dparts);
  }
}

// The sums over the parts of both, and of the bias gradient's, in order
struct GradSums {
  const float* wp; int wparts; long wMN; float* dW; int accumulate; const float* alpha; unsigned w_blocks;
  const float* bp; int bM; float* db; unsigned b_blocks;
  const float* dp; int dparts; long dMN; void* dIn;
};
__device__ __forceinline__ f32x4 sum_parts(const float* p, int parts, long stride) {
  f32x4 v[8], s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (i < parts) v[i] = *(const f32x4*)(p + i * stride);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (i < parts) s += v[i];
  return s;
}
template <class T>
__global__ __launch_bounds__(256) void grad_sums_kernel(GradSums g) {
  unsigned b = blockIdx.x;
  if (b < g.w_blocks) {
    const long i4 = ((long)b * 256 + threadIdx.x) * 4;
    if (i4 >= g.wMN) return;
    const f32x4 old = g.accumulate ? *(const f32x4*)(g.dW + i4) : f32x4{0.f, 0.f, 0.f, 0.f};
    const float a = g.alpha ? *g.alpha : 1.f;
    const f32x4 v = sum_parts(g.wp + i4, g.wparts, g.wMN) * a;
    *(f32x4*)(g.dW + i4) = g.accumulate ? old + v : v;
    return;
  }
  b -= g.w_blocks;
  if (b < g.b_blocks) {
    const int i4 = (b * 256 + threadIdx.x) * 4;
    if (i4 >= g.bM) return;
    const float a = g.alpha ? *g.alpha : 1.f;
    const f32x4 v = sum_parts(g.bp + i4, g.wparts, g.bM) * a;
#pragma unroll
    for (int e = 0; e < 4; ++e) g.db[i4 + e] = g.accumulate ? g.db[i4 + e] + v[e] : v[e];   // any alignment
    return;
  }
  b -= g.b_blocks;
  const long i4 = ((long)b * 256 + threadIdx.x) * 4;
  if (i4 >= g.dMN) return;
  const f32x4 v = sum_parts(g.dp + i4, g.dparts, g.dMN);
  typename Mf<T>::V4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = from_f<T>(v[e]);
  *(typename Mf<T>::V4*)((T*)g.dIn + i4) = o;
}

template <class T, int WMODE, int DMODE, bool KTAIL>
ls_status launch_grads(const DmaArgs& w, int wparts, const DmaArgs& d, int dparts, bool d_first, hipStream_t st) {
  static bool attr_set = false;
  constexpr int lds = 4 * 256 * 128;
  if (!attr_set) {
    LS_CHECK_HIP(hipFuncSetAttribute((const void*)gemm_grads_kernel<T, WMODE, DMODE, KTAIL>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    attr_set = true;
  }
  const unsigned wgs = (unsigned)(w.tiles_m * w.tiles_n * wparts + d.tiles_m * d.tiles_n * dparts);
  gemm_grads_kernel<T, WMODE, DMODE, KTAIL><<<dim3(wgs), 256, lds, st>>>(w, wparts, d, dparts, d_first);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

// Time until n1 workgroups of l1 us and then n2 of l2 <= l1 us have run on 256 compute units, one at a time on each.
float makespan(int n1, float l1, int n2, float l2) {
  const int q = n1 / 256, r = n1 % 256;
  const float busy = (float)q * l1, more = (float)(q + 1) * l1;   // of 256 - r units and of r
  float t = fmaxf(r ? more : busy, ((float)n1 * l1 + (float)n2 * l2) / 256.f);
  for (;; t += l2 * 0.125f) {
    const float a = r ? floorf((t - more) / l2) : 0.f, b = floorf((t - busy) / l2);
    if ((float)r * fmaxf(a, 0.f) + (float)(256 - r) * fmaxf(b, 0.f) >= (float)n2) return t;
  }
}

}  // namespace

float gemm_dma_whole_us(int M, int N, int K);

// Both gradients of a linear map y = x W^T (+ b) over T rows: dIn [T, N] = dOut [T, K] W [K, N] in the operand type, dW [K, N]
// (+)= alpha dOut^T In, db [K] (+)= alpha column sums of dOut (null: none).  LS_ESTATE where two launches are better or the
// shape is not covered (nothing has been launched then).
// Parts of each contraction by the same estimate as splits_to_fill, 0.6 us per k tile and 3 us a workgroup, over the
// order in which the workgroups run; a sum of parts is a launch of 4 us and its traffic.  Two launches, the column sums and
// their reductions -> here, in a task of 999 tokens on d 768: FFN-down 12.5 + 17 + 4 -> 22 us, FFN-up 18 + 17 + 4 -> 22 + 5,
// output projection 10.6 + 20 + 4 -> 19, QKV 16 + 20 + 4 -> 21 + 5; six such blocks, two micro-batches: 3404 -> 2872 us; 4 x
// 1024 tokens 3177 -> 2957.
ls_status gemm_dma_grads(int op_dtype, int T, int K, int N, const void* dOut, const void* W, const void* In, void* dIn,
                         float* dW, float* db, int accumulate, const float* alpha, float* scratch, size_t scratch_floats,
                         int* parts, hipStream_t st) {
  if (!scratch || (uintptr_t)scratch % 16 != 0 || T < TK || N < 64 || K < 64 || K % TK != 0 || N % 8 != 0) return LS_ESTATE;
  if (((uintptr_t)dOut | (uintptr_t)W | (uintptr_t)In | (uintptr_t)dIn | (uintptr_t)dW) % 16 != 0) return LS_ESTATE;
  if (op_dtype != LS_BF16 && op_dtype != LS_F16) return LS_ESTATE;
  const long MNw = (long)K * N, MNd = (long)T * N;
  const long tw = (long)((K + 127) / 128) * ((N + 127) / 128), td = (long)((T + 127) / 128) * ((N + 127) / 128);
  if (tw > 256 || td > 4096) return LS_ESTATE;
  const int nkw = (T + TK - 1) / TK, nkd = K / TK;
  int wparts = 0, dparts = 0;
  bool d_first = false;
  float best = 1e30f;
  for (int a = 1; a <= 8 && (a == 1 || nkw / a >= 4); ++a)
    for (int b = 1; b <= 4 && (b == 1 || nkd / b >= 4); ++b) {
      if ((a > 1 ? (size_t)a * (MNw + K) : 0) + (b > 1 ? (size_t)b * MNd : 0) > scratch_floats) continue;
      if (a * tw > 512 || (b > 1 && b * td > 512)) continue;
      const float lw = (float)((nkw + a - 1) / a) * 0.6f + 3.f, ld = (float)((nkd + b - 1) / b) * 0.6f + 3.f;
      float us = 2.f + (ld > lw ? makespan((int)(b * td), ld, (int)(a * tw), lw) : makespan((int)(a * tw), lw, (int)(b * td), ld));
      if (a > 1 || b > 1)
        us += 4.f + (float)((a > 1 ? MNw * (a + 1) : 0) + (b > 1 ? MNd * (b + 1) : 0)) / 1e6f;
      if (us < 0.97f * best) { best = us; wparts = a; dparts = b; d_first = ld > lw; }
    }
  // launches apart
  const int ws = splits_to_fill(tw, nkw, MNw), ds = splits_to_fill(td, nkd, MNd);
  const float w_us = (float)((nkw + ws - 1) / ws) * 0.65f + 5.f + (ws > 1 ? 4.f + (float)MNw * (ws + 1) / 1e6f : 0.f);
  const float d_us = fminf(gemm_dma_whole_us(T, N, K),
                           (float)((nkd + ds - 1) / ds) * 0.65f + 5.f + (ds > 1 ? 4.f + (float)MNd * (ds + 1) / 1e6f
                                                                               : td > 256 ? 1e30f : 0.f));
  if (best >= w_us + d_us) return LS_ESTATE;
  LsTimed timed(T >= 256 ? LSK_TIMED_GEMM : LSK_TIMED_DECODE_GEMM, st);   // a refusal launches nothing and is not recorded
  if (parts) { parts[0] = wparts; parts[1] = dparts; }

  float *wp = scratch, *bp = wp + wparts * MNw, *dp = wparts > 1 ? bp + (long)wparts * K : scratch;
  const bool ws_parts = wparts > 1, ds_parts = dparts > 1;
  DmaArgs w{K, N, T, dOut, K, 0, In, N, 0, ws_parts ? wp : dW, N, LS_F32, nullptr, 0, nullptr, 0, !ws_parts && accumulate,
            ws_parts ? nullptr : alpha, 0, 0, MNw, nullptr, nullptr, 0};
  w.row_sums = !db ? nullptr : ws_parts ? bp : db;
  w.tiles_m = (K + 127) / 128; w.tiles_n = (N + 127) / 128;
  DmaArgs d{T, N, K, dOut, K, 1, W, N, 0, ds_parts ? (void*)dp : dIn, N, ds_parts ? LS_F32 : op_dtype, nullptr, 0, nullptr, 0, 0,
            nullptr, 0, 0, MNd, nullptr, nullptr, 0};
  d.tiles_m = (T + 127) / 128; d.tiles_n = (N + 127) / 128;
  auto run = [&](auto t) -> ls_status {
    typedef decltype(t) E;
    auto tail = [&](auto wm, auto dm) {
      constexpr int WM = decltype(wm)::value, DM = decltype(dm)::value;
      return T % TK ? launch_grads<E, WM, DM, true>(w, wparts, d, dparts, d_first, st)
                    : launch_grads<E, WM, DM, false>(w, wparts, d, dparts, d_first, st);
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, 4> I4;
    const bool add = w.accumulate;
    LS_TRY(add ? (ds_parts ? tail(I4{}, I2{}) : tail(I4{}, I0{})) : (ds_parts ? tail(I2{}, I2{}) : tail(I2{}, I0{})));
    if (!ws_parts && !ds_parts) return LS_OK;
    auto blocks = [](long n) { return (unsigned)((n / 4 + 255) / 256); };
    GradSums g{wp, wparts, MNw, dW, accumulate, alpha, ws_parts ? blocks(MNw) : 0, bp, K, db,
               ws_parts && db ? blocks(K + 3) : 0, dp, dparts, MNd, dIn};
    grad_sums_kernel<E><<<g.w_blocks + g.b_blocks + (ds_parts ? blocks(MNd) : 0), 256, 0, st>>>(g);
    LS_CHECK_LAUNCH();
    return LS_OK;
  };
  return op_dtype == LS_BF16 ? run(bf16_t{}) : run(f16_t{});
}

// Weight gradient C[M, N] (fp32) = (C +) alpha A^T B over K rows of A [K][M] and B [K][N], split along K into partial
// products where the output has few tiles.  LS_ESTATE where the launch is better in one piece or not covered.
ls_status gemm_dma_wgrad_splitk(int op_dtype, int M, int N, int K, const void* A, long lda, const void* B, long ldb,
                                float* C, long ldc, int accumulate, const float* alpha, float* scratch,
                                size_t scratch_floats, int* splits_out, hipStream_t st) {
  if (!scratch || (uintptr_t)scratch % 16 != 0 || M < 64 || N < 64 || M % 8 != 0 || N % 8 != 0 || K < TK) return LS_ESTATE;
  if (lda % 8 != 0 || ldb % 8 != 0 || ldc % 4 != 0 || ((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % 16 != 0) return LS_ESTATE;
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128), MN = (long)M * N;
  const int splits = splits_to_fill(tiles, (K + TK - 1) / TK, MN);
  if (splits < 2 || (size_t)(splits * MN) > scratch_floats) return LS_ESTATE;
  DmaArgs g{M, N, K, A, lda, 0, B, ldb, 0, scratch, N, LS_F32, nullptr, 0, nullptr, 0, 0, nullptr, 0, 0, 0, nullptr,
            nullptr, 0};
  g.split_stride = MN;
  if (op_dtype == LS_BF16) LS_TRY((launch<bf16_t, 128, 128, false, false, 2>(g, st, splits)));
  else if (op_dtype == LS_F16) LS_TRY((launch<f16_t, 128, 128, false, false, 2>(g, st, splits)));
  else return LS_ESTATE;
  wgrad_reduce_kernel<<<(unsigned)((MN / 4 + 255) / 256), 256, 0, st>>>(scratch, splits, MN, N, C, ldc, accumulate, alpha);
  LS_CHECK_LAUNCH();
  *splits_out = splits;
  return LS_OK;
}

// Input gradient C[M, N] (operand type) = A W over K columns of A [M][K] and rows of W [K][N], split along K into
// partial products where the output has few tiles.  LS_ESTATE where the launch is better in one piece or not covered.
ls_status gemm_dma_dgrad_splitk(int op_dtype, int M, int N, int K, const void* A, long lda, const void* B, long ldb,
                                void* C, long ldc, float* scratch, size_t scratch_floats, int* splits_out,
                                hipStream_t st) {
  if (!scratch || (uintptr_t)scratch % 16 != 0 || M < 64 || N < 64 || N % 8 != 0 || K % TK != 0) return LS_ESTATE;
  if (lda % 8 != 0 || ldb % 8 != 0 || ldc % 8 != 0 || ((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % 16 != 0) return LS_ESTATE;
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128), MN = (long)M * N;
  const int splits = splits_to_fill(tiles, K / TK, MN);
  if (splits < 2 || (size_t)(splits * MN) > scratch_floats) return LS_ESTATE;
  DmaArgs g{M, N, K, A, lda, 1, B, ldb, 0, scratch, N, LS_F32, nullptr, 0, nullptr, 0, 0, nullptr, 0, 0, 0, nullptr,
            nullptr, 0};
  g.split_stride = MN;
  const unsigned grid = (unsigned)((MN / 4 + 255) / 256);
  if (op_dtype == LS_BF16) {
    LS_TRY((launch<bf16_t, 128, 128, true, false, 2>(g, st, splits)));
    splitk_reduce_kernel<bf16_t><<<grid, 256, 0, st>>>(scratch, splits, MN, N, C, ldc, LS_BF16, nullptr, 0, nullptr, 0);
  } else if (op_dtype == LS_F16) {
    LS_TRY((launch<f16_t, 128, 128, true, false, 2>(g, st, splits)));
    splitk_reduce_kernel<f16_t><<<grid, 256, 0, st>>>(scratch, splits, MN, N, C, ldc, LS_F16, nullptr, 0, nullptr, 0);
  } else {
    return LS_ESTATE;
  }
  LS_CHECK_LAUNCH();
  *splits_out = splits;
  return LS_OK;
}

// Weight-streaming product for a few rows (decode batches, M <= 128): tiles of 64 x 128 so that
// three workgroups share a compute unit (128 x 128 and two workgroups above 64 rows), the weights stream through LDS as whole cache lines,
// and the contraction is split until the chip has about three workgroups per compute unit.
ls_status gemm_dma_skinny_partials(int op_dtype, int M, int N, int K, const void* A, long lda, const void* B,
                                   long ldb, float* scratch, size_t scratch_floats, int* splits_out, hipStream_t st) {
  if (!scratch || K % TK != 0 || M < 1 || M > 128 || N < 64 || N % 4 != 0) return LS_ESTATE;
  if ((uintptr_t)scratch % 16 != 0) return LS_ESTATE;
  // up to 64 rows: 64 x 128 tiles, three 48 KB workgroups per compute unit; up to 128 rows: 128 x 128
  // tiles, two 64 KB workgroups
  const bool tall = M > 64;
  const long tiles = (N + 127) / 128;
  const int nk = K / TK;
  int splits = (int)((tall ? 512 : 768) / tiles);   // one round of workgroups
  if (splits < 1) splits = 1;
  if (splits > 16) splits = 16;
  while (splits > 1 && nk / splits < 6) --splits;
  while (splits > 1 && (size_t)splits * M * N > scratch_floats) --splits;
  if ((size_t)splits * M * N > scratch_floats) return LS_ESTATE;
  // (fewer rows than 48 would be a small part of such a tile: 16 rows of 12288 columns over 4096 22.7 us, 23.9)
  const int fewer = M >= 48 && N >= 256 ? parts_of_128x256(M, N, nk, splits) : 0;
  if (fewer > 0) {
    LS_TRY(gemm_dma16_partials(op_dtype, M, N, K, A, lda, B, ldb, scratch, fewer, 128, st));
    *splits_out = fewer;
    return LS_OK;
  }
  DmaArgs g{M, N, K, A, lda, 1, B, ldb, 1, scratch, N, LS_F32, nullptr, 0, nullptr, 0, 0, nullptr, 0, 0, 0, nullptr,
            nullptr, 0};
  g.split_stride = (long)M * N;
  if (op_dtype == LS_BF16) {
    if (tall) LS_TRY((launch<bf16_t, 128, 128, true, true, 2>(g, st, splits)));
    else LS_TRY((launch<bf16_t, 64, 128, true, true, 2>(g, st, splits)));
  } else if (op_dtype == LS_F16) {
    if (tall) LS_TRY((launch<f16_t, 128, 128, true, true, 2>(g, st, splits)));
    else LS_TRY((launch<f16_t, 64, 128, true, true, 2>(g, st, splits)));
  } else {
    return LS_ESTATE;
  }
  *splits_out = splits;
  return LS_OK;
}

ls_status gemm_dma_skinny_try(int op_dtype, int M, int N, int K, const void* A, long lda, const void* B, long ldb,
                              void* C, long ldc, int c_dtype, const void* bias, int bias_dtype,
                              const float* resid, long ldr, float* scratch, size_t scratch_floats,
                              hipStream_t st) {
  const int per16 = c_dtype == LS_F32 ? 4 : 8;
  if (ldc % per16 != 0 || (uintptr_t)C % 16 != 0) return LS_ESTATE;
  if (resid && (ldr % 4 != 0 || (uintptr_t)resid % 16 != 0)) return LS_ESTATE;
  int splits = 0;
  const ls_status r = gemm_dma_skinny_partials(op_dtype, M, N, K, A, lda, B, ldb, scratch, scratch_floats, &splits, st);
  if (r != LS_OK) return r;
  const long MN = (long)M * N;
  const unsigned grid = (unsigned)((MN / 4 + 255) / 256);
  if (op_dtype == LS_BF16)
    splitk_reduce_kernel<bf16_t><<<grid, 256, 0, st>>>(scratch, splits, MN, N, C, ldc, c_dtype, bias, bias_dtype, resid, ldr);
  else
    splitk_reduce_kernel<f16_t><<<grid, 256, 0, st>>>(scratch, splits, MN, N, C, ldc, c_dtype, bias, bias_dtype, resid, ldr);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

ls_status gemm_dma16_try(int, int, int, int, const void*, long, int, const void*, long, int, void*, long, int,
                         const void*, int, const float*, long, int, const float*, const int32_t*, const float*, int,
                         hipStream_t);

// Returns LS_OK after launching, or LS_ESTATE (without touching the error text)
// when the shape is outside what this kernel covers.
ls_status gemm_dma_try(int op_dtype, int M, int N, int K, const void* A, long lda, int a_kmajor,
                       const void* B, long ldb, int b_kmajor, void* C, long ldc, int c_dtype,
                       const void* bias, int bias_dtype, const float* resid, long ldr, int accumulate,
                       const float* alpha, const int32_t* rope_pos, const float* rope_table, int rope_cols,
                       hipStream_t st) {
  if (M < 64 || N < 64) return LS_ESTATE;
  if (a_kmajor || b_kmajor ? K % TK != 0 : K < TK) return LS_ESTATE;
  // the epilogue stores 16-byte pieces of rows
  const int per16 = c_dtype == LS_F32 ? 4 : 8;
  if (N % per16 != 0 || ldc % per16 != 0 || (uintptr_t)C % 16 != 0) return LS_ESTATE;
  if (resid && (ldr % 4 != 0 || (uintptr_t)resid % 16 != 0)) return LS_ESTATE;
  // problems with enough tiles of 128 to 256 rows by 256 run the 16x16x32 kernel (rows_per_tile)
  const ls_status r16 = gemm_dma16_try(op_dtype, M, N, K, A, lda, a_kmajor, B, ldb, b_kmajor, C, ldc, c_dtype, bias,
                                       bias_dtype, resid, ldr, accumulate, alpha, rope_pos, rope_table, rope_cols, st);
  if (r16 != LS_ESTATE) return r16;
  DmaArgs g{M, N, K, A, lda, a_kmajor, B, ldb, b_kmajor, C, ldc, c_dtype, bias, bias_dtype, resid, ldr,
            accumulate, alpha, 0, 0, 0, rope_pos, rope_table, rope_cols};
  if (op_dtype == LS_BF16) return dispatch<bf16_t>(g, st);
  if (op_dtype == LS_F16) return dispatch<f16_t>(g, st);
  return LS_ESTATE;
}
