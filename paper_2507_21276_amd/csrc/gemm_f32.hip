// fp32 products of a few tiles on the fp32 matrix instruction (16x16x4; its peak is that of the vector units, but an
// operand element is read once per 16 results instead of once per 2).
//
// What bounds the launches of a short fp32 task (2 x 64 tokens, width 128) is not arithmetic but how many load latencies
// stand one behind the other: with 16 - 64 workgroups on 256 compute units, every k tile of a workgroup is one.  So the
// wavefronts of a workgroup do not share out the tile but the contraction: each multiplies its own range of k into a whole
// tile, straight from global memory into the fragments (no LDS on the way in, no barrier in the loop, its first loads all
// in flight at once), and the parts are summed in LDS in the order of the wavefronts, so the result depends on the sizes
// alone.  What the epilogue adds is requested before the loop.
//
// A fragment is 16 rows x 16 k: lane -> row lane & 15, k 4 (lane >> 4) .. + 3, and the four elements go to four matrix
// instructions, so that instruction e contracts over k = e, 4 + e, 8 + e, 12 + e: any order of k will do as long as
// both operands have the same one, and a k-major operand is read 16 bytes a lane.
#include "common.h"

namespace {

struct F32Args {
  int M, N, K;
  const float* A; long lda;
  const float* B; long ldb;
  float* C; long ldc;
  const void* bias; int bias_dtype;
  const float* resid; long ldr;
  int accumulate;
  const float* alpha;
  int a_vec, b_vec;   // k-major operands: 16-byte loads
};

// BT x BT results per workgroup, NW wavefronts that share the contraction
template <int BT, int NW, bool AK, bool BK>
__global__ __launch_bounds__(NW * 64) void gemm_f32_kernel(F32Args g) {
  constexpr int NB = BT / 16, U = 2;              // blocks a side; k chunks of 16 per fetch
  constexpr int LD = BT + 4;                      // four rows further = 16 banks further
  constexpr int NO = (BT * BT + NW * 64 - 1) / (NW * 64);   // results per thread
  __shared__ float part[NW][BT * LD];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tiles_m = (g.M + BT - 1) / BT;
  const int m0 = (blockIdx.x % tiles_m) * BT, n0 = (blockIdx.x / tiles_m) * BT;
  const int r = lane & 15, kg = (lane >> 4) * 4;
  const int nch = (g.K + 15) / 16;
  const int c_lo = wave * nch / NW, c_hi = (wave + 1) * nch / NW;
  const int k_end = min(g.K, c_hi * 16);

  // what the epilogue adds
  float add[NO], old[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int at = threadIdx.x + i * NW * 64, m = m0 + at / BT, n = n0 + at % BT;
    add[i] = old[i] = 0.f;
    if (at < BT * BT && m < g.M && n < g.N) {
      if (g.bias) add[i] = load_as_f(g.bias, n, g.bias_dtype);
      if (g.resid) add[i] += g.resid[(long)m * g.ldr + n];
      if (g.accumulate) old[i] = g.C[(long)m * g.ldc + n];
    }
  }
  const float alpha = g.alpha ? *g.alpha : 1.f;

  // rows past the edge repeat the last one and are not stored; k past the end is zero in both operands
  const float *pa[NB], *pb[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const long ra = min(m0 + i * 16 + r, g.M - 1), rb = min(n0 + i * 16 + r, g.N - 1);
    pa[i] = g.A + (AK ? ra * g.lda : ra);
    pb[i] = g.B + (BK ? rb * g.ldb : rb);
  }
  auto load4 = [&](const float* p, long ld, bool kmajor, int vec, int k) {
    f32x4 v;
    if (kmajor && vec) {   // K % 4 == 0: four k are all there or all past the end
      v = *(const f32x4*)(p + min(k, g.K - 4));
      if (k >= k_end) v = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = p[kmajor ? (long)min(k + e, g.K - 1) : (long)min(k + e, g.K - 1) * ld];
        v[e] = k + e < k_end ? x : 0.f;
      }
    }
    return v;
  };
  auto fetch = [&](f32x4 (&a)[U][NB], f32x4 (&b)[U][NB], int c) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        a[u][i] = load4(pa[i], g.lda, AK, g.a_vec, (c + u) * 16 + kg);
        b[u][i] = load4(pb[i], g.ldb, BK, g.b_vec, (c + u) * 16 + kg);
      }
  };
  f32x4 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const f32x4 (&a)[U][NB], const f32x4 (&b)[U][NB]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][e], b[u][j][e], acc[i][j], 0, 0, 0);
  };
  if (c_lo < c_hi) {
    f32x4 a0[U][NB], b0[U][NB], a1[U][NB], b1[U][NB];
    fetch(a0, b0, c_lo);
    for (int c = c_lo; c < c_hi; c += 2 * U) {
      if (c + U < c_hi) fetch(a1, b1, c + U);
      multiply(a0, b0);
      if (c + U < c_hi) {
        if (c + 2 * U < c_hi) fetch(a0, b0, c + 2 * U);
        multiply(a1, b1);
      }
    }
  }
  // block (i, j): lane -> column lane & 15, register e -> row 4 (lane >> 4) + e
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave][(i * 16 + kg + e) * LD + j * 16 + r] = acc[i][j][e];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int at = threadIdx.x + i * NW * 64, m = m0 + at / BT, n = n0 + at % BT;
    if (at >= BT * BT || m >= g.M || n >= g.N) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += part[w][at / BT * LD + at % BT];
    g.C[(long)m * g.ldc + n] = old[i] + (v * alpha + add[i]);
  }
}

template <int BT, int NW>
ls_status launch(const F32Args& g, int a_kmajor, int b_kmajor, hipStream_t st) {
  const dim3 grid((unsigned)(((g.M + BT - 1) / BT) * ((g.N + BT - 1) / BT))), block(NW * 64);
  if (a_kmajor && b_kmajor) gemm_f32_kernel<BT, NW, true, true><<<grid, block, 0, st>>>(g);
  else if (a_kmajor) gemm_f32_kernel<BT, NW, true, false><<<grid, block, 0, st>>>(g);
  else if (b_kmajor) gemm_f32_kernel<BT, NW, false, true><<<grid, block, 0, st>>>(g);
  else gemm_f32_kernel<BT, NW, false, false><<<grid, block, 0, st>>>(g);
  LS_CHECK_LAUNCH();
  return LS_OK;
}

}  // namespace

// C[M, N] = (C +) alpha A B^T + bias + resid in fp32, operands as in lsk_gemm; any sizes, strides and alignment.  The
// caller has checked the pointers and sizes.
// 16 x 16 tiles while there are at most 512 of them (1024 for a short contraction), and as many wavefronts as the
// contraction has work for; 32 x 32 tiles beyond.  us a launch, 32 x 32 tiles on the vector units -> here: 128 x 128 over
// 128 8.8 -> 2.6 (8 wavefronts 3.0, 16 3.4), over 512 28.3 -> 3.8 (4: 5.3); 256 x 256 over 256 15.4 -> 3.1 (4: 3.6, 16:
// 4.0), over 2048 106 -> 10; 512 x 512 over 512 28.5 -> 7.0 (16 x 16 tiles: 9.1); 960 x 1024 over 128 14.3 -> 9.2 (8
// wavefronts 13).
ls_status gemm_f32_few_tiles(int M, int N, int K, const void* A, long lda, int a_kmajor, const void* B, long ldb,
                             int b_kmajor, void* C, long ldc, const void* bias, int bias_dtype, const float* resid, long ldr,
                             int accumulate, const float* alpha, hipStream_t st) {
  F32Args g{M, N, K, (const float*)A, lda, (const float*)B, ldb, (float*)C, ldc, bias, bias_dtype, resid, ldr, accumulate,
            alpha, K % 4 == 0 && lda % 4 == 0 && (uintptr_t)A % 16 == 0, K % 4 == 0 && ldb % 4 == 0 && (uintptr_t)B % 16 == 0};
  const long tiles = (long)((M + 15) / 16) * ((N + 15) / 16);
  if (K <= 192) {
    if (tiles <= 1024) return launch<16, 4>(g, a_kmajor, b_kmajor, st);
    return launch<32, 4>(g, a_kmajor, b_kmajor, st);
  }
  if (tiles > 512) return launch<32, 8>(g, a_kmajor, b_kmajor, st);
  if (K <= 384) return launch<16, 8>(g, a_kmajor, b_kmajor, st);
  return launch<16, 16>(g, a_kmajor, b_kmajor, st);
}
