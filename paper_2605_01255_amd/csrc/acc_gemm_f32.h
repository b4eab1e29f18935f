// float32 GEMM on a ring of LDS stages (the exact products, the sketch's product with a stored S, the factor products
// and the Gram matrices of float32 layers):  C[M, N] = A . B, optionally C = beta C + alpha (A . B), and a split of the K range.
//
//   A_KMAJOR: A[M, K], K contiguous;  else A is given transposed, At[K, M], M contiguous (X^T of the sketch).
//   B_KMAJOR: Bt[N, K], K contiguous; else B[K, N], N contiguous.
//
// v_mfma_f32_16x16x4 multiplies 64 flops a clock and SIMD, so a 64 x 64 x 32 tile takes 1024 clocks against 256 for its 16 KB
// from L2: the matrix pipe bounds every tile from there on, and what matters is that it never waits.  As in gemm_ring_kernel
// the operands go global -> LDS directly, NS stages in flight, waited for by count, one barrier per K tile.
// A K tile is 32 floats = 128 bytes of a K-contiguous row, the same chunks and swizzle as 64 bfloat16.  A lane reads one
// 16-byte chunk (four consecutive k) of its row per k-step of 16: instruction t of the step takes element t, so the four
// lane groups cover k = 4 g4 + t, in another order than memory but the same for A and B.  An operand that is contiguous
// along M or N lies in LDS as 32 rows of k and is read as four single floats at those k.
// Any M, N, K with 16-byte aligned rows: chunks past K of a K-contiguous operand (K % 4 == 0) and rows past K of the other
// kind are out of the buffer's range and read as zero.  Operands below 4 GiB.
#pragma once
#include <type_traits>

#include "acc_gemm_ring.h"

namespace acc {

struct F32GemmParams {
  const float* A;
  const float* B;
  void* C;
  int64_t M, N, K;
  int64_t lda, ldb, ldc;   // row strides in elements
  int tiles_m, tiles_n, super_m;
  int accumulate;          // 0: C = A . B;  1: C = beta C + alpha (A . B), one rounding
  float alpha, beta;
  int tile_blocks;         // work-groups of one K split
  int64_t k_per_split;     // multiple of 32; split s writes its partial product at C + s * c_split_stride
  int64_t c_split_stride;
};

template <int TM, int TN, int NS, bool A_KMAJOR, bool B_KMAJOR, typename TC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int NW = 4, WN = 2;
  constexpr int BM = 2 * TM * 16, BN = 2 * TN * 16, BK = 32;
  constexpr int A_BYTES = BM * BK * 4, B_BYTES = BN * BK * 4, STAGE = A_BYTES + B_BYTES;
  constexpr int A_LOADS = A_BYTES / 1024 / NW, B_LOADS = B_BYTES / 1024 / NW, NG = A_LOADS + B_LOADS;
  static_assert((NS - 1) * NG <= 63, "vmcnt range");

  const int split = (int)blockIdx.x / p.tile_blocks;
  int tm, tn;
  if (!ring_tile(p, (int)blockIdx.x - split * p.tile_blocks, tm, tn)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int64_t k0 = (int64_t)split * p.k_per_split;
  const int64_t kn = k0 + p.k_per_split < p.K ? p.k_per_split : p.K - k0;   // this split's K range
  const int KT = (int)((kn + BK - 1) / BK);

  // ---- global -> LDS ----
  // The same code for both operands: R rows of the output dimension in the tile, `kmajor` its memory order.
  auto rsrc_of = [&](const float* X, int64_t x0, int64_t X_total, int64_t ld, bool kmajor) {
    return kmajor ? make_rsrc(X + x0 * ld + k0, ((X_total - x0 - 1) * ld + kn) * 4)
                  : make_rsrc(X + k0 * ld + x0, ((kn - 1) * ld + (X_total - x0)) * 4);
  };
  const u32x4 a_rsrc = rsrc_of(p.A, m0, p.M, p.lda, A_KMAJOR), b_rsrc = rsrc_of(p.B, n0, p.N, p.ldb, B_KMAJOR);
  const int kchunk = (lane & 7) ^ swz(wave * 8 + (lane >> 3));  // rows 32 apart share swz
  auto src_of = [&](int t, int64_t ld, bool kmajor, int R) -> uint32_t {
    if (kmajor) return (uint32_t)(((t * NW + wave) * 8 + (lane >> 3)) * ld * 4 + (kchunk << 4));
    const int chunks = R / 4, rows = 64 / chunks;  // 16-byte chunks per k row, k rows per wave-load
    const int krow = (t * NW + wave) * rows + lane / chunks;
    // the four lane groups of a read sit four k rows apart: sent to different quarters of the 64 banks (a 32-row tile
    // only has halves to give)
    const int sw = R == 32 ? ((krow >> 2) & 1) << 2 : ((krow >> 2) & 3) << 2;
    return (uint32_t)(krow * ld * 4 + (((lane % chunks) ^ sw) << 4));
  };
  uint32_t a_src[A_LOADS], b_src[B_LOADS];
#pragma unroll
  for (int t = 0; t < A_LOADS; ++t) a_src[t] = src_of(t, p.lda, A_KMAJOR, BM);
#pragma unroll
  for (int t = 0; t < B_LOADS; ++t) b_src[t] = src_of(t, p.ldb, B_KMAJOR, BN);
  const uint32_t tail = kchunk * 4 >= kn - (int64_t)(KT - 1) * BK ? 0xFFFFFFF0u : 0u;  // chunk past K in the last K tile
  const uint32_t a_kstep = A_KMAJOR ? BK * 4 : (uint32_t)(BK * p.lda * 4);
  const uint32_t b_kstep = B_KMAJOR ? BK * 4 : (uint32_t)(BK * p.ldb * 4);
  const uint32_t smem_lds = (uint32_t)(uintptr_t)smem;
  auto issue_one = [&](int g, int kt, uint32_t stage) {
    const uint32_t oob = kt == KT - 1 ? tail : 0u;
    if (g < A_LOADS)
      buffer_to_lds_b128(a_rsrc, A_KMAJOR ? a_src[g] | oob : a_src[g], (uint32_t)kt * a_kstep, stage + (g * NW + wave) * 1024);
    else
      buffer_to_lds_b128(b_rsrc, B_KMAJOR ? b_src[g - A_LOADS] | oob : b_src[g - A_LOADS], (uint32_t)kt * b_kstep,
                         stage + A_BYTES + ((g - A_LOADS) * NW + wave) * 1024);
  };

  // ---- LDS reads: element t of operand row x of k-step s is k = 16 s + 4 g4 + t ----
  const int rswz = swz(l16);
  auto base_of = [&](int x, int R, bool kmajor) -> int {  // x: row of the tile this lane reads
    if (kmajor) return x * 128;
    const int sw = R == 32 ? (g4 & 1) << 2 : g4 << 2;
    return 4 * g4 * (R * 4) + (((x >> 2) ^ sw) << 4) + (x & 3) * 4;
  };
  int a_rd[TM], b_rd[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_rd[i] = base_of((wm * TM + i) * 16 + l16, BM, A_KMAJOR);
#pragma unroll
  for (int j = 0; j < TN; ++j) b_rd[j] = A_BYTES + base_of((wn * TN + j) * 16 + l16, BN, B_KMAJOR);
  auto read = [&](const char* st, int rd, int s, int R, bool kmajor) -> f32x4 {
    if (kmajor) return *(const f32x4*)(st + rd + (((4 * s + g4) ^ rswz) << 4));
    f32x4 v;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = *(const float*)(st + rd + (16 * s + t) * (R * 4));
    return v;
  };
  f32x4 a[2][TM], b[2][TN], acc[TM][TN];
  auto read_one = [&](const char* st, int s, int r) {
    if (r < TM) a[s][r] = read(st, a_rd[r], s, BM, A_KMAJOR);
    else b[s][r - TM] = read(st, b_rd[r - TM], s, BN, B_KMAJOR);
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s < KT) {
#pragma unroll
      for (int g = 0; g < NG; ++g) issue_one(g, s, smem_lds + s * STAGE);
    }
  }
  auto wait_tiles = [&](int later) {  // at most `later` K tiles outstanding
    if (later >= NS - 1) wait_vmcnt<(NS - 1) * NG>();
    else static_for<0, NS - 1>([&](auto n) {
      if (later == decltype(n)::value) wait_vmcnt<decltype(n)::value * NG>();
    });
  };
  wait_tiles((KT < NS ? KT : NS) - 1);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < TM + TN; ++r) read_one(smem, 0, r);

  constexpr int NM = 4 * TM * TN, NR = TM + TN;
  // One K tile in stage `sc`, the next one's in stage sn (see gemm_ring_kernel).
  auto ktile = [&](int kt, int sc, int sn, auto ahead, auto last) {
    constexpr bool AHEAD = decltype(ahead)::value, LAST = decltype(last)::value;
    const char* cur = smem + sc * STAGE;
    const char* nxt = smem + sn * STAGE;
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NM>([&](auto slot) {  // element t outermost: an accumulator comes up again after TM * TN instructions
      constexpr int q = decltype(slot)::value, t = q / (TM * TN), i = q / TN % TM, j = q % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[0][j][t], a[0][i][t], acc[i][j], 0, 0, 0);
      static_for<q * NR / NM, (q + 1) * NR / NM>([&](auto r) { read_one(cur, 1, decltype(r)::value); });
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (!LAST) {
      if constexpr (AHEAD) wait_vmcnt<(NS - 2) * NG>();
      else wait_tiles(KT - 2 - kt);
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
    }
    static_for<0, NM>([&](auto slot) {
      constexpr int q = decltype(slot)::value, t = q / (TM * TN), i = q / TN % TM, j = q % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[1][j][t], a[1][i][t], acc[i][j], 0, 0, 0);
      if constexpr (!LAST) static_for<q * NR / NM, (q + 1) * NR / NM>([&](auto r) { read_one(nxt, 0, decltype(r)::value); });
      if constexpr (AHEAD)
        static_for<q * NG / NM, (q + 1) * NG / NM>([&](auto g) { issue_one(decltype(g)::value, kt + NS, smem_lds + sc * STAGE); });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using T = std::true_type;
  using F = std::false_type;
  int kt = 0, sc = 0;
  auto step = [&]() { ++kt; sc = sc + 1 == NS ? 0 : sc + 1; };
  auto after = [&]() { return sc + 1 == NS ? 0 : sc + 1; };
  for (; kt + NS < KT; step()) ktile(kt, sc, after(), T{}, F{});
  for (; kt + 1 < KT; step()) ktile(kt, sc, after(), F{}, F{});
  ktile(kt, sc, sc, F{}, T{});

  // ---- lane holds output row l16 of each 16 x 16 block and columns 4 g4 .. + 3 ----
  TC* __restrict__ C = (TC*)p.C + (int64_t)split * p.c_split_stride;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t gm = m0 + (wm * TM + i) * 16 + l16;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t gn = n0 + (wn * TN + j) * 16 + 4 * g4;
      if (gm < p.M && gn < p.N) {  // N % 4 == 0
        TC* dst = C + gm * p.ldc + gn;
        f32x4 v = acc[i][j];
        if constexpr (sizeof(TC) == 4) {
          if (p.accumulate) v = p.alpha * v + p.beta * *(const f32x4*)dst;
          *(f32x4*)dst = v;
        } else {
          bf16x4 o;
          if (p.accumulate) {
            const bf16x4 old = *(const bf16x4*)dst;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = p.alpha * v[t] + p.beta * (float)old[t];
          }
#pragma unroll
          for (int t = 0; t < 4; ++t) o[t] = (bf16)v[t];
          *(bf16x4*)dst = o;
        }
      }
    }
  }
}

template <int TM, int TN, int NS>
constexpr int gemm_f32_lds_bytes() {
  return NS * (2 * TM * 16 + 2 * TN * 16) * 32 * 4;
}

// S [n, r] in float32, the generator of the fp32 layers (rows past n are not written).  One thread per four tokens of a
// column; r columns of a row are written side by side.
__global__ __launch_bounds__(256) void sketch_matrix_kernel(SketchParams sk, int64_t n, int64_t r, float* __restrict__ S) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // = q * r + j
  const int64_t q = idx / r;
  if (4 * q >= n) return;
  const uint32_t j = (uint32_t)(idx - q * r);
  uint32_t w[4];
  float z[4];
  sketch_words(sk.key0, sk.key1, (sk.row_offset >> 2) + (uint64_t)q, j, w);
  normals_from_words<true>(w, sk.inv_sqrt_r, sk.neg2_ln2_over_r, z);
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (4 * q + t < n) S[(4 * q + t) * r + j] = z[t];
}

}  // namespace acc
