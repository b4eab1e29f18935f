// GEMM with float32 arithmetic on a ring of LDS stages, operands float32 or bfloat16 (the exact products, the sketch's
// product with a stored S, the factor products and the Gram matrices of float32 layers; products of a bfloat16 factor that
// have to keep 32 bits):  C[M, N] = A . B, optionally C = beta C + alpha (A . B), and a split of the K range.
//
//   A_KMAJOR: A[M, K], K contiguous;  else A is given transposed, At[K, M], M contiguous (X^T of the sketch).
//   B_KMAJOR: Bt[N, K], K contiguous; else B[K, N], N contiguous.
//
// v_mfma_f32_16x16x4 multiplies 64 flops a clock and SIMD, so a 64 x 64 x 32 tile takes 1024 clocks against 256 for its 16 KB
// from L2: the matrix pipe bounds every tile from there on, and what matters is that it never waits.  As in gemm_ring_kernel
// the operands go global -> LDS directly, NS stages in flight, waited for by count, one barrier per K tile.
// A K tile is 32 elements.  A lane takes four consecutive k of its row per k-step of 16: instruction t of the step takes
// element t, so the four lane groups cover k = 4 g4 + t, in another order than memory but the same for A and B.
//   K contiguous  a row is 128 (float32) or 64 bytes; one 16- or 8-byte read
//   otherwise     LDS holds 32 rows of k; four single floats at those k, or one transposing read of bfloat16
// bfloat16 operands are widened in registers (exact).
// Any M, N, K with 16-byte aligned rows: chunks past K of a K-contiguous operand (K a multiple of the chunk) and rows past K
// of the other kind are out of the buffer's range and read as zero.  Operands below 4 GiB.
#pragma once
#include <type_traits>

#include "acc_gemm_ring.h"
#include "acc_rng.h"

namespace acc {

struct F32GemmParams {
  const void* A;
  const void* B;
  void* C;
  int64_t M, N, K;
  int64_t lda, ldb, ldc;   // row strides in elements
  int tiles_m, tiles_n, super_m;
  int accumulate;          // 0: C = A . B;  1: C = beta C + alpha (A . B), one rounding
  float alpha, beta;
  int tile_blocks;         // work-groups of one K split
  int64_t k_per_split;     // multiple of 32; split s writes its partial product at C + s * c_split_stride
  int64_t c_split_stride;
  int sum_tiles;           // K tiles of one running sum, a power of two
};

// One operand of the kernel: R rows of the output dimension (BM or BN) per tile, K_MAJOR its memory order.
template <typename T, int R, bool K_MAJOR> struct F32Tile {
  static constexpr int ES = sizeof(T), NW = 4;
  static constexpr int BYTES = R * 32 * ES, WAVE_LOADS = BYTES / 1024;
  static constexpr int LOADS = WAVE_LOADS < NW ? 1 : WAVE_LOADS / NW;   // per wave; a tile of two is moved twice
  static constexpr int ROW = K_MAJOR ? 32 * ES : R * ES;                // bytes of an LDS row
  static constexpr int CHUNKS = ROW / 16;
  // Position of chunk c of LDS row `row`: c XOR this.  What one clock of a read touches must lie on different banks (64 of
  // four bytes): 16 rows of one chunk (K contiguous); four rows of k, four apart, 64 bytes of each (float32; a 32-row tile only
  // has halves to give); eight rows of k, 32 bytes of each (bfloat16).
  __device__ static __forceinline__ int swizzle(int row) {
    if constexpr (K_MAJOR) return ES == 4 ? swz(row) : (row >> 2) & 3;
    else if constexpr (ES == 4) return R == 32 ? ((row >> 2) & 1) << 2 : ((row >> 2) & 3) << 2;
    else return (R == 32 ? (row >> 2) & 1 : R == 64 ? (row >> 1) & 3 : row & 7) << 1;
  }
  __device__ static __forceinline__ int lds_block(int t, int wave) { return (t * NW + wave) % WAVE_LOADS; }
  // byte offset of the chunk this lane moves in wave-load t
  __device__ static __forceinline__ uint32_t source(int t, int wave, int lane, int64_t ld) {
    const int row = lds_block(t, wave) * (64 / CHUNKS) + lane / CHUNKS;
    return (uint32_t)(row * ld * ES + (((lane % CHUNKS) ^ swizzle(row)) << 4));
  }
  // K contiguous: this lane's chunk lies past the last K tile's `left` elements (all its rows share their swizzle)
  __device__ static __forceinline__ bool past(int wave, int lane, int64_t left) {
    return K_MAJOR && ((lane % CHUNKS) ^ swizzle(lds_block(0, wave) * (64 / CHUNKS) + lane / CHUNKS)) * (16 / ES) >= left;
  }
  // LDS offset of tile row x0 + l16 (x0 % 16 == 0), k = 4 g4; read() adds the k-step
  __device__ static __forceinline__ int base(int x0, int l16, int g4) {
    const int x = x0 + l16;
    if constexpr (K_MAJOR) return x * ROW;
    else if constexpr (ES == 4) return 4 * g4 * ROW + (((x >> 2) ^ swizzle(4 * g4)) << 4) + (x & 3) * 4;
    else {  // transposing read: lane i of a group gives row i / 4 of its four, four columns at 4 (i % 4)
      const int row = 4 * g4 + (l16 >> 2), col = x0 + 4 * (l16 & 3);
      return row * ROW + (((col >> 3) ^ swizzle(row)) << 4) + (col & 7) * 2;
    }
  }
  __device__ static __forceinline__ f32x4 read(const char* tile, int base, int s, int l16, int g4) {
    if constexpr (K_MAJOR && ES == 4) return *(const f32x4*)(tile + base + (((4 * s + g4) ^ swz(l16)) << 4));
    else if constexpr (ES == 4) {
      f32x4 v;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = *(const float*)(tile + base + (16 * s + t) * ROW);
      return v;
    } else {
      bf16x4 h;
      if constexpr (K_MAJOR) h = *(const bf16x4*)(tile + base + (((2 * s + (g4 >> 1)) ^ swizzle(l16)) << 4) + (g4 & 1) * 8);
      else h = __builtin_bit_cast(bf16x4, lds_read_tr16_b64(tile, base + 16 * s * ROW));  // row bits the swizzle uses stay
      return f32x4{(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
    }
  }
};

// What becomes of four consecutive columns gn .. gn + 3 of output row gm.  `Old` is requested before the first transfer.
template <typename TC> struct StoreProduct {
  struct Old {};
  __device__ __forceinline__ Old load(const F32GemmParams&, int64_t, int64_t) const { return Old{}; }
  __device__ __forceinline__ void store(const F32GemmParams& p, int split, int64_t gm, int64_t gn, f32x4 v, const Old&) const {
    TC* dst = (TC*)p.C + (int64_t)split * p.c_split_stride + gm * p.ldc + gn;
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
};

// Work-group `block` of the product.
template <int TM, int TN, int NS, bool A_KMAJOR, bool B_KMAJOR, typename TA, typename TB, typename Output>
__device__ __forceinline__ void gemm_f32_block(const F32GemmParams& p, const Output& output, int block, char* smem) {
  constexpr int NW = 4, WN = 2;
  constexpr int BM = 2 * TM * 16, BN = 2 * TN * 16, BK = 32;
  using TileA = F32Tile<TA, BM, A_KMAJOR>;
  using TileB = F32Tile<TB, BN, B_KMAJOR>;
  constexpr int A_BYTES = TileA::BYTES, STAGE = A_BYTES + TileB::BYTES;
  constexpr int A_LOADS = TileA::LOADS, B_LOADS = TileB::LOADS, NG = A_LOADS + B_LOADS;
  static_assert((NS - 1) * NG <= 63, "vmcnt range");

  const int split = block / p.tile_blocks;
  int tm, tn;
  if (!ring_tile(p, block - split * p.tile_blocks, tm, tn)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int64_t k0 = (int64_t)split * p.k_per_split;
  const int64_t kn = k0 + p.k_per_split < p.K ? p.k_per_split : p.K - k0;   // this split's K range
  const int KT = (int)((kn + BK - 1) / BK);

  // ---- global -> LDS ----
  auto rsrc_of = [&](const auto* X, int64_t x0, int64_t X_total, int64_t ld, bool kmajor) {
    constexpr int64_t ES = sizeof(*X);
    return kmajor ? make_rsrc(X + x0 * ld + k0, ((X_total - x0 - 1) * ld + kn) * ES)
                  : make_rsrc(X + k0 * ld + x0, ((kn - 1) * ld + (X_total - x0)) * ES);
  };
  const u32x4 a_rsrc = rsrc_of((const TA*)p.A, m0, p.M, p.lda, A_KMAJOR), b_rsrc = rsrc_of((const TB*)p.B, n0, p.N, p.ldb, B_KMAJOR);
  uint32_t a_src[A_LOADS], b_src[B_LOADS];
#pragma unroll
  for (int t = 0; t < A_LOADS; ++t) a_src[t] = TileA::source(t, wave, lane, p.lda);
#pragma unroll
  for (int t = 0; t < B_LOADS; ++t) b_src[t] = TileB::source(t, wave, lane, p.ldb);
  const int64_t left = kn - (int64_t)(KT - 1) * BK;
  const uint32_t a_tail = TileA::past(wave, lane, left) ? 0xFFFFFFF0u : 0u, b_tail = TileB::past(wave, lane, left) ? 0xFFFFFFF0u : 0u;
  const uint32_t a_kstep = (uint32_t)((A_KMAJOR ? BK : BK * p.lda) * sizeof(TA));
  const uint32_t b_kstep = (uint32_t)((B_KMAJOR ? BK : BK * p.ldb) * sizeof(TB));
  const uint32_t smem_lds = (uint32_t)(uintptr_t)smem;
  auto issue_one = [&](int g, int kt, uint32_t stage) {
    const bool last = kt == KT - 1;
    if (g < A_LOADS)
      buffer_to_lds_b128(a_rsrc, A_KMAJOR ? a_src[g] | (last ? a_tail : 0u) : a_src[g], (uint32_t)kt * a_kstep,
                         stage + TileA::lds_block(g, wave) * 1024);
    else
      buffer_to_lds_b128(b_rsrc, B_KMAJOR ? b_src[g - A_LOADS] | (last ? b_tail : 0u) : b_src[g - A_LOADS], (uint32_t)kt * b_kstep,
                         stage + A_BYTES + TileB::lds_block(g - A_LOADS, wave) * 1024);
  };

  // ---- LDS reads: element t of an operand row of k-step s is k = 16 s + 4 g4 + t ----
  int a_rd[TM], b_rd[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_rd[i] = TileA::base((wm * TM + i) * 16, l16, g4);
#pragma unroll
  for (int j = 0; j < TN; ++j) b_rd[j] = TileB::base((wn * TN + j) * 16, l16, g4);
  f32x4 a[2][TM], b[2][TN], acc[TM][TN], total[TM][TN];
  auto read_one = [&](const char* st, int s, int r) {
    if (r < TM) a[s][r] = TileA::read(st, a_rd[r], s, l16, g4);
    else b[s][r - TM] = TileB::read(st + A_BYTES, b_rd[r - TM], s, l16, g4);
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = total[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // lane holds output row l16 of each 16 x 16 block and columns 4 g4 .. + 3 (N % 4 == 0)
  typename Output::Old old[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t gm = m0 + (wm * TM + i) * 16 + l16, gn = n0 + (wn * TN + j) * 16 + 4 * g4;
      if (gm < p.M && gn < p.N) old[i][j] = output.load(p, gm, gn);
    }
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
  // Sums of sum_tiles K tiles (256 elements as a rule), then the sum of those: the rounding of one running sum grows with
  // the root of its length (K = 4096: 1.2e-6 relative; 3e-7 so), and a sketch that keeps S in its workspace has few token
  // splits left to cut it.
  const int sum_mask = p.sum_tiles - 1;
  auto fold = [&]() {
    if ((kt & sum_mask) != sum_mask) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        total[i][j] += acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
  for (; kt + NS < KT; step()) {
    ktile(kt, sc, after(), T{}, F{});
    fold();
  }
  for (; kt + 1 < KT; step()) {
    ktile(kt, sc, after(), F{}, F{});
    fold();
  }
  ktile(kt, sc, sc, F{}, T{});

#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t gm = m0 + (wm * TM + i) * 16 + l16, gn = n0 + (wn * TN + j) * 16 + 4 * g4;
      if (gm < p.M && gn < p.N) output.store(p, split, gm, gn, total[i][j] + acc[i][j], old[i][j]);
    }
}

template <int TM, int TN, int NS, bool A_KMAJOR, bool B_KMAJOR, typename TA, typename TB, typename Output>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32GemmParams p, Output output) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  gemm_f32_block<TM, TN, NS, A_KMAJOR, B_KMAJOR, TA, TB>(p, output, (int)blockIdx.x, smem);
}

// Two products that do not depend on each other in one launch, both on 32 x 32 tiles: the sketch's (both operands with their
// rows contiguous; `sketch_blocks` work-groups) and the exact one.  A small layer's launch is its latency: at 256 x 256 x 512, rank 16,
// the sketch's 5.1 us (backward 5.4) and the product's 5.5 (7.4) follow each other no more; a forward and backward pass with the dense
// dW takes 20.4 us, 29.6 with seven launches instead of five.
// `before`: work-groups of the exact product in front of the sketch's, all or none: those with the longer contraction start first, or
// they are what the launch waits for at its end (854 x 2656 x 896 at rank 256, us of a forward pass: two launches 66.6 to 68.5, the
// sketch first 69.3, the product first 60.5; 825 x 384 x 712 at rank 128, where the sketch's is the longer: 22.2, 15.6, 16.4).  All three
// counts are multiples of eight, which keeps a product's tiles on their dies.
template <bool B_KMAJOR>
__global__ __launch_bounds__(256) void gemm_f32_pair_kernel(F32GemmParams sketch, F32GemmParams exact, int sketch_blocks, int before) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int block = (int)blockIdx.x, s = block - before;
  if (s >= 0 && s < sketch_blocks) gemm_f32_block<1, 1, 4, false, false, float, float>(sketch, StoreProduct<float>{}, s, smem);
  else gemm_f32_block<1, 1, 4, true, B_KMAJOR, float, float>(exact, StoreProduct<float>{}, s < 0 ? block : block - sketch_blocks, smem);
}

template <int TM, int TN, int NS, typename TA, typename TB>
constexpr int gemm_f32_lds_bytes() {
  return NS * (F32Tile<TA, 32 * TM, true>::BYTES + F32Tile<TB, 32 * TN, true>::BYTES);
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
