// bf16 GEMM on a ring of LDS stages, for products that do not fill whole rounds of the chip with 256 x 256 tiles (steps F1, B1, B3):
// C[M, N] = A[M, K] . B, fp32 accumulate, bf16 or fp32 output, optionally C = beta C + alpha (A . B).
//
//   A is row-major with K contiguous.  B_KMAJOR = true: Bt[N, K];  false: B[K, N], N contiguous.
//
// With one tile of 128 x 128 (or 64 x 64) per compute unit a work-group's time is the latency of its transfers: a K
// tile multiplies for 0.2 us and a transfer takes one to two.  So NS stages are kept in flight (NS - 1 of them while one
// is multiplied) and waited for by count, instead of one stage ahead with a full drain per K tile (384 x 3072 x 3072: 16.5
// against 34 us, 4096 x 1024 x 3072: 28 against 36 - 41).  What is left is the path from L2 to LDS, 32 KB per K tile and
// compute unit at about 35 of its 64 bytes a clock.  With several tiles per compute unit NS = 2 and two work-groups each.
// Four waves in a 2 x 2 arrangement, each TM x TN blocks of the 16x16x32 matrix instruction; one K tile = 64 = two
// k-steps; the operands of a k-step are read while the previous one multiplies, across the K tile's one barrier:
//   k-step 0   the operands of k-step 1 are read
//   wait       K tile kt + 1 has landed (at most the NS - 2 tiles after it are outstanding), barrier
//   k-step 1   the operands of K tile kt + 1's k-step 0 are read; K tile kt + NS goes into the stage just released
// Any K % 8 == 0: in the last K tile the 16-byte chunks past K (and the rows of an N-contiguous B past K) are sent out
// of the buffer's range and read as zero on both sides.  M, N as in gemm_bf16_tile; operands below 4 GiB.
#pragma once
#include <type_traits>

#include "acc_gemm16.h"

namespace acc {

// Swizzles of an N-contiguous B tile (see swz_n16): the 4 k rows x 2 groups that 32 lanes of a transposing read touch
// fall on 8 different 32-byte bank groups.  A 64-column row covers half the banks, rows alternate between the halves.
template <int BN> __device__ __forceinline__ int swz_ring(int krow) {
  // (so do the 384-byte rows of 192 columns, whose chunks stay inside an aligned group of eight)
  if constexpr (BN == 64 || BN == 192) return (((krow >> 1) & 1) << 1) | (((krow >> 3) & 1) << 2);
  else return swz_n16(krow);
}

// Tile number -> tile: XCD x (work-groups are dealt round-robin) owns a contiguous run of tile numbers, and consecutive
// numbers walk down super_m tile rows before they move one column on, so that a run is a compact block of the output.
template <typename P> __device__ __forceinline__ bool ring_tile(const P& p, int b, int& tm, int& tn) {
  const int total = p.tiles_m * p.tiles_n, per = (total + 7) >> 3;
  const int id = (b & 7) * per + (b >> 3);
  if ((b >> 3) >= per || id >= total) return false;
  const int group = id / (p.super_m * p.tiles_n), in = id - group * p.super_m * p.tiles_n;
  const int first = group * p.super_m;
  const int rows = p.tiles_m - first < p.super_m ? p.tiles_m - first : p.super_m;
  tm = first + in % rows;
  tn = in / rows;
  return true;
}

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// SPLIT: the K range is split over groups of tile_blocks work-groups (skinny products of the RSVD path), each storing its
// partial product at C + split * c_split_stride; kb_rows as in FastGemmParams.  A running sum is then four K tiles, 256
// elements, long and these are added up: the number of splits (512 to 1536 elements each) does not decide how exact the
// result is (error of a [16384, 3072] x [3072, 64] product: 6.3e-7 with one sum per split of 1536, 6.0e-7 so, 6.1e-7 with
// the four splits of 768 that the two-stage kernel took; the time is the same).
// SUM: C = beta C + alpha (A . B).  A form of its own: behind a branch its registers cost the plain one occupancy.
template <int TM, int TN, int NS, bool B_KMAJOR, typename TC, bool SPLIT = false, bool SUM = false>
__global__ __launch_bounds__(256) void gemm_ring_kernel(FastGemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int NW = 4, WN = 2;
  constexpr int BM = 2 * TM * 16, BN = 2 * TN * 16, BK = 64;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int A_LOADS = A_BYTES / 1024 / NW, B_LOADS = B_BYTES / 1024 / NW, NG = A_LOADS + B_LOADS;
  constexpr int BN_CHUNKS = BN / 8;
  static_assert(BN == 64 || BN == 128 || BN == 192, "N-contiguous swizzle");
  static_assert((NS - 1) * NG <= 63, "vmcnt range");

  int tm, tn;
  const int split = SPLIT ? (int)blockIdx.x / p.tile_blocks : 0;
  const bool has_tile = ring_tile(p, (int)blockIdx.x - split * (SPLIT ? p.tile_blocks : 0), tm, tn);
  if (!has_tile && p.red_count == 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t m0 = has_tile ? (int64_t)tm * BM : 0, n0 = has_tile ? (int64_t)tn * BN : 0;
  const int64_t k0 = SPLIT ? (int64_t)split * p.k_per_split : 0;
  const int64_t kn = SPLIT && k0 + p.k_per_split < p.K ? p.k_per_split : p.K - k0;   // this work-group's K range
  const int64_t kb = SPLIT && p.kb_rows && p.kb_rows < k0 + kn ? p.kb_rows - k0 : kn;  // rows of an N-contiguous B in it
  const int KT = (int)((kn + BK - 1) / BK);

  // ---- global -> LDS: wave-load t of wave w fills LDS bytes [(t * NW + w) * 1024, +1024) of the operand tile ----
  const u32x4 a_rsrc = make_rsrc(p.A + m0 * p.lda + k0, ((p.M - m0 - 1) * p.lda + kn) * 2);
  const u32x4 b_rsrc = B_KMAJOR ? make_rsrc(p.B + n0 * p.ldb + k0, ((p.N - n0 - 1) * p.ldb + kn) * 2)
                                : make_rsrc(p.B + k0 * p.ldb + n0, kb > 0 ? ((kb - 1) * p.ldb + (p.N - n0)) * 2 : 0);
  uint32_t a_src[A_LOADS], b_src[B_LOADS];
  const int kchunk = (lane & 7) ^ swz(wave * 8 + (lane >> 3));  // the same for every wave-load: rows 32 apart share swz
#pragma unroll
  for (int t = 0; t < A_LOADS; ++t) a_src[t] = (uint32_t)(((t * NW + wave) * 8 + (lane >> 3)) * p.lda * 2 + (kchunk << 4));
#pragma unroll
  for (int t = 0; t < B_LOADS; ++t) {
    if (B_KMAJOR) {
      b_src[t] = (uint32_t)(((t * NW + wave) * 8 + (lane >> 3)) * p.ldb * 2 + (kchunk << 4));
    } else {
      const int c = (t * NW + wave) * 64 + lane;  // 16-byte chunk of the tile in LDS order
      const int krow = c / BN_CHUNKS;
      b_src[t] = (uint32_t)(krow * p.ldb * 2 + (((c % BN_CHUNKS) ^ swz_ring<BN>(krow)) << 4));
    }
  }
  // last K tile: this lane's chunk lies past K (whole chunks: K % 8 == 0)
  const uint32_t tail = kchunk * 8 >= kn - (int64_t)(KT - 1) * BK ? 0xFFFFFFF0u : 0u;
  const uint32_t b_kstep = B_KMAJOR ? BK * 2 : (uint32_t)(BK * p.ldb * 2);
  const uint32_t smem_lds = (uint32_t)(uintptr_t)smem;
  auto issue_one = [&](int g, int kt, uint32_t stage) {
    const uint32_t oob = kt == KT - 1 ? tail : 0u;
    if (g < A_LOADS) buffer_to_lds_b128(a_rsrc, a_src[g] | oob, (uint32_t)kt * (BK * 2), stage + (g * NW + wave) * 1024);
    else buffer_to_lds_b128(b_rsrc, B_KMAJOR ? b_src[g - A_LOADS] | oob : b_src[g - A_LOADS], (uint32_t)kt * b_kstep,
                            stage + A_BYTES + ((g - A_LOADS) * NW + wave) * 1024);
  };

  // ---- LDS read offsets of this lane's operands (see gemm16_persist_kernel) ----
  const int rswz = swz(l16);
  const int a_row = (wm * TM * 16 + l16) * 128;
  int kc[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) kc[s] = ((4 * s + g4) ^ rswz) << 4;
  int b_rd[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    if (B_KMAJOR) {
      b_rd[j] = A_BYTES + (wn * TN * 16 + j * 16 + l16) * 128;
    } else {
      const int n_off = (wn * TN + j) * 16 + 4 * (l16 & 3);
      const int krow = 8 * g4 + (l16 >> 2);
      b_rd[j] = A_BYTES + krow * (BN * 2) + (((n_off >> 3) ^ swz_ring<BN>(krow)) << 4) + (n_off & 7) * 2;
    }
  }
  bf16x8 a[2][TM], b[2][TN];
  auto read_one = [&](const char* st, int s, int r) {  // r-th operand of k-step s: A operands first
    if (r < TM) {
      a[s][r] = lds_read_b128(st, a_row + r * 2048 + kc[s]);
    } else if (B_KMAJOR) {
      b[s][r - TM] = lds_read_b128(st, b_rd[r - TM] + kc[s]);
    } else {  // k rows + 32 s and + 4: the row bits the swizzle uses do not change
      const s16x4 lo = lds_read_tr16_b64(st, b_rd[r - TM] + 32 * s * (BN * 2));
      // + 4 rows: bit 2 of the row index, which no swizzle uses
      const s16x4 hi = lds_read_tr16_b64(st, b_rd[r - TM] + (32 * s + 4) * (BN * 2));
      b[s][r - TM] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  f32x4 acc[TM][TN], total[SPLIT ? TM : 1][SPLIT ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (SPLIT) total[i][j] = acc[i][j];
    }

  if (has_tile) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (s < KT) {
#pragma unroll
        for (int g = 0; g < NG; ++g) issue_one(g, s, smem_lds + s * STAGE);
      }
    }
  }
  if (p.red_count) {
    fold_pending(p, 256);
    if (!has_tile) return;
    wait_vmcnt0();  // from here on only the ring's transfers are counted
  }
  // K tile `first` of those requested has landed when at most `later` K tiles are outstanding behind it
  auto wait_tiles = [&](int later) {
    if (later >= NS - 1) wait_vmcnt<(NS - 1) * NG>();
    else static_for<0, NS - 1>([&](auto n) {
      if (later == decltype(n)::value) wait_vmcnt<decltype(n)::value * NG>();
    });
  };
  wait_tiles((KT < NS ? KT : NS) - 1);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < TM + TN; ++r) read_one(smem, 0, r);

  constexpr int NM = TM * TN, NR = TM + TN;
  // One K tile in stage `sc` (and the next one's in stage sn).  AHEAD: K tile kt + NS exists; LAST: no K tile follows.
  auto ktile = [&](int kt, int sc, int sn, auto ahead, auto last) {
    constexpr bool AHEAD = decltype(ahead)::value, LAST = decltype(last)::value;
    const char* cur = smem + sc * STAGE;
    const char* nxt = smem + sn * STAGE;
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NM>([&](auto slot) {
      constexpr int q = decltype(slot)::value, i = q / TN, j = q % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[0][i], acc[i][j], 0, 0, 0);
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
      constexpr int q = decltype(slot)::value, i = q / TN, j = q % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[1][j], a[1][i], acc[i][j], 0, 0, 0);
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
  auto add_up = [&]() {
    if constexpr (SPLIT) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          total[i][j] += acc[i][j];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  };
  for (; kt + NS < KT; step()) {
    ktile(kt, sc, after(), T{}, F{});
    if (kt % 4 == 3) add_up();
  }
  for (; kt + 1 < KT; step()) {
    ktile(kt, sc, after(), F{}, F{});
    if (kt % 4 == 3) add_up();
  }
  ktile(kt, sc, sc, F{}, T{});
  if constexpr (SPLIT) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += total[i][j];
  }

  // ---- epilogue: lane holds output row l16 of each 16 x 16 block and columns 4 g4 .. + 3; a wave stages one block
  //      row (16 x TN * 16) in a private padded LDS region and moves 16 bytes per lane (whole rows); a product that is added
  //      to C is staged as float, so that only the sum is rounded ----
  constexpr int ES = sizeof(TC), CH16 = TN * 16 * ES / 16;
  static_assert((16 * CH16) % 64 == 0, "epilogue staging");
  __syncthreads();  // every wave is done with the ring; nothing is in flight (the last wait was for all)
  TC* __restrict__ C = (TC*)p.C + (SPLIT ? (int64_t)split * p.c_split_stride : 0);
  constexpr int SE = SUM ? 4 : ES, PITCH = TN * 16 * SE + 16;   // SE: bytes of a staged element
  static_assert(NW * 16 * PITCH <= NS * STAGE, "epilogue staging");
  char* stage_w = smem + wave * (16 * PITCH);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      char* dst = stage_w + l16 * PITCH + (j * 16 + g4 * 4) * SE;
      if constexpr (SE == 2) {
        bf16x4 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = (bf16)acc[i][j][t];
        *(bf16x4*)dst = v;
      } else {
        *(f32x4*)dst = acc[i][j];
      }
    }
#pragma unroll
    for (int t = 0; t < 16 * CH16 / 64; ++t) {
      const int idx = t * 64 + lane, row = idx / CH16, ch = idx % CH16;
      const char* staged = stage_w + row * PITCH + ch * (16 / ES) * SE;
      const int64_t gm = m0 + (wm * TM + i) * 16 + row;
      const int64_t gn = n0 + wn * TN * 16 + ch * (16 / ES);
      if (gm < p.M && gn < p.N) {
        u32x4* dst = (u32x4*)(C + gm * p.ldc + gn);
        if constexpr (SUM) *dst = scaled_sum<TC>((const float*)staged, *dst, p.alpha, p.beta);
        else *dst = *(const u32x4*)staged;
      }
    }
  }
}

template <int TM, int TN, int NS>
constexpr int gemm_ring_lds_bytes() {
  return NS * (2 * TM * 16 + 2 * TN * 16) * 64 * 2;
}

// Fill the tiling fields of p for the ring kernel's BM x BN tile; returns the 1-D grid size.
template <typename P> static inline unsigned gemm_ring_plan(P& p, int BM, int BN) {
  p.tiles_m = (int)ceil_div(p.M, BM);
  p.tiles_n = (int)ceil_div(p.N, BN);
  const int64_t total = (int64_t)p.tiles_m * p.tiles_n, per = ceil_div(total, 8);
  int sm = 1;  // a run of `per` tiles as a block about as tall as wide
  while ((int64_t)(sm + 1) * (sm + 1) <= per && sm < p.tiles_m) ++sm;
  p.super_m = sm;
  return (unsigned)(per * 8);
}

}  // namespace acc
