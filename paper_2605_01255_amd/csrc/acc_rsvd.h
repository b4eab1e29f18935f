// Small dense kernels of the RSVD compressor (Experimental Setup: randomized SVD of Halko et al.): the
// triangular factor R of a k x k Gram matrix and Yr.R^-1 by substitution, the middle steps of a Cholesky QR,
// with the Gram products and the helpers around them.  The large products (X.Omega, X^T.U, U^T.dY) run on the
// GEMM kernels.
#pragma once
#include "acc_common.h"
#include "acc_gemm.h"
#include "acc_rng.h"

namespace acc {

constexpr int kQrMaxRank = 256;            // a k x k factorisation up to this size is one launch of one work-group
constexpr int kRsvdMaxRankBlocked = 512;   // larger ranks: the same kernels on 256 x 256 diagonal blocks (blocked Cholesky)
constexpr int kCholMaxThreads = 1024;

// Storage of a k x k triangle for the two kernels below: 16 x 16 blocks (i, l), i >= l, of 1 KB, row by row; block (i, l)
// at index i (i + 1) / 2 + l.  A lane that owns row l16 and columns 4 g4 .. 4 g4 + 3 of a block (the accumulator layout of
// the 16x16x4 instruction with its operands swapped, and the layout of its operands when instruction t of four takes
// element t) reads 16 bytes at 64 l16 + 16 g4: a wave reads a whole block contiguously.
__host__ __device__ constexpr int tri_block(int i, int l) { return i * (i + 1) / 2 + l; }

struct TriIndex { int i, l; };
// block b -> (i, l), wave-uniform; b < 2^15
__device__ __forceinline__ TriIndex tri_index(int b) {
  int i = __builtin_amdgcn_readfirstlane((int)((__builtin_amdgcn_sqrtf(8.f * (float)b + 1.f) - 1.f) * 0.5f));
  i += tri_block(i + 1, 0) <= b ? 1 : 0;   // the root may be off by a rounding either way
  i -= tri_block(i, 0) > b ? 1 : 0;
  return TriIndex{i, b - tri_block(i, 0)};
}

// v of lane J of each aligned group of 16 lanes, to all of them (DPP row_newbcast).
template <int J> __device__ __forceinline__ float bcast16(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + J, 0xF, 0xF, true));
}

__device__ __forceinline__ float lane_bcast(float v, int src_lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src_lane));
}

// v[k] of lane (l16, group G) to lane (l16, group k), for the four groups of 16 lanes: what four registers of one group hold,
// in the layout of an operand of the 16x16x4 instruction.  Three lane swaps, no LDS.
template <int G> __device__ __forceinline__ float group_to_operand(f32x4 v) {
  uint32_t u[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) u[t] = __float_as_uint(v[t]);
  const auto a = __builtin_amdgcn_permlane16_swap(u[0], u[1], false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(u[2], u[3], false, false);
  const auto c = __builtin_amdgcn_permlane32_swap(a[G & 1], b[G & 1], false, false);
  return __builtin_bit_cast(float, (uint32_t)c[G >> 1]);
}

// The triangle of G [k, k] (symmetric positive semi-definite, fp32, row stride ldg, k <= 256) into LDS (tri_block storage) by
// a whole work-group, global -> LDS directly; rows and columns past k as the identity.  Ends on a barrier.
__device__ __forceinline__ void chol_load(const float* G, int64_t ldg, int k, char* smem) {
  const int tid = threadIdx.x, lane = tid & 63, waves = (int)(blockDim.x >> 6);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = (k + 15) / 16, blocks = tri_block(nb, 0);
  const u32x4 rsrc = make_rsrc(G, ((k - 1) * ldg + k) * 4);
  const uint32_t smem_lds = (uint32_t)(uintptr_t)smem;
  for (int b = wave; b < blocks; b += waves) {
    const TriIndex x = tri_index(b);
    const int row = x.i * 16 + (lane >> 2), col = x.l * 16 + (lane & 3) * 4;   // LDS order of a block: 16 bytes a lane
    const uint32_t off = row < k && col < k ? (uint32_t)((row * ldg + col) * 4) : 0xFFFFFFF0u;   // k % 4 == 0; past k reads zero
    buffer_to_lds_b128(rsrc, off, 0, smem_lds + b * 1024);
  }
  wait_vmcnt0();
  __syncthreads();
  if ((k & 15) && tid < 16 && (nb - 1) * 16 + tid >= k) ((float*)smem)[tri_block(nb - 1, nb - 1) * 256 + tid * 17] = 1.f;
  if (k & 15) __syncthreads();
}

// The upper triangular factor R of G = R^T R (positive diagonal of R), G in LDS as chol_load leaves it, by one work-group of at
// least two waves, in the square-root-free form A = L D L^T, V = L D (one reciprocal per column on the chain), R = D^-1/2 V^T.
// Left in place, in the form that a solve multiplies with (tri_block storage):
//   off-diagonal block (J, I): V_JI;  diagonal block: (L_JJ)^-1, both [n][t];  behind the blocks D^-1/2, nb * 16 values
//
// The k columns of an elimination are a serial chain; what a column costs is everything.  Wave 0 runs the chain alone: the
// diagonal block in the accumulator layout (lane (l16, g4): row l16, columns 4 g4 .. + 3), so that lane group g holds four whole
// columns.  A micro-panel of four columns is eliminated inside that group, pivot rows by DPP broadcast, and its rank-4 update of
// the block is ONE 16x16x4 instruction, whose operand three lane swaps form.  The rows of the identity go through the same
// elimination beside the block's and come out as L^-T: every row block below takes its part of the panel as a product with it
// (four instructions).  Wave 0 then takes the next block row itself and with it the next diagonal block; the other waves do
// the remaining block rows and the trailing blocks meanwhile:
//   barrier   L^-1 of panel p and its reciprocals are in LDS, trailing blocks of panel p - 1 are done
//   wave 0    V_(p+1,p), next diagonal block              others   V_(i,p), i > p + 1
//   barrier   panel p is whole
//   wave 0    elimination of the next diagonal block      others   A_il -= (V_i D^-1) V_l^T, 16x16x4 instruction
// A launch of it alone at k = 32 / 64 / 128 / 256: 4.2 / 6.7 / 13.4 / 43 us (one row per lane and a 16-column panel in registers,
// DPP broadcasts but two barriers and a whole work-group per panel: 8 / 12 / 23 / 62); a panel's chain is 2350 clocks of it, up to
// k = 128 the trailing blocks hide behind it.  Tried: the other waves carrying an identity along, so that the solve becomes a
// plain product with R^-1 (solve 12 000 -> 2 900 clocks at k = 128, factor 27 000 -> 34 000: no gain, and 256 columns 20 % slower).
// A pivot at or below rel_tol times the largest diagonal entry (of G, or *scale_ref: of the matrix G is a block of) counts
// as zero: column j of the factored matrix depends on the earlier ones.  Its row and column of R^-1 are zero, so the
// corresponding basis vector comes out as zero and the span of the others is unchanged.
__device__ __forceinline__ void chol_factor_lds(char* smem, int k, const float* scale_ref, float rel_tol) {
  const int NW = (int)(blockDim.x >> 6);
  float* const A = (float*)smem;                                     // tri_block storage
  const int nb = (k + 15) / 16;
  float* const scale = A + tri_block(nb, 0) * 256;                   // the pivot per column, 0 for a dropped one; then D^-1/2
  float* const inv = scale + nb * 16;                                // 1 / pivot, likewise
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  auto at = [&](int i, int l) -> f32x4* { return (f32x4*)(A + tri_block(i, l) * 256 + l16 * 16 + g4 * 4); };
  auto mfma4 = [](f32x4 a, f32x4 b, f32x4 c) -> f32x4 {
#pragma unroll
    for (int t = 0; t < 4; ++t) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[t], c, 0, 0, 0);
    return c;
  };
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

  if (wave == 0) {
    float maxdiag = 0.f;
    for (int c = lane; c < k; c += 64) {
      const float d = A[tri_block(c >> 4, c >> 4) * 256 + (c & 15) * 17];
      maxdiag = d > maxdiag ? d : maxdiag;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      const float d = __shfl_xor(maxdiag, m);
      maxdiag = d > maxdiag ? d : maxdiag;
    }
    const float tol = (scale_ref ? *scale_ref : maxdiag) * rel_tol;
    f32x4 c = *at(0, 0);
    for (int p = 0;; ++p) {
      f32x4 ci, lt = zero, inverses = zero, pivots = zero;   // ci: rows of the identity
#pragma unroll
      for (int t = 0; t < 4; ++t) ci[t] = l16 == 4 * g4 + t ? 1.f : 0.f;
      static_for<0, 4>([&](auto micro) {
        constexpr int g = decltype(micro)::value;
        f32x4 v = c, vi = ci, s, si, iv, pv;   // columns 4 g .. 4 g + 3 of both, in lane group g (the others' are not used)
        static_for<0, 4>([&](auto step) {
          constexpr int j = decltype(step)::value;
          const float piv = bcast16<4 * g + j>(v[j]);
          const bool dead = !(piv > tol);
          // reciprocal: hardware estimate + one Newton step (about 1 ulp); the factor's own scaling uses square roots
          float inv_p = __builtin_amdgcn_rcpf(piv);
          inv_p = fmaf(fmaf(-piv, inv_p, 1.f), inv_p, inv_p);
          iv[j] = dead ? 0.f : inv_p;
          pv[j] = dead ? 0.f : piv;
          s[j] = -(v[j] * iv[j]);
          si[j] = -(vi[j] * iv[j]);
#pragma unroll
          for (int e = j + 1; e < 4; ++e) {
            const float u = bcast16<4 * g + j>(v[e]);
            vi[e] = fmaf(u, si[j], vi[e]);
            v[e] = fmaf(u, s[j], v[e]);
          }
        });
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          lt[t] = g4 == g ? vi[t] : lt[t];
          inverses[t] = g4 == g ? iv[t] : inverses[t];
          pivots[t] = g4 == g ? pv[t] : pivots[t];
        }
        if constexpr (g < 3) {
          const float a = group_to_operand<g>(v);
          c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, group_to_operand<g>(s), c, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f32_16x16x4f32(a, group_to_operand<g>(si), ci, 0, 0, 0);
        }
      });
      float* const block = A + tri_block(p, p) * 256;    // [n][t] of L^-1; this lane has row t = l16 of L^-T
#pragma unroll
      for (int t = 0; t < 4; ++t) block[(g4 * 4 + t) * 16 + l16] = lt[t];
      if (l16 == 0) {
        *(f32x4*)(inv + p * 16 + g4 * 4) = inverses;
        *(f32x4*)(scale + p * 16 + g4 * 4) = pivots;
      }
      __syncthreads();
      if (p + 1 == nb) break;
      const f32x4 v = mfma4(*at(p, p), *at(p + 1, p), zero), d = *(const f32x4*)(inv + p * 16 + g4 * 4);
      *at(p + 1, p) = v;
      c = *at(p + 1, p + 1);
      __syncthreads();
      c = mfma4(v, -(v * d), c);
    }
  } else {
    for (int p = 0;; ++p) {
      __syncthreads();
      if (p + 1 == nb) break;
      const f32x4 linv = *at(p, p), d = *(const f32x4*)(inv + p * 16 + g4 * 4);
      for (int i = p + 1 + wave; i < nb; i += NW - 1) *at(i, p) = mfma4(linv, *at(i, p), zero);
      __syncthreads();
      // trailing blocks (i, l), p < l <= i, but for (p + 1, p + 1), four at a time
      const int count = (nb - p - 1) * (nb - p) / 2;
      for (int b0 = wave; b0 < count; b0 += 4 * (NW - 1)) {
        f32x4 c[4], vi[4], vl[4];
        f32x4* dst[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int b = b0 + u * (NW - 1);
          if (b < count) {
            const TriIndex x = tri_index(b);
            const int i = x.i + p + 1, l = x.l + p + 1;
            vi[u] = *at(i, p); vl[u] = *at(l, p); dst[u] = at(i, l);
            c[u] = *dst[u];
          }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (b0 + u * (NW - 1) < count)
              c[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(vl[u][t], -(vi[u][t] * d[t]), c[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (b0 + u * (NW - 1) < count) *dst[u] = c[u];
      }
    }
  }
  if (tid < nb * 16) {   // every wave is past the last panel's barrier
    const float piv = scale[tid];
    scale[tid] = piv > 0.f ? 1.f / sqrtf(piv) : 0.f;
  }
  __syncthreads();
}

// Work-group of a factorisation of up to 16 KB columns.
constexpr int chol_threads(int KB) { return KB > 8 ? kCholMaxThreads : 512; }

constexpr int chol_lds_bytes(int k) { return tri_block((k + 15) / 16, 0) * 1024 + (k + 15) / 16 * 16 * 2 * 4; }

// Bytes of the factor that a solve needs, in LDS or as an image in global memory: the blocks and D^-1/2.
constexpr int chol_image_bytes(int k) { return tri_block((k + 15) / 16, 0) * 1024 + (k + 15) / 16 * 64; }

// The factor (chol_factor_lds) of G [k, k] to global memory, one work-group: ranks above 128, and the diagonal blocks of the
// blocked form above rank 256.
template <int KB>
__global__ __launch_bounds__(chol_threads(KB)) void chol_factor_kernel(const float* __restrict__ G, float* __restrict__ image,
                                                                       int k, int64_t ldg, const float* __restrict__ scale_ref,
                                                                       float rel_tol) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  chol_load(G, ldg, k, smem);
  chol_factor_lds(smem, k, scale_ref, rel_tol);
  const int chunks = chol_image_bytes(k) / 16;
  for (int e = threadIdx.x; e < chunks; e += (int)blockDim.x) ((f32x4*)image)[e] = ((const f32x4*)smem)[e];
}

// Q = Y . R^-1 for a tall Y [n, k] fp32 by forward substitution over 16-column blocks:
//   Q_J = (Y_J - sum_{I < J} (Q_I D_I^-1/2) V_JI^T) L_JJ^-T D_J^-1/2
// with the factor (chol_factor_lds) in LDS; every product on the 16x16x4 instruction.  A wave owns 16 rows and keeps all their
// columns in registers: a finished block sits in the accumulator layout, which is the layout the next products want their left
// operand in, so nothing moves between lanes.
// Outputs, each optional, rows up to n_rows_out (>= n; rows past n count as zero):
//   Qf  [n, k] fp32 (may be Y itself: a wave reads its rows before it writes them);  Qt [n, k] in TU (the stored
//   factor);  Ut [k, ldt] bf16, the transpose with its columns n .. n_rows_out - 1 written as zero (K padding of the later
//   products over tokens); with `hilo` rows lo_rows .. hold the bf16 rounding of what the rounding of Q^T leaves, so that hi +
//   lo carries Q to about 2^-17 relative through a bf16 matrix product.
// ldy: row stride of Y; ldq: row stride of Qf and Qt (a column block of a wider matrix passes the wide stride).
template <typename TU> struct TriSolve {
  const float* Y;
  float* Qf;
  TU* Qt;
  bf16* Ut;
  int64_t n, ldy, ldq, ldt, n_rows_out;
  int k, hilo, lo_rows;

  template <int KB> __device__ __forceinline__ void load(f32x4 (&q)[KB], int64_t row, int g4) const {
#pragma unroll
    for (int J = 0; J < KB; ++J) {
      q[J] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int col = J * 16 + g4 * 4;
      if (row < n && col < k) q[J] = *(const f32x4*)(Y + row * ldy + col);
    }
  }
  template <int KB> __device__ __forceinline__ void solve(const char* factor, f32x4 (&q)[KB], int64_t row, int l16, int g4) const {
    const int nb = (k + 15) / 16;
    const float* const scale = (const float*)(factor + tri_block(nb, 0) * 1024);
    auto block = [&](int J, int I) -> f32x4 { return *(const f32x4*)(factor + tri_block(J, I) * 1024 + l16 * 64 + g4 * 16); };
#pragma unroll
    for (int J = 0; J < KB; ++J) {
      if (J < nb) {
        // what the block subtracts is summed by itself and joins the row at the end: a product added to the row is rounded at
        // the row's size, 16 J times (error of U [4096, 256] against 64 bits: 2.4e-7 so, 0.9e-7 with the sums by themselves)
        f32x4 sum[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int I = 0; I < J; I += 2) {   // two chains, in turn
          const f32x4 r0 = block(J, I), r1 = block(J, I + 1 < J ? I + 1 : I);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            sum[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(r0[t], q[I][t], sum[0], 0, 0, 0);
            if (I + 1 < J) sum[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(r1[t], q[I + 1][t], sum[1], 0, 0, 0);
          }
        }
        const f32x4 rest = q[J] - (sum[0] + sum[1]), d = block(J, J) * scale[J * 16 + l16];
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) o = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t], rest[t], o, 0, 0, 0);
        q[J] = o * *(const f32x4*)(scale + J * 16 + g4 * 4);   // Q_J D^-1/2: what the later columns subtract V's multiples of
        store(o, row, J * 16 + g4 * 4);
      }
    }
  }
  __device__ __forceinline__ void store(f32x4 o, int64_t row, int col) const {
    if (col >= k) return;
    if (row < n) {
      if (Qf) *(f32x4*)(Qf + row * ldq + col) = o;
      if (Qt) {
        if constexpr (sizeof(TU) == 2) *(bf16x4*)(Qt + row * ldq + col) = bf16x4{(bf16)o[0], (bf16)o[1], (bf16)o[2], (bf16)o[3]};
        else *(f32x4*)(Qt + row * ldq + col) = o;
      }
    }
    if (Ut && row < n_rows_out) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bf16 hi = row < n ? (bf16)o[t] : (bf16)0.f;
        Ut[(int64_t)(col + t) * ldt + row] = hi;
        if (hilo) Ut[(int64_t)(lo_rows + col + t) * ldt + row] = row < n ? (bf16)(o[t] - (float)hi) : (bf16)0.f;
      }
    }
  }
};

// The solve with a factor from global memory, copied to LDS once per work-group.  Work-groups of any number
// of waves; grid: rows of the launch / 16.  k % 8 == 0, k <= 16 KB.
template <int KB, typename TU>
__global__ __launch_bounds__(512) void chol_solve_kernel(TriSolve<TU> p, const float* __restrict__ image) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int bytes = chol_image_bytes(p.k), blocks = (bytes + 1023) / 1024;
  const int tid = threadIdx.x, lane = tid & 63, waves = (int)(blockDim.x >> 6);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  {
    const u32x4 rsrc = make_rsrc(image, bytes);
    const uint32_t smem_lds = (uint32_t)(uintptr_t)smem;
    for (int b = wave; b < blocks; b += waves) buffer_to_lds_b128(rsrc, (uint32_t)(lane * 16), (uint32_t)(b * 1024), smem_lds + b * 1024);
  }
  const int64_t row = ((int64_t)blockIdx.x * waves + wave) * 16 + l16;
  f32x4 q[KB];
  p.template load<KB>(q, row, g4);
  wait_vmcnt0();
  __syncthreads();
  p.template solve<KB>(smem, q, row, l16, g4);
}

// Factor and solve in one launch (ranks up to 128): EVERY work-group factors the same G (36 KB at k = 128, from L2), then its
// waves solve blocks of 16 rows.  The factorisation is a chain that one work-group cannot share with others, so doing it 256
// times over costs nothing, and the factor neither leaves the compute unit nor waits for a launch.
// Row blocks go to the work-groups first: with few of them each has a compute unit of its own.
template <int KB, typename TU>
__global__ __launch_bounds__(512) void cholesky_qr_kernel(TriSolve<TU> p, const float* __restrict__ G, float rel_tol) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, waves = (int)(blockDim.x >> 6);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t step = (int64_t)gridDim.x * waves * 16;
  int64_t r0 = ((int64_t)wave * gridDim.x + blockIdx.x) * 16;
  f32x4 q[KB];
  p.template load<KB>(q, r0 + l16, g4);   // arrives under the factorisation
  chol_load(G, p.k, p.k, smem);
  chol_factor_lds(smem, p.k, nullptr, rel_tol);
  for (bool first = true; r0 < p.n_rows_out; r0 += step, first = false) {
    if (!first) p.template load<KB>(q, r0 + l16, g4);
    p.template solve<KB>(smem, q, r0 + l16, l16, g4);
  }
}

// out[0] = the largest diagonal entry of the symmetric matrix G [k, k] (row stride ldg).  One wave.
__global__ __launch_bounds__(64) void diag_max_kernel(const float* __restrict__ G, int k, int64_t ldg,
                                                      float* __restrict__ out) {
  float m = 0.f;
  for (int i = threadIdx.x; i < k; i += 64) {
    const float d = G[i * ldg + i];
    m = d > m ? d : m;
  }
#pragma unroll
  for (int l = 0; l < 64; ++l) {
    const float d = lane_bcast(m, l);
    if (threadIdx.x == 0 && l > 0) m = d > m ? d : m;
  }
  if (threadIdx.x == 0) out[0] = m;
}

// out[e] = sum over p of part[p * E + e] in a fixed order: a work-group owns 64 elements, its wave w adds parts w,
// w + 16, ..., then the 16 wave sums are added pairwise.  Grid ceil(E / 64) x 1024 threads.
__global__ __launch_bounds__(1024) void sum_parts_kernel(const float* __restrict__ part, int P, int64_t E,
                                                         float* __restrict__ out) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  float s = 0.f;
  if (e < E) {
#pragma unroll 8
    for (int p = wave; p < P; p += 16) s += part[(int64_t)p * E + e];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && e < E) {
    float sum[16];
#pragma unroll
    for (int w = 0; w < 16; ++w) sum[w] = red[w][lane];
#pragma unroll
    for (int half = 8; half > 0; half >>= 1)
#pragma unroll
      for (int w = 0; w < half; ++w) sum[w] += sum[w + half];
    out[e] = sum[0];
  }
}

// Omega [d_in, k] of the range finder as two bfloat16 matrices, Omega = hi + lo to about 2^-17 relative
// (one bfloat16 MFMA pass per part gives fp32-grade products with exact bf16 inputs).  Output layout
// [2k, ld] K-contiguous rows: row j = hi of column j, row k + j = lo of column j; entry (c, j) is the
// Philox normal of (token index := c, column j), scaled by 1 / sqrt(k) like S.  One thread per (4
// channels, column).  d_in % 4 == 0.
__global__ __launch_bounds__(256) void omega_hilo_kernel(SketchParams sk, int64_t d_in, int k, int64_t ld,
                                                         bf16* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // = q * k + j
  const int64_t nq = d_in / 4;
  if (idx >= nq * k) return;
  const int64_t q = idx / k;
  const int j = (int)(idx - q * k);
  uint32_t w[4];
  sketch_words(sk.key0, sk.key1, (uint64_t)q, (uint32_t)j, w);
  float z[4];
  normals_from_words<true>(w, sk.inv_sqrt_r, sk.neg2_ln2_over_r, z);
  bf16x4 hi, lo;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    hi[t] = (bf16)z[t];
    lo[t] = (bf16)(z[t] - (float)hi[t]);
  }
  *(bf16x4*)(out + (int64_t)j * ld + 4 * q) = hi;
  *(bf16x4*)(out + (int64_t)(k + j) * ld + 4 * q) = lo;
}

// The kernels below fold the splits of a skinny product in a fixed order, one thread per element with coalesced reads.  They are
// bound by the latency of those reads, so a thread asks for several splits at a time.

// Yr[i, j] = sum over splits of (part[s][i][j] + part[s][i][k + j]): folds the K splits and the hi / lo
// halves of X . [Omega_hi Omega_lo].
__global__ __launch_bounds__(256) void combine_hilo_kernel(const float* __restrict__ part, int splits, int64_t n,
                                                           int k, float* __restrict__ Yr) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n * k) return;
  const int64_t i = idx / k;
  const int j = (int)(idx - i * k);
  float sum = 0.f;
#pragma unroll 4
  for (int s = 0; s < splits; ++s) {
    const float* row = part + ((int64_t)s * n + i) * (2 * k);
    sum += row[j] + row[k + j];
  }
  Yr[idx] = sum;
}

// Z [cols, k] = transpose of the sum over splits of (part[s][j][c] + part[s][k + j][c]), part[s] being
// [2k, cols] fp32: folds the K splits and the hi / lo halves of [Q_hi; Q_lo]^T-type products.
__global__ __launch_bounds__(256) void combine_hilo_t_kernel(const float* __restrict__ part, int splits, int64_t cols,
                                                             int k, float* __restrict__ Z) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // = j * cols + c
  if (idx >= (int64_t)k * cols) return;
  const int64_t j = idx / cols, c = idx - j * cols;
  float sum = 0.f;
#pragma unroll 4
  for (int s = 0; s < splits; ++s) {
    const float* p = part + (int64_t)s * 2 * k * cols;
    sum += p[j * cols + c] + p[(k + j) * cols + c];
  }
  Z[c * k + j] = sum;
}

// Ut [k, ld] = U^T with the columns n .. ld - 1 zeroed (ld = n rounded up to 64: the K padding of the products over tokens).  A
// work-group takes a 16 x 16 tile through LDS, so that the writes are runs of 16 tokens instead of single ones: 4096 x 128 3.9
// us (7.0 one by one).  Folds with many splits to read gained nothing from the same tile.
// Grid: ld / 16 * ceil(k / 16).
template <typename TU>
__global__ __launch_bounds__(256) void transpose_pad_kernel(const TU* __restrict__ U, int64_t n, int k, int64_t ld,
                                                            bf16* __restrict__ Ut) {
  __shared__ float tile[16][17];
  const int col_tiles = (k + 15) / 16, x = threadIdx.x & 15, y = threadIdx.x >> 4;
  const int64_t i0 = (int64_t)(blockIdx.x / (unsigned)col_tiles) * 16;
  const int j0 = (int)(blockIdx.x % (unsigned)col_tiles) * 16;
  if (i0 + y < n && j0 + x < k) tile[y][x] = to_f32(U[(i0 + y) * k + j0 + x]);
  __syncthreads();
  if (j0 + y < k) Ut[(int64_t)(j0 + y) * ld + i0 + x] = i0 + x < n ? (bf16)tile[x][y] : (bf16)0.f;
}

// out = sum over splits of part[s] ([rows, cols] fp32 each), stored transposed ([cols, rows]) when
// TRANSPOSE, converted to TO.  128 x 2048 in 16 splits 7.0 us with one split requested at a time.
template <typename TO, bool TRANSPOSE>
__global__ __launch_bounds__(256) void reduce_store_kernel(const float* __restrict__ part, int splits, int64_t rows,
                                                           int64_t cols, TO* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= rows * cols) return;
  float sum = part[idx];
#pragma unroll 8
  for (int s = 1; s < splits; ++s) sum += part[(int64_t)s * rows * cols + idx];
  if (TRANSPOSE) {
    const int64_t r = idx / cols, c = idx - r * cols;
    out[c * rows + r] = from_f32<TO>(sum);
  } else {
    out[idx] = from_f32<TO>(sum);
  }
}

}  // namespace acc
