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

// The upper triangular factor R of G = R^T R (G [k, k] symmetric positive semi-definite, fp32, k <= 256, positive diagonal
// of R) in the form chol_solve_kernel multiplies with, by ONE work-group.  The k steps of an elimination are a serial chain;
// what a step costs is everything.  Blocked by 16 columns, G in LDS:
//   panel     one row below the diagonal block per lane, its 16 panel columns in registers, and beside it row lane % 16 of
//             the block itself, the same in every 16 lanes: the pivot row comes from lane j of each 16 by a DPP broadcast
//             inside the multiply-add, so the 16 steps need neither LDS, scalar registers nor a barrier, and no wave
//             waits for another.  (With v_readlane broadcasts instead, two wait states each: 25 / 73 us at k = 128 / 256.)
//   trailing  A_il -= (V_i D^-1) V_l^T on the 16x16x4 instruction, blocks dealt to the waves
// in the square-root-free form (A = L D L^T, one reciprocal per step on the chain).  Rows of finished panels are never read
// again above the diagonal, so the elimination runs unmasked.
// Image (tri_block layout): off-diagonal block (J, I): [n][t] = -R[16 I + t][16 J + n]; diagonal block: the inverse of
// R_JJ, transposed, [n][t] = (R_JJ^-1)[t][n].
// A pivot at or below rel_tol times the largest diagonal entry (of G, or *scale_ref: of the matrix G is a block of) counts
// as zero: column j of the factored matrix depends on the earlier ones.  Its row and column of the image are zero, so the
// corresponding basis vector comes out as zero and the span of the others is unchanged.
// Measured at k = 32 / 64 / 128 / 256: 8 / 12 / 23 / 62 us.  The one-wave elimination this replaced (the pivot row
// through LDS at every step, one matrix row per lane, 64 columns at most) took 12 / 39 us, and ranks above 64 a chain of
// three launches per 64 columns: about 115 us at k = 128.
__global__ __launch_bounds__(kCholMaxThreads) void chol_factor_kernel(const float* __restrict__ G, float* __restrict__ image,
                                                                      int k, int64_t ldg, const float* __restrict__ scale_ref,
                                                                      float rel_tol) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int NW = (int)(blockDim.x >> 6);
  float* const A = (float*)smem;                                     // tri_block storage
  const int nb = (k + 15) / 16;
  float* const inv = A + tri_block(nb, 0) * 256;                     // 1 / pivot per column, 0 for a dropped one
  float* const scale = inv + nb * 16;                                // 1 / sqrt(pivot), likewise
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  auto at = [&](int i, int l) -> f32x4* { return (f32x4*)(A + tri_block(i, l) * 256 + l16 * 16 + g4 * 4); };

  // ---- load: block b of the triangle by wave b mod NW, four requested at a time; rows and columns past k as the identity ----
  const int blocks = tri_block(nb, 0);
  for (int b0 = wave; b0 < blocks; b0 += 4 * NW) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + u * NW;
      if (b < blocks) {
        const TriIndex x = tri_index(b);
        const int row = x.i * 16 + l16, col = x.l * 16 + g4 * 4;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[u][t] = row == col + t ? 1.f : 0.f;
        if (row < k && col < k) v[u] = *(const f32x4*)(G + row * ldg + col);  // k % 4 == 0
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + u * NW;
      if (b < blocks) *(f32x4*)(A + b * 256 + l16 * 16 + g4 * 4) = v[u];
    }
  }
  __syncthreads();
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

  // Inverse of diagonal block J by lanes 0 .. 15 of one wave: lane n solves R x = e_n from the last row up.
  // R[j][t] = V[t][j] scale[j] with V the stored lower triangle; a dropped row has scale 0, which makes x[j] zero.
  auto invert = [&](int J) {
    const float* V = A + tri_block(J, J) * 256;
    float x[16];
#pragma unroll
    for (int j = 15; j >= 0; --j) {
      const float s = scale[J * 16 + j];
      float sum = 0.f;
#pragma unroll
      for (int t = j + 1; t < 16; ++t) sum = fmaf(V[t * 16 + j], x[t], sum);
      x[j] = l16 == j ? s : (l16 > j ? -(s * s) * sum : 0.f);
    }
    float* dst = image + tri_block(J, J) * 256 + l16 * 16;
    if (lane < 16) {
#pragma unroll
      for (int c = 0; c < 16; c += 4) *(f32x4*)(dst + c) = f32x4{x[c], x[c + 1], x[c + 2], x[c + 3]};
    }
  };

  for (int p = 0; p < nb; ++p) {
    // ---- panel ----
    const int below = (nb - p - 1) * 16;
    float d[16];
    if (wave == 0 || wave * 64 < below) {
      const int r = wave * 64 + lane;     // row below the diagonal block
      const bool real = r < below;
      const float* diag = A + tri_block(p, p) * 256 + l16 * 16;
      float* row = A + tri_block(p + 1 + (r >> 4), p) * 256 + l16 * 16;
      float a[16], pivots[16], inverses[16];
#pragma unroll
      for (int c = 0; c < 16; c += 4) {
        const f32x4 v = real ? *(const f32x4*)(row + c) : f32x4{0.f, 0.f, 0.f, 0.f}, w = *(const f32x4*)(diag + c);
#pragma unroll
        for (int t = 0; t < 4; ++t) { a[c + t] = v[t]; d[c + t] = w[t]; }
      }
      static_for<0, 16>([&](auto step) {
        constexpr int j = decltype(step)::value;
        const float piv = bcast16<j>(d[j]);
        const bool dead = !(piv > tol);
        // reciprocal: hardware estimate + one Newton step (about 1 ulp); the factor's own scaling uses square roots
        float inv_p = __builtin_amdgcn_rcpf(piv);
        inv_p = fmaf(fmaf(-piv, inv_p, 1.f), inv_p, inv_p);
        inv_p = dead ? 0.f : inv_p;
        inverses[j] = inv_p;
        pivots[j] = dead ? 0.f : piv;
        const float td = -(d[j] * inv_p), ta = -(a[j] * inv_p);
#pragma unroll
        for (int c = j + 1; c < 16; ++c) {
          const float u = bcast16<j>(d[c]);
          d[c] = fmaf(u, td, d[c]);
          a[c] = fmaf(u, ta, a[c]);
          // used under a condition only: without this the compiler moves the rows' updates there, behind the block's
          // sixteen steps, and keeps (spills) all their broadcasts until then
          asm volatile("" : "+v"(a[c]));
        }
      });
      if (real) {
#pragma unroll
        for (int c = 0; c < 16; c += 4) *(f32x4*)(row + c) = f32x4{a[c], a[c + 1], a[c + 2], a[c + 3]};
      }
      if (wave == 0 && lane == 0) {  // every lane holds all 16 pivots
#pragma unroll
        for (int c = 0; c < 16; c += 4) {
          *(f32x4*)(inv + p * 16 + c) = f32x4{inverses[c], inverses[c + 1], inverses[c + 2], inverses[c + 3]};
          *(f32x4*)(scale + p * 16 + c) = f32x4{pivots[c], pivots[c + 1], pivots[c + 2], pivots[c + 3]};
        }
      }
    }
    __syncthreads();
    if (wave == 0 && lane < 16) {  // only now: until the barrier the other waves were reading the block; all their copies are the same
      float* row = A + tri_block(p, p) * 256 + lane * 16;
#pragma unroll
      for (int c = 0; c < 16; c += 4) *(f32x4*)(row + c) = f32x4{d[c], d[c + 1], d[c + 2], d[c + 3]};
      const float piv = scale[p * 16 + lane];
      scale[p * 16 + lane] = piv > 0.f ? 1.f / sqrtf(piv) : 0.f;
    }
    // ---- trailing blocks (i, l), p < l <= i: rows of V_i against rows of V_l over the panel's 16 columns, two at a time ----
    {
      const f32x4 d = *(const f32x4*)(inv + p * 16 + g4 * 4);
      const int count = (nb - p - 1) * (nb - p) / 2;
      for (int b0 = wave; b0 < count; b0 += 2 * NW) {
        f32x4 c[2], vi[2], vl[2];
        f32x4* dst[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int b = b0 + u * NW;
          const TriIndex x = tri_index(b < count ? b : b0);
          const int i = x.i + p + 1, l = x.l + p + 1;
          vi[u] = *at(i, p); vl[u] = *at(l, p); dst[u] = at(i, l);
          c[u] = *dst[u];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            c[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(vl[u][t], -(vi[u][t] * d[t]), c[u], 0, 0, 0);
        *dst[0] = c[0];
        if (b0 + NW < count) *dst[1] = c[1];
      }
    }
    __syncthreads();
  }
  for (int J = wave; J < nb; J += NW) invert(J);  // all at once: one beside each panel was the slower of the two

  // ---- off-diagonal blocks of the image ----
  for (int b = wave; b < blocks; b += NW) {
    const TriIndex x = tri_index(b);
    if (x.l < x.i) {
      const f32x4 s = *(const f32x4*)(scale + x.l * 16 + g4 * 4);
      const f32x4 v = *(const f32x4*)(A + b * 256 + l16 * 16 + g4 * 4);
      *(f32x4*)(image + b * 256 + l16 * 16 + g4 * 4) = f32x4{-(v[0] * s[0]), -(v[1] * s[1]), -(v[2] * s[2]), -(v[3] * s[3])};
    }
  }
}

constexpr int chol_lds_bytes(int k) { return tri_block((k + 15) / 16, 0) * 1024 + (k + 15) / 16 * 16 * 2 * 4; }

// Q = Y . R^-1 for a tall Y [n, k] fp32 by forward substitution over 16-column blocks:
//   Q_J = (Y_J - sum_{I < J} Q_I R_IJ) R_JJ^-1
// with the 16 x 16 inverses of chol_factor_kernel's image; every product on the 16x16x4 instruction.  A wave owns 16 rows
// and keeps all their columns in registers: a finished block sits in the accumulator layout, which is the layout the next
// products want their left operand in, so nothing moves between lanes.  The image is copied to LDS once per work-group.
// Replaced one lane per row with the columns in registers and R broadcast from LDS, 64 columns at most (22 us each).
// Outputs, each optional, rows up to n_rows_out (>= n; rows past n count as zero):
//   Qf  [n, k] fp32 (may be Y itself: a wave reads its rows before it writes them);  Qt [n, k] in TU (the stored factor);
//   Ut [k, ldt] bf16, the transpose with its columns n .. n_rows_out - 1 written as zero (K padding of the later products
//   over tokens); with `hilo` rows lo_rows .. hold the bf16 rounding of what the rounding of Q^T leaves, so that hi + lo
//   carries Q to about 2^-17 relative through a bf16 matrix product.
// Work-groups of any number of waves; grid: rows of the launch / 16.  k % 8 == 0, k <= 16 KB.
template <int KB, typename TU>
__global__ __launch_bounds__(512) void chol_solve_kernel(const float* __restrict__ Y, int64_t n, int k,
                                                         const float* __restrict__ image, float* Qf,
                                                         TU* __restrict__ Qt, bf16* __restrict__ Ut, int64_t ldt,
                                                         int64_t n_rows_out, int hilo, int64_t ldy, int64_t ldq, int lo_rows) {
  // ldy: row stride of Y; ldq: row stride of Qf and Qt (a column block of a wider matrix passes the wide stride)
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int nb = (k + 15) / 16, blocks = tri_block(nb, 0);
  const int tid = threadIdx.x, lane = tid & 63, waves = (int)(blockDim.x >> 6);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  {
    const u32x4 rsrc = make_rsrc(image, (int64_t)blocks * 1024);
    const uint32_t smem_lds = (uint32_t)(uintptr_t)smem;
    for (int b = wave; b < blocks; b += waves) buffer_to_lds_b128(rsrc, (uint32_t)(lane * 16), (uint32_t)(b * 1024), smem_lds + b * 1024);
  }
  const int64_t row = ((int64_t)blockIdx.x * waves + wave) * 16 + l16;
  f32x4 q[KB];
#pragma unroll
  for (int J = 0; J < KB; ++J) {
    q[J] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int col = J * 16 + g4 * 4;
    if (row < n && col < k) q[J] = *(const f32x4*)(Y + row * ldy + col);
  }
  wait_vmcnt0();
  __syncthreads();
  auto block = [&](int J, int I) -> f32x4 { return *(const f32x4*)(smem + tri_block(J, I) * 1024 + l16 * 64 + g4 * 16); };
#pragma unroll
  for (int J = 0; J < KB; ++J) {
    if (J < nb) {
      // two chains, and the row itself joins at the end: a product added to it is rounded at the row's size, 16 J times
      // (error of U [4096, 256] against 64 bits: 2.4e-7 so, 0.9e-7 with the sums by themselves)
      f32x4 c[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int I = 0; I < J; ++I) {
        const f32x4 r = block(J, I);
#pragma unroll
        for (int t = 0; t < 4; ++t) c[I & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[t], q[I][t], c[I & 1], 0, 0, 0);
      }
      const f32x4 rest = q[J] + (c[0] + c[1]), d = block(J, J);
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t) o = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t], rest[t], o, 0, 0, 0);
      q[J] = o;
      const int col = J * 16 + g4 * 4;
      if (col < k) {
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
    }
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

// Yr[i, j] = sum over splits of (part[s][i][j] + part[s][i][k + j]): folds the K splits and the hi / lo
// halves of X . [Omega_hi Omega_lo] in a fixed order.  One thread per element.
__global__ __launch_bounds__(256) void combine_hilo_kernel(const float* __restrict__ part, int splits, int64_t n,
                                                           int k, float* __restrict__ Yr) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n * k) return;
  const int64_t i = idx / k;
  const int j = (int)(idx - i * k);
  float sum = 0.f;
  for (int s = 0; s < splits; ++s) {
    const float* row = part + ((int64_t)s * n + i) * (2 * k);
    sum += row[j] + row[k + j];
  }
  Yr[idx] = sum;
}

// Z [cols, k] = transpose of the sum over splits of (part[s][j][c] + part[s][k + j][c]), part[s] being
// [2k, cols] fp32: folds the K splits and the hi / lo halves of [Q_hi; Q_lo]^T-type products in a fixed
// order.  One thread per input column pair (c, j), coalesced reads.
__global__ __launch_bounds__(256) void combine_hilo_t_kernel(const float* __restrict__ part, int splits, int64_t cols,
                                                             int k, float* __restrict__ Z) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // = j * cols + c
  if (idx >= (int64_t)k * cols) return;
  const int64_t j = idx / cols, c = idx - j * cols;
  float sum = 0.f;
  for (int s = 0; s < splits; ++s) {
    const float* p = part + (int64_t)s * 2 * k * cols;
    sum += p[j * cols + c] + p[(k + j) * cols + c];
  }
  Z[c * k + j] = sum;
}

// Ut [k, ld] = U^T with the columns n .. ld - 1 zeroed (ld = n rounded up to 64: the K padding of the
// products over tokens).  One thread per output element.
template <typename TU>
__global__ __launch_bounds__(256) void transpose_pad_kernel(const TU* __restrict__ U, int64_t n, int k, int64_t ld,
                                                            bf16* __restrict__ Ut) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // = i * k + j: coalesced read
  if (idx >= ld * k) return;
  const int64_t i = idx / k;
  const int j = (int)(idx - i * k);
  Ut[(int64_t)j * ld + i] = i < n ? (bf16)to_f32(U[idx]) : (bf16)0.f;
}

// out = sum over splits of part[s] ([rows, cols] fp32 each), stored transposed ([cols, rows]) when
// TRANSPOSE, converted to TO.  One thread per input element (coalesced reads).
template <typename TO, bool TRANSPOSE>
__global__ __launch_bounds__(256) void reduce_store_kernel(const float* __restrict__ part, int splits, int64_t rows,
                                                           int64_t cols, TO* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= rows * cols) return;
  float sum = part[idx];
  for (int s = 1; s < splits; ++s) sum += part[(int64_t)s * rows * cols + idx];
  if (TRANSPOSE) {
    const int64_t r = idx / cols, c = idx - r * cols;
    out[c * rows + r] = from_f32<TO>(sum);
  } else {
    out[idx] = from_f32<TO>(sum);
  }
}

}  // namespace acc
