// The B x B solve of stochastic reconfiguration on the device (Sec. 2.1: natural gradient
// with the Fisher information of the per-sample scores; Sec. 5.1: SR with a ridge lambda).
// In sample space the SR direction for the batch gradient g = O^T c is x = O^T y with
//
//     (K + lambda B I) y = B c,      K = O O^T   (symmetric positive semi-definite),
//
// so the only dense linear algebra is this B x B system.  It is solved in FP64 by a blocked
// right-looking Cholesky factorisation L L^T = K + shift I (64 x 64 blocks, the matrix padded
// to a multiple of 64 with identity rows) and a blocked back substitution L^T y = w.  The
// right-hand side is one more row of the matrix (row ld; as block row nb every row of the block is that
// one, and the first is stored): the block-row solve that makes L_ij out of A_ij turns it into
// w = L^-1 rhs.  The factor of a diagonal block is kept right of it (chol_diag), above the diagonal,
// where the matrix is not used.
//
// Launches, nb = padded B / 64 block columns:
//   chol_init_kernel    the lower triangle of K + shift I in FP64, and the right-hand side;
//   chol_step_kernel    one per block column (j = -1 .. nb - 2): block column j + 1 is updated from
//                       column j, factored and solved for, beside the rest of column j's update;
//   chol_back_kernel    one: the block rows of L^T y = w, each workgroup waiting for the later ones.
#include "common.hpp"
#include "kernels.hpp"

#include <utility>

namespace vqmc {

constexpr int CB = 64;       // block edge
constexpr int CP = 16;       // columns factored at a time inside a diagonal block
constexpr int CL = CB + 2;   // LDS row stride (doubles): 16-byte aligned rows, 16 rows spread over the banks

// y entries not yet known to chol_back_kernel: a NaN no arithmetic produces
constexpr unsigned long long kUnknown = 0xFFF8C0DEC0DEC0DEull;

// Lower triangle (by blocks) of K + shift I on the B x B part, identity on the padding; row ld is
// scale * rhs.
__global__ void chol_init_kernel(const float* __restrict__ K, int64_t B, int64_t ld, double shift,
                                 const float* __restrict__ rhs, double scale, double* __restrict__ A,
                                 unsigned long long* __restrict__ y) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= ld * (ld + 1)) return;
  const int64_t r = idx / ld, c = idx - r * ld;
  if (r / CB < c / CB) return;
  double v;
  if (r == ld) v = c < B ? scale * (double)rhs[c] : 0.0;
  else if (r < B && c < B) v = (double)K[r * B + c] + (r == c ? shift : 0.0);
  else v = (r == c) ? 1.0 : 0.0;
  A[idx] = v;
  if (r == ld) y[c] = kUnknown;
}

// The factor of diagonal block i (row stride ld): in the block right of it, which nothing else uses; the
// last one in place, where the one workgroup of its step has read the block already
__device__ inline double* chol_diag(double* A, int64_t ld, int nb, int i) {
  return A + (int64_t)i * CB * ld + (int64_t)min(i + 1, nb - 1) * CB;
}

// The counter that deals the blocks of the back substitution: in the first diagonal block, which is free once its
// factor lies beside it (nb > 1); cleared by the second step
__device__ inline int* chol_ticket(double* A) { return (int*)A; }

// 1 / sqrt(d): the hardware estimate (about 24 bits) and one step of third order,
// r (1 + e/2 + 3 e^2/8) with e = 1 - d r^2, accurate to a few ulp; NaN for d <= 0.
__device__ inline double chol_rsqrt(double d) {
  const double r = __builtin_amdgcn_rsq(d);
  const double e = fma(-(d * r), r, 1.0);
  return fma(r, e * fma(e, 0.375, 0.5), r);
}

__device__ inline double chol_bcast(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Operands of v_mfma_f64_16x16x4: lane (r = l % 16, g = l / 16) supplies row r at one k of four.
// Both operands take the ks in the same permuted order - lane group g the ks 4 g .. 4 g + 3 of each
// run of sixteen - so that a lane's values are 32 contiguous bytes.  Entry e of the result sits at
// row 4 e + g, column r.
template <int NK>
__device__ inline void chol_frag(const double* row, double (&v)[NK]) {
#pragma unroll
  for (int q = 0; q < NK / 4; ++q) {
    const double2 a = *(const double2*)(row + 16 * q), b = *(const double2*)(row + 16 * q + 2);
    v[4 * q] = a.x;
    v[4 * q + 1] = a.y;
    v[4 * q + 2] = b.x;
    v[4 * q + 3] = b.y;
  }
}

// acc -= (src of lane N of the lane's row of 16) * mul.  The DPP read of src needs two wait states after
// the instruction that wrote it, which the compiler does not see in here: chol_scale and
// chol_next, the only writers of a src, end with them.  (tests/test_dpp_wait_states.py reads the built assembly for copies
// that the register allocator might put in between.)
template <int N>
__device__ inline void chol_fnma_row(double& acc, double src, double mul) {
  __asm__("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(src), "v"(mul), "n"(N));
}
template <int N>
__device__ inline void chol_next(double& acc, double src, double mul) {
  __asm__("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n\ts_nop 1"
          : "+v"(acc)
          : "v"(src), "v"(mul), "n"(N));
}
__device__ inline void chol_scale(double& x, double s) {
  __asm__("v_mul_f64 %0, %0, %1\n\ts_nop 1" : "+v"(x) : "v"(s));
}
template <int N>
__device__ inline double chol_row(double v) {  // v of lane N of the lane's row of 16
  return __builtin_amdgcn_update_dpp(v, v, 0x150 + N, 0xF, 0xF, true);
}

// Columns C .. 15 of a 16 x 16 diagonal tile and of the rows below it, one wave: every row of 16 lanes
// holds the tile (x, a row per lane) and a row y of its own, so that pivots and multipliers are
// broadcasts inside the 16 lanes (DPP, an operand of the multiply-add itself) and never pass through
// scalar registers or LDS.  y ends up as y L^-T, x as the rows of L.
// columns C0 + I of v -= (column C of L, by its rows C0 + I) * m
template <int C, int C0, int... I>
__device__ inline void chol_rank1(double (&v)[CP], const double (&x)[CP], double m, std::integer_sequence<int, I...>) {
  (chol_fnma_row<C0 + I>(v[C0 + I], x[C], m), ...);
}
template <int C>
__device__ inline void chol_columns(double (&x)[CP], double (&y)[CP], double rs) {
  chol_scale(x[C], rs);
  y[C] *= rs;
  if constexpr (C + 1 < CP) {
    chol_next<C + 1>(x[C + 1], x[C], x[C]);
    const double next = chol_rsqrt(chol_row<C + 1>(x[C + 1]));
    chol_rank1<C, C + 1>(y, x, y[C], std::make_integer_sequence<int, CP - 1 - C>{});
    if constexpr (C + 2 < CP) chol_rank1<C, C + 2>(x, x, x[C], std::make_integer_sequence<int, CP - 2 - C>{});
    chol_columns<C + 1>(x, y, next);
  }
}

// Block column j is factored (j = -1: none yet) and blocks right of column j still lack its update.
// The first nb - j - 1 workgroups carry the critical path: workgroup p takes block row
// i = j + 2 + p (i = nb: the right-hand side), updates the diagonal block (j + 1, j + 1) and its own
// block (i, j + 1) from column j with FP64 MFMA, factors the diagonal block and solves
// X L^T = A_i,j+1; every one of them factors the diagonal block for itself (the same arithmetic),
// which costs nothing next to a second launch.  The other workgroups apply column j to the
// remaining blocks (i, k), k >= j + 2, meanwhile.
//
// What bounds it: the chain of 64 columns, one pivot after another, and the instruction fetch of code
// that every launch runs once (so the loops over panels and tiles stay rolled).  Wave 0 factors
// sixteen columns at a time (chol_columns), the identity riding along as sixteen more rows that come
// out as L_pp^-T; waves 0 - 3 apply column j and the panels to the rest of the diagonal block with
// MFMA, the tiles of the next sixteen columns first, the others while wave 0 is at work on those.
// Four waves (1, 5 - 7) hold sixteen rows of the own block each, as transposed tiles: a result tile of an
// MFMA is then the operand of the next one as it stands, and the block-row solve, a panel behind
// wave 0, is a product with L_pp^-1 and an update per panel.  FP64 MFMA and FP64 vector instructions
// of a SIMD share their units, so nothing else runs on the SIMD of wave 0 (wave 4 stands idle).
//
// Measured, cycles of a panel workgroup per block column at B = 2048: 28 000, of which the loads 5 000, column
// j on the first tiles 2 200, the four panels 3 400 each and 800 - 2 200 between them.  The whole
// solve takes 0.60 ms at B = 2048 and 0.285 ms at B = 1024 (1.63 and 0.77 ms with the diagonal factor,
// the block-row solve and the update in two launches per block column, their chains through LDS, and
// a launch per block of the back substitution).  On the way, same shapes: the block-row solve in
// wave 0 beside the factor 0.95 ms; the panels' multipliers through v_readlane (8 - 10 cycles each)
// 0.69 ms; the panel and tile loops unrolled (32 KB of code, fetched anew by every launch) 0.74 ms.
constexpr int CW = 8;   // waves per workgroup
__global__ __launch_bounds__(64 * CW) void chol_step_kernel(double* __restrict__ A, int64_t ld, int nb, int j) {
  __shared__ __align__(16) double D[CB][CL];               // diagonal block (j + 1, j + 1)
  __shared__ __align__(16) double Ls[CB][CL];              // L_j+1,j
  __shared__ __align__(16) double V[CB / CP][CP][CP + 2];  // L_pp^-1
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int64_t jc = (int64_t)j * CB;  // first column of block column j
  const int npanel = nb - j - 1;
  if ((int)blockIdx.x >= npanel) {
    // remaining blocks of column j's update, row by row: row q (block row j + 2 + q, the last one
    // the right-hand side) holds min(q + 1, m) blocks, m = nb - j - 2 columns
    const int m = nb - j - 2;
    const int x = (int)blockIdx.x - npanel;
    int q = (int)((sqrtf(8.f * (float)x + 1.f) - 1.f) * 0.5f);
    while ((int64_t)q * (q + 1) / 2 > x) --q;
    while ((int64_t)(q + 1) * (q + 2) / 2 <= x) ++q;
    const int k = x - (int)((int64_t)q * (q + 1) / 2);
    if (q > m || k >= m ) return;
    // each wave sixteen rows, half of the columns
    const int64_t i0 = (int64_t)(j + 2 + q) * CB + 16 * (w & 3), k0 = (int64_t)(j + 2 + k) * CB + 32 * (w >> 2);
    double a[16], b0[16], b1[16], c0[4], c1[4];
    chol_frag<16>(A + min(i0 + r, ld) * ld + jc + 4 * g, a);
    chol_frag<16>(A + (k0 + r) * ld + jc + 4 * g, b0);
    chol_frag<16>(A + (k0 + 16 + r) * ld + jc + 4 * g, b1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double* c = A + min(i0 + g + 4 * e, ld) * ld + k0 + r;
      c0[e] = c[0];
      c1[e] = c[16];
    }
    doublex4_t s0 = {0.0, 0.0, 0.0, 0.0}, s1 = s0;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], b0[kk], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], b1[kk], s1, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (i0 + g + 4 * e > ld) continue;
      double* c = A + (i0 + g + 4 * e) * ld + k0 + r;
      c[0] = c0[e] - s0[e];
      c[16] = c1[e] - s1[e];
    }
    return;
  }
  const int64_t d0 = jc + CB;                                  // first row and column of the diagonal block
  const int64_t i0 = (int64_t)(j + 2 + (int)blockIdx.x) * CB;  // first row of the own block
  // own block: column 4 g + e of tile ct of row r, so that a lane's entries are contiguous; the MFMA row
  // that gives it is m = 4 e + g, so operand row m holds column pi(m) = 4 (m % 4) + m / 4
  const int pi = 4 * (r & 3) + (r >> 2);
  const bool owner = w == 1 || w > 4;
  const int ow = w == 1 ? 3 : (w - 5) & 3;  // rows 16 ow .. of the own block
  const int64_t orow = min(i0 + 16 * ow + r, ld);
  const bool keep = orow == i0 + 16 * ow + r;  // not a copy of the right-hand side
  double* own = A + orow * ld + d0 + 4 * g;
  doublex4_t o[4];  // tiles from the current panel's on
  double ob[16];
  // every load is issued before the first is waited for
  const int rq = t >> 5, cq = 2 * (t & 31);  // rows rq + 12 i, columns cq, cq + 1
  if (owner) {
    if (j >= 0) chol_frag<16>(A + orow * ld + jc + 4 * g, ob);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const double2 u = *(const double2*)(own + 16 * ct), v = *(const double2*)(own + 16 * ct + 2);
      o[ct] = (doublex4_t){u.x, u.y, v.x, v.y};
    }
  }
  if (w < 4) {
    double2 dv[CB / 8], lv[CB / 8];
    const double* src = A + (d0 + rq) * ld + d0 + cq;
#pragma unroll
    for (int i = 0; i < CB / 8; ++i) dv[i] = *(const double2*)(src + (int64_t)8 * i * ld);
    if (j >= 0) {
#pragma unroll
      for (int i = 0; i < CB / 8; ++i) lv[i] = *(const double2*)(src + (int64_t)8 * i * ld - CB);
#pragma unroll
      for (int i = 0; i < CB / 8; ++i) *(double2*)&Ls[rq + 8 * i][cq] = lv[i];
    }
#pragma unroll
    for (int i = 0; i < CB / 8; ++i) *(double2*)&D[rq + 8 * i][cq] = dv[i];
  }
  __syncthreads();
  // D tile (ti, tk) -= NK columns from k0 on of rows ti and tk of X
  auto diag_tile = [&](auto nk, int ti, int tk, const double(*X)[CL], int k0) {
    constexpr int NK = decltype(nk)::value;
    double a[NK / 4], b[NK / 4], c[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = D[16 * ti + 4 * e + g][16 * tk + r];
    chol_frag<NK / 4>(&X[16 * ti + r][k0 + 4 * g], a);
    chol_frag<NK / 4>(&X[16 * tk + r][k0 + 4 * g], b);
    doublex4_t s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < NK / 4; ++kk) s = __builtin_amdgcn_mfma_f64_16x16x4f64(a[kk], b[kk], s, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) D[16 * ti + 4 * e + g][16 * tk + r] = c[e] - s[e];
  };
  constexpr std::integral_constant<int, CB> kBlock{};
  constexpr std::integral_constant<int, CP> kPanel{};
  // o[0] = tile p with column j's update
  auto own_update = [&](int p) {
    double a[16];
    chol_frag<16>(&Ls[16 * p + pi][4 * g], a);
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) o[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[kk], ob[kk], o[0], 0, 0, 0);
  };
  // o[0] = tile p: X_p^T = L_pp^-1 A_p^T, stored; then the tiles right of it move up, updated
  auto own_panel = [&](int p) {
    double v[4];
    chol_frag<4>(&V[p][pi][4 * g], v);
    doublex4_t xp = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) xp = __builtin_amdgcn_mfma_f64_16x16x4f64(v[kk], o[0][kk], xp, 0, 0, 0);
    if (keep) {
      *(double2*)(own + 16 * p) = make_double2(xp[0], xp[1]);
      *(double2*)(own + 16 * p + 2) = make_double2(xp[2], xp[3]);
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      o[u] = o[u + 1];
      if (p + 1 + u < 4) {
        double a[4];
        chol_frag<4>(&D[16 * (p + 1 + u) + pi][CP * p + 4 * g], a);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) o[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[kk], xp[kk], o[u], 0, 0, 0);
      }
    }
  };
  // step p: the tiles of column p, then panel p and, beside it, what nothing waits for yet
#pragma unroll 1
  for (int p = 0; p <= CB / CP; ++p) {
    if (p < CB / CP && w < CB / CP - p) {
      // column p's tiles lack column j (p = 0) or panel p - 1
      if (p > 0) diag_tile(kPanel, p + w, p, D, CP * (p - 1));
      else if (j >= 0) diag_tile(kBlock, w, 0, Ls, 0);
    }
    __syncthreads();
    if (w == 0 && p < CB / CP) {
      // lanes 16 q + r: row r of the identity (q = 0), of tile p + q
      double x[CP], y[CP];
      const int yr = min(CP * (p + g) + r, CB - 1);
#pragma unroll
      for (int c = 0; c < CP; c += 2) {
        const double2 u = *(const double2*)&D[CP * p + r][CP * p + c], v = *(const double2*)&D[yr][CP * p + c];
        x[c] = u.x;
        x[c + 1] = u.y;
        y[c] = g ? v.x : (r == c ? 1.0 : 0.0);
        y[c + 1] = g ? v.y : (r == c + 1 ? 1.0 : 0.0);
      }
      chol_columns<0>(x, y, chol_rsqrt(chol_row<0>(x[0])));  // NaN if the block is not positive definite
      if (g == 0) {
#pragma unroll
        for (int c = 0; c < CP; ++c) V[p][c][r] = y[c];
      }
      if (p + g < CB / CP) {
#pragma unroll
        for (int c = 0; c < CP; c += 2) {
          const bool tile = g == 0;
          *(double2*)&D[CP * (p + g) + r][CP * p + c] = make_double2(tile ? x[c] : y[c], tile ? x[c + 1] : y[c + 1]);
        }
      }
    } else if (owner) {
      if (p > 0) own_panel(p - 1);
      if (j >= 0 && p < CB / CP) own_update(p);
    } else if (w == 2 || w == 3) {
      // what the next column of tiles still lacks, wave 2: (1, 1), (3, 1); (2, 2); (3, 3), wave 3: (2, 1); (3, 2)
      for (int ti = p + w - 1; ti < 4; ti += 2) {
        if (j >= 0) diag_tile(kBlock, ti, p + 1, Ls, 0);
        for (int q = 0; q < p; ++q) diag_tile(kPanel, ti, p + 1, D, CP * q);
      }
    }
    __syncthreads();
  }
  if (j == 0 && t == 64 * CW - 1 && (int)blockIdx.x == npanel - 1) *chol_ticket(A) = 0;
  if (w < 4 && (int)blockIdx.x == npanel - 1) {
    // the diagonal block's factor goes to its own place: other workgroups may still be reading the block
    double* L = chol_diag(A, ld, nb, j + 1);
    for (int row = rq; row < CB; row += 8) {
      const double2 v = *(const double2*)&D[row][cq];
      *(double2*)(L + row * ld + cq) = make_double2(cq <= row ? v.x : 0.0, cq + 1 <= row ? v.y : 0.0);
    }
  }
}

// Back substitution: the x-th workgroup to start solves block i = nb - 1 - x of L^T y = w,
//   y_i = L_ii^-T (w_i - sum_{j > i} L_ji^T y_j),
// taking the later blocks' y_j as they appear in memory.  A workgroup draws its x when it runs, so it only waits for
// workgroups that run already or have ended: the waits end whatever the order in which workgroups are dispatched, and
// with other solves on other streams.  (By blockIdx, two solves could each hold one XCD's slots with workgroups that wait
// for ones the other keeps out of another XCD.)  A wait is bounded all the same: after kSpin polls, seconds, the
// workgroup goes on with NaN, and y is NaN from there on, as for a matrix that is not positive definite.  An entry of y
// is published by one 8-byte store over the kUnknown that chol_init_kernel left, so no flag or fence is needed.  The chain
// per block is one such hand-over and two 64 x 64 matrix-vector products: the inverse of L_ii is
// formed before the first wait and the next L_ji is loaded before its y_j is awaited.
constexpr int kSpin = 1 << 22;
__device__ inline void chol_publish(unsigned long long* y, float* out, int64_t at, int64_t B, double v) {
  unsigned long long u = (unsigned long long)__double_as_longlong(v);
  if (u == kUnknown) u ^= 1ull;  // a NaN all the same
  __hip_atomic_store(y + at, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (at < B) out[at] = (float)v;
}

__global__ __launch_bounds__(256) void chol_back_kernel(double* __restrict__ A, int64_t ld, int nb, unsigned long long* y,
                                                        int64_t B, float* __restrict__ out) {
  __shared__ __align__(16) double L[CB][CL];
  __shared__ __align__(16) double X[CB][CL];  // L_ii^-1
  __shared__ double part[4][CB];
  __shared__ double v[CB];
  __shared__ int ticket;
  const int t = threadIdx.x, c = t & 63, q = t >> 6;
  if (t == 0) ticket = nb > 1 ? __hip_atomic_fetch_add(chol_ticket(A), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  __syncthreads();
  const int i = nb - 1 - __builtin_amdgcn_readfirstlane(ticket);
  const int64_t i0 = (int64_t)i * CB;
  const double* Ld = chol_diag(A, ld, nb, i);
  for (int e = t; e < CB * CB; e += 256) L[e >> 6][e & 63] = Ld[(e >> 6) * ld + (e & 63)];
  __syncthreads();
  if (i == nb - 1) {
    // nothing to wait for: substitution by one wave, lane c column c, instead of the inverse (B = 64: the kernel 5 us
    // instead of 37)
    if (q == 0) {
      double acc = A[ld * ld + i0 + c], yc = 0.0;
      const double rd = 1.0 / L[c][c];
#pragma unroll 8
      for (int r = CB - 1; r >= 0; --r) {
        const double yr = chol_bcast(acc * rd, r);
        if (c == r) yc = yr;
        acc = fma(-L[r][c], yr, acc);  // (lanes past r: not used any more)
      }
      chol_publish(y, out, i0 + c, B, yc);
    }
    return;
  }
  // column c of the inverse, row after row: X[rr] = (e_rr - sum_{k < rr} L[rr][k] X[k]) / L[rr][rr],
  // the sum shared by four threads
  for (int rr = 0; rr < CB; ++rr) {
    double s = 0.0;
    for (int k = q; k < rr; k += 4) s = fma(L[rr][k], X[k][c], s);
    part[q][c] = s;
    __syncthreads();
    if (q == 0) X[rr][c] = ((rr == c ? 1.0 : 0.0) - ((part[0][c] + part[1][c]) + (part[2][c] + part[3][c]))) / L[rr][rr];
    __syncthreads();
  }
  // thread (c, q): rows 16 q .. 16 q + 15 of column c of each L_ji
  double sum = 0.0, l[16];
  auto fetch = [&](int jj) {
    const double* p = A + ((int64_t)jj * CB + 16 * q) * ld + i0 + c;
#pragma unroll
    for (int e = 0; e < 16; ++e) l[e] = p[(int64_t)e * ld];
  };
  if (nb - 1 > i) fetch(nb - 1);
  int spin = kSpin;
  for (int jj = nb - 1; jj > i; --jj) {
    unsigned long long* src = y + (int64_t)jj * CB + 16 * q + (c & 15);
    unsigned long long u = kUnknown;
    int n = 0;
    for (; n < spin; ++n) {
      u = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__ballot(u == kUnknown) == 0) break;
    }
    if (n == spin) spin = 1;  // the result is lost: no second wait
    const double yv = __longlong_as_double((long long)u);
#pragma unroll
    for (int e = 0; e < 16; ++e) sum = fma(l[e], chol_bcast(yv, e), sum);
    if (jj - 1 > i) fetch(jj - 1);
  }
  part[q][c] = sum;
  __syncthreads();
  if (q == 0) v[c] = A[ld * ld + i0 + c] - ((part[0][c] + part[1][c]) + (part[2][c] + part[3][c]));
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < 16; ++e) s = fma(X[16 * q + e][c], v[16 * q + e], s);  // X[rr][c] = 0 for rr < c
  part[q][c] = s;
  __syncthreads();
  if (q == 0) {
    chol_publish(y, out, i0 + c, B, (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]));
  }
}

// the matrix, the right-hand side as its last row, y
size_t sr_solve_ws_bytes(int64_t B) {
  const int64_t ld = round_up(B, CB);
  return (size_t)round_up(ld * ld * 8, 256) + 2 * (size_t)round_up(ld * 8, 256);
}

hipError_t launch_sr_solve(const float* K, int64_t B, double shift, const float* rhs, double scale, float* y,
                           void* ws, hipStream_t st) {
  const int64_t ld = round_up(B, CB);
  const int nb = (int)(ld / CB);
  double* A = (double*)ws;
  unsigned long long* yd = (unsigned long long*)(A + ld * (ld + 1));
  chol_init_kernel<<<(unsigned)((ld * (ld + 1) + 255) / 256), 256, 0, st>>>(K, B, ld, shift, rhs, scale, A, yd);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  for (int j = -1; j < nb - 1; ++j) {
    // m columns right of j + 1 with their rows down to the right-hand side; none before the first column
    const int64_t m = nb - j - 2, rest = j < 0 ? 0 : m * (m + 1) / 2 + m;
    chol_step_kernel<<<(unsigned)(nb - j - 1 + rest), 64 * CW, 0, st>>>(A, ld, nb, j);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  chol_back_kernel<<<(unsigned)nb, 256, 0, st>>>(A, ld, nb, yd, B, y);
  return hipGetLastError();
}

}  // namespace vqmc
