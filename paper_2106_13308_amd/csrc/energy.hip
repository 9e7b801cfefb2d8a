// Diagonal local energy and batch statistics.
//
// Local energy (Sec. 2.1): l(x) = (H psi)(x) / psi(x), which for a diagonal H
// (alpha_i = 0 in eq. hamiltonian) is H_xx = sum_{i<j} J_ij s_i s_j with beta_i = 0.
// Statistics (Sec. 2.1, eq. stochastic_variance and the gradient population form):
// mean, population variance, min/argmin and baseline coefficients c_b = (E_b - mean)/B.
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <type_traits>

namespace vqmc {

// ---------------------------------------------------------------- sparse (CSR upper)
// One workgroup of 1024 threads handles EMSE samples.  Their spins are staged in LDS as
// one byte per site (bit q = [s_q = +1]), so an edge costs one byte read for all samples,
// and so is the row pointer (int32) when it fits.  A group of `lanes` threads walks rows i, i + groups, ..., each
// its share of a row's edges, two per step with their loads issued together.  Row i of the upper triangle
// contributes (each lane the sums over its share)
//   s_iq sum_j w_ij s_jq = s_iq (2 Y_q - W_i),  Y_q = sum_j w_ij [s_jq = +1],  W_i = sum_j w_ij,
// accumulated exactly in int64 (integer weights) or in double (float weights, whose sums
// of exact terms only differ from the oracle's by summation order).  A fixed thread -> row
// map and fixed-shape reductions make the result deterministic.
// SHARED: several lanes a row; without it the row loop is that of one lane.  WAVES = 8: 64 registers, so that two workgroups
// share a CU (float weights, degree 20, n = 3000, B = 16384: 152 against 219 us with 66; mean row 3, n = 1000: 43 against 66).
// Shared float rows spill two registers so; with no more workgroups than CUs they take WAVES = 4 (n = 1973, 25 % of the edges,
// B = 271, with the sampler: 310 against 316 us).
constexpr int EMSE = 8;
constexpr int EB_THREADS = 1024;
template <typename WT, typename AT, bool RP_LDS, bool SHARED, int WAVES = 8>
__global__ __launch_bounds__(EB_THREADS, WAVES) void energy_csr_bits_kernel(int n, int64_t lds,
                                                                    const int64_t* __restrict__ rowptr,
                                                                    const int32_t* __restrict__ col,
                                                                    const WT* __restrict__ w,
                                                                    const int8_t* __restrict__ S, int64_t B,
                                                                    int nst, int row_lanes, AT* __restrict__ E) {
  const int lanes = SHARED ? row_lanes : 1;
  // nst bytes of site bits, then the row pointer (n + 1 int32, if staged), then scratch
  extern __shared__ __attribute__((aligned(16))) uint8_t shb[];
  uint8_t* bits = shb;
  int32_t* rp = (int32_t*)(shb + nst);
  AT* red = (AT*)(shb + nst + (RP_LDS ? round_up((int64_t)(n + 1) * 4, 16) : 0));
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t b0 = (int64_t)blockIdx.x * EMSE;
  const int nq = (int)min<int64_t>(EMSE, B - b0);
  // nst = round_up(n, 16) <= lds: every 16-byte chunk lies inside the padded row.  The
  // spins are +1 = 0x01 and -1 = 0xFF: bit 7 of a byte is clear exactly for +1 (the row
  // padding, 0, also reads +1 and is never referenced).
  for (int c0 = t; c0 < nst / 16; c0 += EB_THREADS) {
    uint32_t a[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < EMSE; ++q) {
      if (q < nq) {
        const uint4 v = *(const uint4*)(S + (b0 + q) * lds + 16 * c0);
        a[0] |= ((~v.x >> 7) & 0x01010101u) << q;
        a[1] |= ((~v.y >> 7) & 0x01010101u) << q;
        a[2] |= ((~v.z >> 7) & 0x01010101u) << q;
        a[3] |= ((~v.w >> 7) & 0x01010101u) << q;
      }
    }
    *(uint4*)(bits + 16 * c0) = make_uint4(a[0], a[1], a[2], a[3]);
  }
  if constexpr (RP_LDS)
    for (int i = t; i <= n; i += EB_THREADS) rp[i] = (int32_t)rowptr[i];
  __syncthreads();
  auto rowp = [&](int i) -> int64_t {
    if constexpr (RP_LDS) return rp[i];
    else return rowptr[i];
  };
  AT acc[EMSE];
#pragma unroll
  for (int q = 0; q < EMSE; ++q) acc[q] = 0;
  // row sums Y: int32 for integer weights while the row's sum of |w| fits (then no partial
  // sum can overflow; a row beyond that is summed again in int64), else AT
  constexpr bool INT = std::is_integral<WT>::value;
  typedef typename std::conditional<INT, int32_t, AT>::type RT;
  const int groups = EB_THREADS / lanes, sub = t & (lanes - 1);
  for (int i = t / lanes; i < n; i += groups) {
    const int64_t e0 = rowp(i) + sub, e1 = rowp(i + 1);  // the lane's edges: e0, e0 + lanes, ..
    RT y[EMSE];
#pragma unroll
    for (int q = 0; q < EMSE; ++q) y[q] = 0;
    AT wsum = 0;
    int64_t wabs = 0;
    int64_t e = e0;
    for (; e + lanes < e1; e += 2 * lanes) {  // two edges per step: their loads are issued together
      const int j0 = col[e], j1 = col[e + lanes];
      const RT w0 = (RT)w[e], w1 = (RT)w[e + lanes];
      const uint32_t m0 = bits[j0], m1 = bits[j1];
      wsum += (AT)w0 + (AT)w1;
      if constexpr (INT) wabs += llabs((int64_t)w0) + llabs((int64_t)w1);
#pragma unroll
      for (int q = 0; q < EMSE; ++q) y[q] += (((m0 >> q) & 1u) ? w0 : (RT)0) + (((m1 >> q) & 1u) ? w1 : (RT)0);
    }
    if (e < e1) {
      const RT w0 = (RT)w[e];
      const uint32_t m0 = bits[col[e]];
      wsum += (AT)w0;
      if constexpr (INT) wabs += llabs((int64_t)w0);
#pragma unroll
      for (int q = 0; q < EMSE; ++q) y[q] += ((m0 >> q) & 1u) ? w0 : (RT)0;
    }
    AT ya[EMSE];
#pragma unroll
    for (int q = 0; q < EMSE; ++q) ya[q] = (AT)y[q];
    if (INT && wabs > (int64_t)INT32_MAX) {
#pragma unroll
      for (int q = 0; q < EMSE; ++q) ya[q] = 0;
      for (int64_t f = e0; f < e1; f += lanes) {
        const AT wf = (AT)w[f];
        const uint32_t mf = bits[col[f]];
#pragma unroll
        for (int q = 0; q < EMSE; ++q) ya[q] += ((mf >> q) & 1u) ? wf : (AT)0;
      }
    }
    const uint32_t mi = bits[i];
#pragma unroll
    for (int q = 0; q < EMSE; ++q) {
      const AT r = 2 * ya[q] - wsum;
      acc[q] += ((mi >> q) & 1u) ? r : -r;
    }
  }
  // per sample: fixed butterfly over the wave, then the sixteen waves in order
  constexpr int NW = EB_THREADS / 64;
#pragma unroll
  for (int q = 0; q < EMSE; ++q) {
    AT v = acc[q];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) red[q * NW + wv] = v;
  }
  __syncthreads();
  if (t < nq) {
    AT s = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += red[t * NW + k];
    E[b0 + t] = s;
  }
}

// ---------------------------------------------------------------- sparse, byte lanes
// Integer weights, each site staged as eight bytes (byte q = 0xFF where s_q = +1, else 0) instead of
// eight bits.  An edge adds w s_i s_j = w - 2 w [s_i != s_j], so
//   E_q = W - 2 Y_q,   Y_q = sum_edges w [s_iq != s_jq],   W = sum_edges w,
// and (w in every byte) & (site i ^ site j) holds w or 0 for all eight samples, to be added byte by byte.
// No edge needs its row's sum, so L lanes share a row with nothing to add up between
// them (L from the mean row length: a lane gets 8 to 16 edges of a row, or one lane a whole row), and the
// bytes run on across rows; they are added to 64-bit sums before the weights in them exceed 255.
// A step of a lane (sixteen edges) whose weights do not fit so - negative ones, or a sum above 255 - adds its edges to
// those sums directly, a 64-bit multiply-add by 0 or 1 per sample (selects and adds with carry took five instructions:
// weights +-1 at n = 10000, degree 10, B = 2048 52 us, 32 so, 58 by a thread per row; one vertex with 9999 edges of
// large weights 5.9 ms, 2.3 so and 2.3 by a thread).
//
// What bounds it: the address coalescing of the rows' loads (16 cycles a load instruction when the lanes lie
// apart), then their latency.  So a lane takes four edges by one 16-byte load of each array, and
// EC_RB = 4 (or 2) rows at a time with their loads issued together.  Measured (us; before: a thread per row, two
// edges a step, 64-bit sums per row): n = 500, 75 % of the edges, B = 1024: 35 -> 18; n = 10000, degree 10, B = 2048:
// 41 -> 30.
constexpr int EC_U = 4;
template <bool RP_LDS, int EC_RB>
__global__ __launch_bounds__(EB_THREADS, EC_RB == 2 ? 8 : 4) void energy_csr_bytes_kernel(int n, int64_t lds,
                                                                     const int64_t* __restrict__ rowptr,
                                                                     const int32_t* __restrict__ col,
                                                                     const int32_t* __restrict__ w, int64_t nnz,
                                                                     const int8_t* __restrict__ S, int64_t B,
                                                                     int nsp, int lanes, int64_t* __restrict__ E) {
  // nsp uint2 site words (n rounded up to 16), then the row pointer (n + 1 int32, if staged),
  // then scratch
  extern __shared__ __attribute__((aligned(16))) uint8_t shb[];
  uint2* sw = (uint2*)shb;
  int32_t* rp = (int32_t*)(shb + (size_t)nsp * 8);
  int64_t* red = (int64_t*)(shb + (size_t)nsp * 8 + (RP_LDS ? round_up((int64_t)(n + 1) * 4, 16) : 0));
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t b0 = (int64_t)blockIdx.x * EMSE;
  const int nq = (int)min<int64_t>(EMSE, B - b0);
  // four sites per item (of sixteen, the lanes' stores would all meet in one LDS bank): a word of
  // each sample's row, gathered into a bit per sample, then spread to a byte per sample
  for (int c0 = t; c0 < nsp / 4; c0 += EB_THREADS) {
    uint32_t a = 0u;
#pragma unroll
    for (int q = 0; q < EMSE; ++q)
      if (q < nq) a |= ((~*(const uint32_t*)(S + (b0 + q) * lds + 4 * c0) >> 7) & 0x01010101u) << q;
    uint32_t x[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t m = (a >> (8 * e)) & 0xFFu;
      // bit k of a 4-bit value to bit 8k: the four shifted copies (x 1, 2^7, 2^14, 2^21) do not
      // overlap, so the product carries nothing; then the bit to the whole byte
      x[2 * e] = (((m & 0xFu) * 0x00204081u) & 0x01010101u) * 0xFFu;
      x[2 * e + 1] = (((m >> 4) * 0x00204081u) & 0x01010101u) * 0xFFu;
    }
    *(uint4*)(sw + 4 * c0) = make_uint4(x[0], x[1], x[2], x[3]);
    *(uint4*)(sw + 4 * c0 + 2) = make_uint4(x[4], x[5], x[6], x[7]);
  }
  if constexpr (RP_LDS)
    for (int i = t; i <= n; i += EB_THREADS) rp[i] = (int32_t)rowptr[i];
  __syncthreads();
  auto rowp = [&](int i) -> uint32_t {  // nnz < 2^31
    if constexpr (RP_LDS) return (uint32_t)rp[i];
    else return (uint32_t)rowptr[i];
  };
  int64_t y[EMSE], wsum = 0;
#pragma unroll
  for (int q = 0; q < EMSE; ++q) y[q] = 0;
  uint32_t ylo = 0u, yhi = 0u, held = 0u;  // Y_q in byte q (q < 4 in ylo), and the weights in them
  auto flush = [&]() {
#pragma unroll
    for (int q = 0; q < EMSE; ++q) y[q] += ((q < 4 ? ylo : yhi) >> (8 * (q & 3))) & 0xFFu;
    ylo = yhi = held = 0u;
  };
  const int groups = EB_THREADS / lanes, sub = t & (lanes - 1);
  const __amdgpu_buffer_rsrc_t rcol = __builtin_amdgcn_make_buffer_rsrc((void*)col, 0, (int)(uint32_t)(4 * nnz), 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, (int)(uint32_t)(4 * nnz), 0x00020000);
  const uint32_t last = (uint32_t)nnz - EC_U;  // nnz >= EC_U: the last place for a load
  for (int i0 = t / lanes; i0 < n; i0 += EC_RB * groups) {
    uint32_t e[EC_RB], e1[EC_RB];
    int left = 0;
    uint2 si[EC_RB];
#pragma unroll
    for (int r = 0; r < EC_RB; ++r) {
      const int i = i0 + r * groups, ic = min(i, n - 1);
      e[r] = rowp(ic) + EC_U * sub;
      e1[r] = i < n ? rowp(ic + 1) : e[r];
      si[r] = sw[ic];
      left = max(left, (int)(e1[r] - e[r]));
    }
    for (; left > 0; left -= EC_U * lanes) {
      uint32_t j[EC_RB][EC_U], wt[EC_RB][EC_U];
#pragma unroll
      for (int r = 0; r < EC_RB; ++r) {
        const int at = (int)(min(e[r], last) * 4u);
        const uint4 c4 = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rcol, at, 0, 0));
        const uint4 w4 = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, at, 0, 0));
        j[r][0] = c4.x; j[r][1] = c4.y; j[r][2] = c4.z; j[r][3] = c4.w;
        wt[r][0] = w4.x; wt[r][1] = w4.y; wt[r][2] = w4.z; wt[r][3] = w4.w;
      }
      uint32_t all = 0u, sum = 0u;
#pragma unroll
      for (int r = 0; r < EC_RB; ++r) {
        // the edges e .. e1 - 1 among those loaded
        const uint32_t off = min(e[r], last) - e[r], len = (int)(e1[r] - e[r]) > 0 ? e1[r] - e[r] : 0u;
#pragma unroll
        for (int u = 0; u < EC_U; ++u) {
          wt[r][u] = off + u < len ? wt[r][u] : 0u;
          all |= wt[r][u];
          sum += wt[r][u];
        }
      }
      if (all <= 255u && sum <= 255u) {
        if (held + sum > 255u) flush();
        held += sum;
        wsum += sum;
#pragma unroll
        for (int r = 0; r < EC_RB; ++r)
#pragma unroll
          for (int u = 0; u < EC_U; ++u) {
            const uint2 sj = sw[j[r][u]];
            const uint32_t w4 = __builtin_amdgcn_perm(0u, wt[r][u], 0u);  // byte 0 in all four
            ylo += w4 & (si[r].x ^ sj.x);
            yhi += w4 & (si[r].y ^ sj.y);
          }
      } else {
#pragma unroll
        for (int r = 0; r < EC_RB; ++r)
#pragma unroll
          for (int u = 0; u < EC_U; ++u) {
            if (wt[r][u] == 0u) continue;
            const uint2 sj = sw[j[r][u]];
            const uint32_t dx = si[r].x ^ sj.x, dy = si[r].y ^ sj.y;
            const int64_t we = (int32_t)wt[r][u];
            wsum += we;
#pragma unroll
            for (int q = 0; q < EMSE; ++q) y[q] += we * (int32_t)(((q < 4 ? dx : dy) >> (8 * (q & 3))) & 1u);  // one multiply-add
          }
      }
#pragma unroll
      for (int r = 0; r < EC_RB; ++r) e[r] += EC_U * lanes;
    }
  }
  flush();
  // E_q of the lane, then the sums over the wave: three exchanges that halve the samples a lane holds,
  // three over the eight lanes with the same sample, then the sixteen waves in order
#pragma unroll
  for (int q = 0; q < EMSE; ++q) y[q] = wsum - 2 * y[q];
#pragma unroll
  for (int k = 4; k > 0; k >>= 1) {
    const bool up = lane & (8 * k);
#pragma unroll
    for (int q = 0; q < k; ++q) {
      const int64_t mine = up ? y[q + k] : y[q], theirs = up ? y[q] : y[q + k];
      y[q] = mine + __shfl_xor(theirs, 8 * k);
    }
  }
  int64_t v = y[0];
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) v += __shfl_xor(v, o);
  constexpr int NW = EB_THREADS / 64;
  if ((lane & 7) == 0) red[(lane >> 3) * NW + wv] = v;  // sample 4 [lane & 32] + 2 [lane & 16] + [lane & 8]
  __syncthreads();
  if (t < nq) {
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += red[t * NW + k];
    E[b0 + t] = s;
  }
}

// ---------------------------------------------------------------- dense J
// E_b = sum_i s_bi y_bi with y_bi = sum_{j>i} J_ij s_bj (strict upper triangle only).
//
// The spins are integers, so y is a contraction of integers once row i of J is written in fixed
// point: with 2^e_i above the row's largest entry, J_ij = 2^(e_i - 54) q_ij and |q_ij| < 2^54.  A row is taken this
// way if that is exact for every entry: no bit of a non-zero entry below 2^(e_i - 54) (so any row whose entries lie
// within 2^30 of each other).  q is split into seven signed bytes, each plane is
// multiplied with the spins on the int8 matrix cores (exact 32-bit sums: 128 n < 2^31), and the
// seven sums of a row are joined by six double-precision multiply-adds, the only roundings.  A tile with a row of
// another kind (entries further apart, NaN, infinities) is summed by the FP64 matrix cores, every entry a double.
//
// Tile: 16 IB rows x 32 samples per wave, NW waves with the same rows, 64 columns of J per step.  The
// workgroup turns each step's FP32 entries into byte planes in LDS itself (13 instructions an entry
// plus the byte transposes, shared by its 32 NW samples) - a separate pass over J would write and
// read 7 n^2 bytes; the spins are matrix operands as they lie in memory.  Lane group g takes the bytes
// 16 g .. 16 g + 15 of either operand's 64.
//
// A step's products run beside the conversion of the next step, one barrier per step.
//
// n = 2000, B = 8192: 154 us, of which 12 for the exponents and the sum of the tiles' partials (the products run at
// 1.45 POPS of the 4.6 that a loop of them reaches); n = 1000, B = 512: 24 us.  Copies without the conversion take
// 133 us, without the spin loads 150, with 12 of the 28 products of a step 106: what is left is each workgroup's start
// and end, one workgroup per CU.  With every row in FP64, as before, 1188 us and 65; through this kernel's FP64 tiles,
// a matrix of such rows alone, 1155 and 50.  Against 64-bit sums of the N(0, 1/n) couplings the energies are off by
// 1.3e-16 of their norm, as before.
constexpr int DK = 64;  // columns of J per step
constexpr int DD = 7;            // byte planes
constexpr int DWIDE = INT32_MIN;
struct __attribute__((aligned(8))) Bytes16 {  // spin rows may start on any 8-byte boundary
  uint32_t x[4];
};
typedef __attribute__((ext_vector_type(4))) int32_t i32x4_t;

// ex[i] = e with |J_ij| < 2^e for every j > i, DWIDE if 2^(e - 54) does not divide every entry of the row or it has a
// NaN or infinity; a wave a row.
__global__ __launch_bounds__(256) void energy_rowmax_kernel(int n, const float* __restrict__ J, int32_t* __restrict__ ex) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  const float* row = J + (int64_t)i * n;
  uint32_t m = 0;
  int low = INT32_MAX;  // the lowest bit set in an entry, as the exponent field of 2^23 times it
  auto take = [&](uint32_t v) {
    m = max(m, v);
    const uint32_t f = v >> 23, sig = (v & 0x7FFFFFu) | (f ? 0x800000u : 0u);
    if (sig) low = min(low, (int)max(f, 1u) + __builtin_ctz(sig));
  };
  int j = i + 1 + lane;
  for (; j + 192 < n; j += 256) {
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __float_as_uint(row[j + 64 * u]) & 0x7FFFFFFFu;
#pragma unroll
    for (int u = 0; u < 4; ++u) take(v[u]);
  }
  for (; j < n; j += 64) take(__float_as_uint(row[j]) & 0x7FFFFFFFu);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    m = max(m, (uint32_t)__shfl_xor((int)m, o));
    low = min(low, __shfl_xor(low, o));
  }
  const int f = max((int)(m >> 23), 1);
  // e = f - 126; a bit of exponent field low weighs 2^(low - 150)
  if (lane == 0) ex[i] = m >= 0x7F800000u || low < f - 30 ? DWIDE : f - 126;
}

// q of one entry as eight bytes, the low seven of them the signed digits
__device__ inline uint2 fixed_digits(float v, int e) {
  const float x = ldexpf(v, 23 - e);      // |x| < 2^23
  const int32_t hi = (int32_t)x;
  const float r = x - (float)hi;          // exact
  const int64_t lo = (int32_t)rintf(r * 2147483648.f);
  // 128 added to every digit turns the balanced digits into the plain bytes of the sum
  constexpr uint64_t bias = 0x0080808080808080ull;
  const uint64_t q = ((uint64_t)((int64_t)hi * 2147483648ll) + (uint64_t)lo + bias) ^ bias;
  return make_uint2((uint32_t)q, (uint32_t)(q >> 32));
}

// Sums over 16 IB rows from i0 and the wave's 32 samples (rows srow of S, clamped) by v_mfma_f64_16x16x4, the columns
// in rising order: y[ib][sb][e] belongs to row i0 + 16 ib + 4 e + lane / 16 and sample 16 sb + lane % 16.  Operands
// straight from memory, the next sixteen columns' loads in flight: a product takes 64 cycles, so the matrix
// cores bound it (a tile's J entries serve 32 samples a load).
template <int IB>
__device__ inline void dense_rows_f64(int n, const float* __restrict__ J, int i0, const int8_t* const (&srow)[2],
                                      doublex4_t (&y)[IB][2]) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int ib = 0; ib < IB; ++ib)
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) y[ib][sb] = (doublex4_t){0.0, 0.0, 0.0, 0.0};
  float jv[2][IB][4];
  uint4 sv[2][2];
  auto fetch = [&](int j0, const int q) {
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      const float* row = J + (int64_t)min(i0 + 16 * ib + r, n - 1) * n;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) jv[q][ib][kk] = row[min(j0 + 4 * kk + g, n - 1)];
    }
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) sv[q][sb] = *(const uint4*)(srow[sb] + j0);
  };
  const int jlast = (n - 1) / 16 * 16;  // past the end: the last columns' loads again, never used
  auto step = [&](int j0, const int q) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int j = j0 + 4 * kk + g;
      double a[IB], s[2];
#pragma unroll
      for (int ib = 0; ib < IB; ++ib) {
        const int i = i0 + 16 * ib + r;
        a[ib] = i < n && j < n && j > i ? (double)jv[q][ib][kk] : 0.0;
      }
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const uint32_t w = kk == 0 ? sv[q][sb].x : kk == 1 ? sv[q][sb].y : kk == 2 ? sv[q][sb].z : sv[q][sb].w;
        s[sb] = j < n ? (double)(int8_t)(w >> (8 * g)) : 0.0;
      }
#pragma unroll
      for (int ib = 0; ib < IB; ++ib)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) y[ib][sb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ib], s[sb], y[ib][sb], 0, 0, 0);
    }
  };
  int j0 = i0 / 16 * 16;
  fetch(j0, 0);
  for (; j0 < n; j0 += 32) {
    fetch(min(j0 + 16, jlast), 1);
    step(j0, 0);
    fetch(min(j0 + 32, jlast), 0);
    if (j0 + 16 < n) step(j0 + 16, 1);
  }
}

// sum_i s_bi y_bi of dense_rows_f64's rows, stored by the lanes of the first group
template <int IB>
__device__ inline void dense_store_f64(int n, int i0, const int8_t* const (&srow)[2], const doublex4_t (&y)[IB][2],
                                       int64_t b0, int64_t B, double* __restrict__ part) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int sb = 0; sb < 2; ++sb) {
    double v = 0.0;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + 16 * ib + 4 * e + g;
        if (i < n) v += (double)srow[sb][i] * y[ib][sb][e];
      }
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    const int64_t b = b0 + 16 * sb + r;
    if (g == 0 && b < B) part[b] = v;
  }
}

// Every row in FP64: for couplings so few that the pass for the exponents costs more than the products
template <int NW>
__global__ __launch_bounds__(64 * NW) void energy_dense_f64_kernel(int n, int64_t lds, const float* __restrict__ J,
                                                                   const int8_t* __restrict__ S, int64_t B,
                                                                   double* __restrict__ part) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, i0 = blockIdx.y * 16;
  const int64_t b0 = (int64_t)blockIdx.x * (32 * NW) + 32 * wv;
  const int8_t* srow[2];
#pragma unroll
  for (int sb = 0; sb < 2; ++sb) srow[sb] = S + min(b0 + 16 * sb + (lane & 15), B - 1) * lds;
  doublex4_t y[1][2];
  dense_rows_f64<1>(n, J, i0, srow, y);
  dense_store_f64<1>(n, i0, srow, y, b0, B, part + (int64_t)blockIdx.y * B);
}

// VEC: rows of J start 16-byte aligned (n a multiple of four and J 16-byte aligned)
template <int NW, int IB, bool VEC>
__global__ __launch_bounds__(64 * NW, 2) void energy_dense_kernel(int n, int64_t lds, const float* __restrict__ J,
                                                               const int32_t* __restrict__ ex,
                                                               const int8_t* __restrict__ S, int64_t B,
                                                               double* __restrict__ part) {
  constexpr int DT = 16 * IB;                  // rows of the tile
  constexpr int NQ = DT * DK / 4 / (64 * NW);  // quads of columns converted per thread and step
  __shared__ __align__(16) uint8_t planes[2][DD][DT * DK];
  __shared__ int32_t se[DT];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, r = lane & 15, g = lane >> 4;
  const int i0 = blockIdx.y * DT;
  const int64_t b0 = (int64_t)blockIdx.x * (32 * NW) + 32 * wv;
  if (t < DT) se[t] = (i0 + t < n) ? ex[i0 + t] : 0;
  __syncthreads();
  bool wide = false;
#pragma unroll
  for (int q = 0; q < DT; ++q) wide |= se[q] == DWIDE;
  // spins of samples b0 + 16 sb + r (clamped: results past B are never stored); the row padding meets
  // zero digits
  const int8_t* srow[2];
#pragma unroll
  for (int sb = 0; sb < 2; ++sb) srow[sb] = S + min(b0 + 16 * sb + r, B - 1) * lds;
  if (__builtin_amdgcn_readfirstlane(wide)) {
    doublex4_t y[IB][2];
    dense_rows_f64<IB>(n, J, i0, srow, y);
    dense_store_f64<IB>(n, i0, srow, y, b0, B, part + (int64_t)blockIdx.y * B);
    return;
  }
  // quad u of the thread: row tr + (4 NW) u, columns 4 tq .. 4 tq + 3 of the step.  Addresses are
  // clamped into the matrix and entries masked when they are converted, so that a load has a step
  // or two to arrive.
  const int tr = t >> 4, tq = t & 15;
  float jr[2][NQ][4];
  auto fetch_j = [&](int j0, float(&jv)[NQ][4]) {
    const int j = j0 + 4 * tq;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const float* row = J + (int64_t)min(i0 + tr + 4 * NW * u, n - 1) * n;
      if constexpr (VEC) {
        const float4 a = *(const float4*)(row + min(j, n - 4));
        jv[u][0] = a.x; jv[u][1] = a.y; jv[u][2] = a.z; jv[u][3] = a.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) jv[u][e] = row[min(j + e, n - 1)];
      }
    }
  };
  i32x4_t sr[2][2];
  auto fetch_s = [&](int j0, i32x4_t(&v)[2]) {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) v[sb] = __builtin_bit_cast(i32x4_t, *(const Bytes16*)(srow[sb] + j0 + 16 * g));
  };
  i32x4_t acc[DD][IB][2];  // plane, 16-row block, 16-sample block; entry e: row 4 g + e, sample r
#pragma unroll
  for (int p = 0; p < DD; ++p)
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) acc[p][ib][sb] = (i32x4_t){0, 0, 0, 0};
  const int jbeg = i0 / DK * DK;
  const int jlast = (n - 1) / DK * DK;  // past the end: the last step's loads again, never used
  // the step at j0 from registers into the byte planes
  auto convert = [&](int j0, const float(&jv)[NQ][4], uint8_t (*dstp)[DT * DK]) {
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const int row = tr + 4 * NW * u, i = i0 + row, j = j0 + 4 * tq;
      const int e = se[row];
      uint2 d[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t keep = 0u - (uint32_t)((i < n) & (j + c < n) & (j + c > i));  // no branch around a load's first use
        d[c] = fixed_digits(__uint_as_float(__float_as_uint(jv[u][c]) & keep), e);
      }
      // byte p of the four entries, together
      uint8_t* dst = dstp[0] + row * DK + 4 * tq;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const uint32_t a0 = half ? d[0].y : d[0].x, a1 = half ? d[1].y : d[1].x, a2 = half ? d[2].y : d[2].x,
                       a3 = half ? d[3].y : d[3].x;
        const uint32_t l01 = __builtin_amdgcn_perm(a1, a0, 0x05010400u), l23 = __builtin_amdgcn_perm(a3, a2, 0x05010400u);
        const uint32_t h01 = __builtin_amdgcn_perm(a1, a0, 0x07030602u), h23 = __builtin_amdgcn_perm(a3, a2, 0x07030602u);
        const uint32_t w[4] = {__builtin_amdgcn_perm(l23, l01, 0x05040100u), __builtin_amdgcn_perm(l23, l01, 0x07060302u),
                               __builtin_amdgcn_perm(h23, h01, 0x05040100u), __builtin_amdgcn_perm(h23, h01, 0x07060302u)};
#pragma unroll
        for (int p = 0; p < 4; ++p)
          if (4 * half + p < DD) *(uint32_t*)(dst + (4 * half + p) * (DT * DK)) = w[p];
      }
    }
  };
  // step j0: its products beside the conversion of the next step
  auto step = [&](int j0, const int q) {
    lds_barrier();
    i32x4_t a[IB][DD];
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int p = 0; p < DD; ++p) a[ib][p] = *(const i32x4_t*)(planes[q][p] + (16 * ib + r) * DK + 16 * g);
    fetch_s(min(j0 + DK, jlast), sr[q ^ 1]);
    convert(j0 + DK, jr[q ^ 1], planes[q ^ 1]);
    fetch_j(min(j0 + 3 * DK, jlast), jr[q ^ 1]);
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int p = 0; p < DD; ++p)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
          acc[p][ib][sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[ib][p], sr[q][sb], acc[p][ib][sb], 0, 0, 0);
  };
  fetch_j(jbeg, jr[0]);
  fetch_s(jbeg, sr[0]);
  convert(jbeg, jr[0], planes[0]);
  fetch_j(min(jbeg + DK, jlast), jr[1]);
  fetch_j(min(jbeg + 2 * DK, jlast), jr[0]);
  int j0 = jbeg;
  for (; j0 + DK < n; j0 += 2 * DK) {
    step(j0, 0);
    step(j0 + DK, 1);
  }
  if (j0 < n) step(j0, 0);
  // sum_i s_bi y_bi over the tile's rows: a lane's eight, then the four lane groups
#pragma unroll
  for (int sb = 0; sb < 2; ++sb) {
    double v = 0.0;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      const uint32_t sw = *(const uint32_t*)(srow[sb] + i0 + 16 * ib + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int il = 16 * ib + 4 * g + e, i = i0 + il;
        double y = (double)acc[DD - 1][ib][sb][e];
#pragma unroll
        for (int p = DD - 2; p >= 0; --p) y = fma(y, 256.0, (double)acc[p][ib][sb][e]);
        y = ldexp(y, se[il] - 54);
        if (i < n) v += (double)(int8_t)(sw >> (8 * e)) * y;
      }
    }
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    const int64_t b = b0 + 16 * sb + r;
    if (g == 0 && b < B) part[(int64_t)blockIdx.y * B + b] = v;
  }
}

// E[b] = the row tiles' partial sums: eight loads in flight, four running sums, joined in a fixed order
__global__ void sum_partials_kernel(const double* __restrict__ part, int ntiles, int64_t B,
                                    double* __restrict__ E) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  int tt = 0;
  for (; tt + 8 <= ntiles; tt += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(tt + u) * B + b];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u & 3] += v[u];
  }
  for (; tt < ntiles; ++tt) s[tt & 3] += part[(int64_t)tt * B + b];
  E[b] = (s[0] + s[1]) + (s[2] + s[3]);
}

// Every row by energy_dense_f64_kernel up to so many sites and samples times 16-row tiles: a launch less (13.6 against
// 16.2 us at n = 100, B = 1024); from about 200 sites the integer cores gain more (16.2 against 20.4 us at n = 255, B = 64),
// and with more samples (n = 32: 13.9 against 16.6 us at B = 65536, 23 against 16.5 at 131072; n = 64: 13.8 against 16.6 at
// 20000, 19.8 against 16.3 at 40000; n = 128: 14.9 against 16.0 at 8192, 19.8 against 16.3 at 12000)
static bool dense_f64(int n, int ntiles, int64_t B) {
  return n <= 160 && (int64_t)ntiles * B <= std::max(65536, (13 << 19) / n);
}

// partial sums of the row tiles (of 16 rows at least), the rows' exponents
size_t energy_dense_ws_bytes(int n, int64_t B) {
  return (size_t)((n + 15) / 16) * (size_t)B * sizeof(double) + (size_t)round_up((int64_t)n * 4, 256);
}

size_t energy_workspace_bytes(const vqmc_hamiltonian& H, int64_t B) {
  return H.kind == VQMC_H_DENSE_F32 ? energy_dense_ws_bytes(H.n, B) : 0;
}

hipError_t launch_energy(const vqmc_hamiltonian& H, const int8_t* S, int64_t B, void* E, void* ws,
                         hipStream_t st) {
  const int n = H.n;
  const int64_t lds = round_up(n, kPad);
  if (H.kind == VQMC_H_DENSE_F32) {
    int ntiles = (n + 15) / 16;
    int32_t* ex = (int32_t*)((double*)ws + (int64_t)ntiles * B);
    hipError_t e;
    auto groups = [&](int nw) { return (B + 32 * nw - 1) / (32 * nw); };
    if (dense_f64(n, ntiles, B)) {
      energy_dense_f64_kernel<4><<<dim3((unsigned)groups(4), (unsigned)ntiles), 256, 0, st>>>(n, lds, H.J, S, B, (double*)ws);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      sum_partials_kernel<<<(unsigned)((B + 255) / 256), 256, 0, st>>>((const double*)ws, ntiles, B, (double*)E);
      return hipGetLastError();
    }
    energy_rowmax_kernel<<<(unsigned)((n + 3) / 4), 256, 0, st>>>(n, H.J, ex);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const bool vec = (n & 3) == 0 && ((uintptr_t)H.J & 15) == 0;
    // samples fastest: the longest row tiles start first
    auto go = [&](auto kern, int nw) {
      kern<<<dim3((unsigned)groups(nw), (unsigned)ntiles), 64 * nw, 0, st>>>(n, lds, H.J, ex, S, B, (double*)ws);
      e = hipGetLastError();
    };
    // 256 samples per conversion of J and 32 rows per spin operand while that leaves two workgroups
    // for every CU, else smaller tiles (n = 1000, B = 512: 18 us with 16 rows, 31 with 32)
    const int ntiles32 = (n + 31) / 32;
    if (groups(8) * ntiles32 >= 512) {
      ntiles = ntiles32;
      go(vec ? energy_dense_kernel<8, 2, true> : energy_dense_kernel<8, 2, false>, 8);
    } else if (groups(4) * ntiles >= 512) {
      go(vec ? energy_dense_kernel<4, 1, true> : energy_dense_kernel<4, 1, false>, 4);
    } else {
      go(vec ? energy_dense_kernel<2, 1, true> : energy_dense_kernel<2, 1, false>, 2);
    }
    if (e != hipSuccess) return e;
    sum_partials_kernel<<<(unsigned)((B + 255) / 256), 256, 0, st>>>((const double*)ws, ntiles, B,
                                                                       (double*)E);
    return hipGetLastError();
  }
  const int nst = (int)round_up(n, 16);
  // site bytes and reduction scratch always in LDS; the row pointer too when two
  // workgroups still fit on a CU
  const size_t rpb = (size_t)round_up((int64_t)(n + 1) * 4, 16);
  const size_t redb = (size_t)EMSE * (EB_THREADS / 64) * 8;
  const bool rp_lds = H.nnz < (int64_t)1 << 31 && (size_t)nst + rpb + redb <= 64 * 1024;
  const size_t shbytes = (size_t)nst + (rp_lds ? rpb : 0) + redb;
  const unsigned grid = (unsigned)((B + EMSE - 1) / EMSE);
  hipError_t e;
  // lanes that share a row: 8 to 16 edges each on average, one lane below 16 edges a row (float weights, n = 1001,
  // mean row 125, B = 1024: 66 us, 138 with one lane, 87 with 4 to 8 edges; mean row 10: 14 us with one
  // lane, 18 with four, each of which repeats the row's start and end)
  int lanes = 1;
  while (lanes < 64 && (int64_t)16 * lanes * n <= H.nnz) lanes *= 2;
  auto go = [&](auto kern, auto wptr, auto eptr) {
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shbytes);
    if (e != hipSuccess) return;
    kern<<<grid, EB_THREADS, shbytes, st>>>(n, lds, H.rowptr, H.col, wptr, S, B, nst, lanes, eptr);
    e = hipGetLastError();
  };
  if (H.kind == VQMC_H_CSR_INT) {
    // byte lanes when the site words fit in one CU's LDS (the row pointer too if it fits)
    const size_t swb = (size_t)nst * 8;
    if (H.nnz >= EC_U && H.nnz < (int64_t)1 << 30 && swb + redb <= 160 * 1024) {
      const bool rpl = swb + rpb + redb <= 160 * 1024;
      const size_t sb = swb + (rpl ? rpb : 0) + redb;
      // two workgroups a CU where there is work and LDS for them, two rows at a time then (64 registers): n = 500, 8 % of the
      // edges, B = 16384: 35 against 74 us; one workgroup a CU: four rows, 17 against 29 us at n = 16000, degree 6, B = 1
      const bool pair = grid > 256 && 2 * sb <= 160 * 1024;
      auto kern = pair ? (rpl ? energy_csr_bytes_kernel<true, 2> : energy_csr_bytes_kernel<false, 2>)
                       : (rpl ? energy_csr_bytes_kernel<true, 4> : energy_csr_bytes_kernel<false, 4>);
      if ((e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sb)) !=
          hipSuccess)
        return e;
      kern<<<grid, EB_THREADS, sb, st>>>(n, lds, H.rowptr, H.col, (const int32_t*)H.w, H.nnz, S, B, nst, lanes,
                                         (int64_t*)E);
      return hipGetLastError();
    }
    auto kern = lanes > 1 ? (rp_lds ? energy_csr_bits_kernel<int32_t, int64_t, true, true> : energy_csr_bits_kernel<int32_t, int64_t, false, true>)
                          : (rp_lds ? energy_csr_bits_kernel<int32_t, int64_t, true, false> : energy_csr_bits_kernel<int32_t, int64_t, false, false>);
    go(kern, (const int32_t*)H.w, (int64_t*)E);
  } else {
    const bool pair = grid > 256;  // more workgroups than CUs
    // one lane a row up to 32 edges a row where there are rows for most of the threads and a CU has one workgroup
    // (n = 1421, mean row 26, B = 2: 26.6 against 29.2 us with two lanes; n = 638 17.5 against 16.7; two workgroups a CU,
    // n = 3400, mean row 25, B = 4017: 163 against 117)
    if (!pair && n >= 768 && H.nnz < (int64_t)32 * n) lanes = 1;
    auto kern = lanes > 1 ? (pair ? (rp_lds ? energy_csr_bits_kernel<float, double, true, true> : energy_csr_bits_kernel<float, double, false, true>)
                                  : (rp_lds ? energy_csr_bits_kernel<float, double, true, true, 4> : energy_csr_bits_kernel<float, double, false, true, 4>))
                          : (rp_lds ? energy_csr_bits_kernel<float, double, true, false> : energy_csr_bits_kernel<float, double, false, false>);
    go(kern, (const float*)H.w, (double*)E);
  }
  return e;
}

// ---------------------------------------------------------------- statistics
// One workgroup of 1024 threads; every reduction has a fixed shape, so the result is
// bit-reproducible.  int64 energies are summed exactly before the single division.
template <typename ET>
__global__ __launch_bounds__(1024) void stats_kernel(const ET* __restrict__ E, int64_t B,
                                                      vqmc_stats* __restrict__ out,
                                                      float* __restrict__ coef) {
  constexpr int NW = 1024 / 64;
  __shared__ ET wsum[NW];
  __shared__ ET wmin[NW];
  __shared__ int64_t warg[NW];
  __shared__ double wsd[NW];
  __shared__ double s_mean;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  ET s = 0;
  ET mn = 0;
  int64_t am = -1;
  for (int64_t b = t; b < B; b += 1024) {
    const ET v = E[b];
    s += v;
    if (am < 0 || v < mn) {
      mn = v;
      am = b;
    }
  }
  // butterflies over the wave (lane 0's result is used), then the sixteen waves in order
  auto better = [](ET m1, int64_t a1, ET m0, int64_t a0) {  // (m1, a1) replaces (m0, a0)
    return a1 >= 0 && (a0 < 0 || m1 < m0 || (m1 == m0 && a1 < a0));
  };
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o);
    const ET mo = __shfl_xor(mn, o);
    const int64_t ao = __shfl_xor(am, o);
    if (better(mo, ao, mn, am)) {
      mn = mo;
      am = ao;
    }
  }
  if (lane == 0) {
    wsum[wv] = s;
    wmin[wv] = mn;
    warg[wv] = am;
  }
  __syncthreads();
  if (t == 0) {
    ET ts = wsum[0], tm = wmin[0];
    int64_t ta = warg[0];
    for (int k = 1; k < NW; ++k) {
      ts += wsum[k];
      if (better(wmin[k], warg[k], tm, ta)) {
        tm = wmin[k];
        ta = warg[k];
      }
    }
    s_mean = (double)ts / (double)B;
    out->mean_E = s_mean;
    out->min_E = (double)tm;
    out->argmin = ta;
    out->sum_E = (double)ts;
  }
  __syncthreads();
  const double mean = s_mean;
  double v2 = 0.0;
  for (int64_t b = t; b < B; b += 1024) {
    const double dv = (double)E[b] - mean;
    v2 += dv * dv;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v2 += __shfl_xor(v2, o);
  if (lane == 0) wsd[wv] = v2;
  __syncthreads();
  if (t == 0) {
    double tv = wsd[0];
    for (int k = 1; k < NW; ++k) tv += wsd[k];
    out->var_E = tv / (double)B;
  }
  if (coef)
    for (int64_t b = t; b < B; b += 1024) coef[b] = (float)(((double)E[b] - mean) / (double)B);
}

hipError_t launch_stats(const void* E, int e_is_int, int64_t B, vqmc_stats* stats, float* coef,
                        hipStream_t st) {
  if (e_is_int)
    stats_kernel<int64_t><<<1, 1024, 0, st>>>((const int64_t*)E, B, stats, coef);
  else
    stats_kernel<double><<<1, 1024, 0, st>>>((const double*)E, B, stats, coef);
  return hipGetLastError();
}

}  // namespace vqmc
