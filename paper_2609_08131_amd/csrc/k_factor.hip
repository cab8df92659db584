// Capacity matrix A = ridge I + M (Eq. 9) -- or R + M with a caller-supplied
// SPD matrix R (the output-projection variant) -- its Cholesky factor A = L L^T and
// the triangular inverse L^{-1}, one workgroup per unit, in fp64 in LDS.
// ||L^{-1} v||^2 = v^T A^{-1} v is what the leverage score of Eq. 10 needs.
//
// Input: the unit's Gram in the layout of its pass (see k_gram.hip): its
// per-chunk partials, summed here in chunk order in fp64, or (units of many
// chunks) the reduce kernel's sum of them. Output, after the
// first factorisation of an fp32-accumulated
// Gram (bf16 inputs): L^{-1} rounded to fp32 and split into bf16 hi + lo
// terms, stored directly in the per-lane B-fragment order of the 16x16x32
// MFMA (only the K-blocks that touch the lower triangle). After a
// factorisation of an fp64 Gram (fp32 inputs; the bf16 units marked for the
// fp64 path): L^{-1} in fp64, over the unit's slot of the reduced-Gram buffer
// in the operand order of the fp64 leverage pass (store_lower_f64).
//
// Blocked algorithm on 16x16 blocks. A unit's latency is what counts (a layer has
// few units, and thousands of them still share each compute unit two at a
// time), and the chain of 128 pivots bounds it, so nothing else stands in line
// with that chain that can run beside it:
//   Cholesky, for each block column k:
//     1. two waves factor the diagonal block in registers and, with the same
//        broadcasts, solve the panel below it (a row per lane) and 16 rows of
//        the identity, which become L_kk^{-T}; the other waves meanwhile
//        take the part of the previous rank-16 update that this column does
//        not need;
//     2. all waves update the next block column (fp64 MFMA).
//   Inverse X = L^{-1}, from the diagonal blocks (which step 1 leaves inverted),
//   by doubling: [[X11, 0], [-X22 L21 X11, X22]] for halves of 1, 2 and 4
//   blocks -- two products per level, their 16x16 output blocks spread over
//   all waves, instead of a serial sweep over seven block columns.
// LDS holds only the lower 16x16 blocks of A (about 78 KB at d = 128, so two
// workgroups share a compute unit); L replaces A and X replaces L there,
// block by block as each part is consumed.
//
// Measured (MI355X, d = 128): 8 units 51 us and 4096 units 604 us with the panel as
// a phase of its own, the diagonal blocks inverted after the factorisation and
// the column sweep; 40 us and 506 us here.
#include <algorithm>
#include <type_traits>

#include "jacap_internal.hpp"

namespace jacap {

// Bound on cond(A) above which the bf16 path recomputes the unit in fp64: the
// fp32-accumulated two-term Gram and the two-term L^{-1} products carry errors
// that A^{-1} amplifies by up to cond(A) (~1e-8 cond(A) in the scores, so at
// most ~2e-4 below the threshold; the bound itself can exceed cond(A) by one
// or two orders of magnitude).
constexpr double kRefineCond = 2e4;
// Smallest pivot, relative to its diagonal entry, taken as positive. On the
// fp32-accumulated Gram a smaller one sends the unit to the fp64 path. On an
// fp64 Gram it means A is numerically singular at the score tolerance: a
// pivot ratio r implies cond(A) >= 1 / r, and fp64 rounding (any evaluation
// order, ~1e-14 relative in A) then moves the scores by about 5e-15 / r, so
// below 1e-13 / tol (1e-10 for the 1e-3 of bf16 inputs, 1e-8 for the 1e-5 of
// fp32 inputs) the scores are not determined to the tolerance -- at ridge 0,
// a rank-deficient M or a saturated softmax's weights spanning 1e30.
constexpr double kPivRelRefine = 1e-4;
constexpr double kPivRelSingularBf16 = 1e-10;
constexpr double kPivRelSingularFp32 = 1e-8;

// Eight waves: two per SIMD, so that one wave's LDS and fp64 latencies
// overlap the other's work (the capacity factorisation also has a
// four-wave shape, see factor_kernel).
constexpr int kFactorThreads = 512;

// Lane n of each 16-lane row, broadcast to the row (one 64-bit DPP move,
// row_newbcast); n is a constant once the caller's loop is unrolled.
template <int N>
__device__ __forceinline__ double row_bcast_f64(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xF, 0xF, false);
}
__device__ __forceinline__ double row_bcast_f64_at(double v, int n) {
  switch (n) {
    case 0: return row_bcast_f64<0>(v);
    case 1: return row_bcast_f64<1>(v);
    case 2: return row_bcast_f64<2>(v);
    case 3: return row_bcast_f64<3>(v);
    case 4: return row_bcast_f64<4>(v);
    case 5: return row_bcast_f64<5>(v);
    case 6: return row_bcast_f64<6>(v);
    case 7: return row_bcast_f64<7>(v);
    case 8: return row_bcast_f64<8>(v);
    case 9: return row_bcast_f64<9>(v);
    case 10: return row_bcast_f64<10>(v);
    case 11: return row_bcast_f64<11>(v);
    case 12: return row_bcast_f64<12>(v);
    case 13: return row_bcast_f64<13>(v);
    case 14: return row_bcast_f64<14>(v);
    default: return row_bcast_f64<15>(v);
  }
}

// 1 / sqrt(x): the hardware estimate (relative error 2^-24.2, measured on
// the device) and Newton steps, one (2^-47.8) or two (2^-51.9, full fp64).
template <bool FULL>
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  y = y * fma(-h, y * y, 1.5);
  if constexpr (FULL) y = y * fma(-h, y * y, 1.5);
  return y;
}

// LDS layout of A (and of L, then X = L^{-1}, which replace it): only the
// lower 16x16 blocks (I >= J), packed by rows of blocks; block (I, J) starts
// at (I (I + 1) / 2 + J) * kBlk and holds element (r, c) at r * kBP + c. The
// pitch of 17 doubles puts the 16 rows of a block column in distinct banks.
// Diagonal blocks are stored whole.
constexpr int kBP = 17;
constexpr int kBlk = 16 * kBP;
__device__ __forceinline__ int lidx(int row, int col) {
  const int I = row >> 4, J = col >> 4;
  return (I * (I + 1) / 2 + J) * kBlk + (row & 15) * kBP + (col & 15);
}

// Lower-triangle index e -> (row i, column j), j <= i (row-major over the triangle).
__device__ __forceinline__ void tri_index(int e, int& i, int& j) {
  int r = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
  while ((r + 1) * (r + 2) / 2 <= e) ++r;
  while (r * (r + 1) / 2 > e) --r;
  i = r;
  j = e - r * (r + 1) / 2;
}

// Elements (u16) of one unit's two-term B fragments of a lower-triangular
// d x d matrix (see store_lower_frags).
__host__ __device__ constexpr int lower_frag_elems(int d) {
  return (d / 32) * (d / 32 + 1) * 2 * 64 * 8;
}

// A lower-triangular matrix X (x(a, b) = X[a][b] for b <= a, any value at the other
// entries of the 32-wide blocks on the diagonal) rounded to fp32
// and split into bf16 hi + lo terms, stored in the per-lane B-fragment order
// of the 16x16x32 MFMA for Y = V X^T: B fragment of output block j
// (a = 16 j + ch) and K block kb (b = 32 kb + 8 kg + q), only the pairs with
// kb <= j / 2 (the rest of X^T is zero); lane (ch, kg) holds 8 bf16, hi then
// lo.
template <int D, typename F>
__device__ __forceinline__ void store_lower_frags(uint16_t* __restrict__ out, F x) {
  constexpr int NB = D / 16;
  constexpr int NLP = (NB / 2) * (NB / 2 + 1);  // lower (j, kb) pairs: sum_j (j/2 + 1)
  static_assert(NLP * 2 * 64 * 8 == lower_frag_elems(D), "fragment count");
  for (int e = threadIdx.x; e < NLP * 64; e += blockDim.x) {
    const int qp = e / 64, ln = e % 64, ch = ln & 15, kg = ln >> 4;
    int j = 0, kb = 0, q = qp;
    for (int jj = 0; jj < NB; ++jj) {
      const int cnt = jj / 2 + 1;
      if (q < cnt) { j = jj; kb = q; break; }
      q -= cnt;
    }
    const int a = 16 * j + ch;
    uint16_t hi[8], lo[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int b = 32 * kb + 8 * kg + t;
      const float xr = (float)x(a, b);  // read also where it is not used (in range)
      const float xv = (b <= a) ? xr : 0.0f;
      const __bf16 h = (__bf16)xv;
      const __bf16 l = (__bf16)(xv - (float)h);
      hi[t] = __builtin_bit_cast(uint16_t, h);
      lo[t] = __builtin_bit_cast(uint16_t, l);
    }
    uint16_t* dh = out + ((int64_t)(qp * 2 + 0) * 64 + ln) * 8;
    uint16_t* dl = out + ((int64_t)(qp * 2 + 1) * 64 + ln) * 8;
#pragma unroll
    for (int t = 0; t < 8; ++t) { dh[t] = hi[t]; dl[t] = lo[t]; }
  }
}

// A lower-triangular matrix (x(a, b) for b <= a) in fp64, in the order in which
// the fp64 leverage pass supplies it to the MFMA 16x16x4: block (J, B), B <= J, at
// (J (J + 1) / 2 + B) * 256; its K-step s of lane l at (s / 2) * 128 + 2 l + s % 2,
// holding X[16 J + l % 16][16 B + 4 (l / 16) + s] (zero above the diagonal).
template <int D, typename F>
__device__ __forceinline__ void store_lower_f64(double* __restrict__ out, F x) {
  constexpr int NB = D / 16;
  for (int e = threadIdx.x; e < NB * (NB + 1) / 2 * 256; e += blockDim.x) {
    int J, B;
    tri_index(e >> 8, J, B);
    const int l = (e >> 1) & 63, s = 2 * ((e >> 7) & 1) + (e & 1);
    const int a = 16 * J + (l & 15), b = 16 * B + 4 * (l >> 4) + s;
    const double xr = x(a, b);
    out[e] = b <= a ? xr : 0.0;
  }
}

// Blocked Cholesky A = L L^T in place on the lower blocks in LDS (see lidx),
// given dg = diag(A) before factorisation and *bad == 0 (both visible to
// every thread). INV: the diagonal blocks receive X_kk = L_kk^{-1} (whole, zeros
// above the diagonal) instead of L_kk. Returns 0, or the flag that stopped
// it -- kUnitNonfinite for a non-finite pivot, `fail` for a pivot at or below
// piv_rel times its diagonal entry -- the same value in every thread.
// FULL: the pivots' reciprocal square roots to full fp64 accuracy; else to
// 2^-47.8, for factors that are rounded to two bf16 terms afterwards.
template <int D, int NT, bool FULL, bool INV>
__device__ __forceinline__ int cholesky_lds(double* A, const double* dg, int* bad, double piv_rel,
                                            int fail) {
  constexpr int NB = D / 16;
  constexpr int NW = NT / 64;
  constexpr int CW = 2;  // waves of the pivot chain: D - 16 panel rows and 16 of the identity
  static_assert(CW * 64 >= D, "a lane per row");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // 1. Block column kb. Every 16-lane row of a chain wave holds the diagonal
  //    block (lane s row s) and each lane one row of the panel or of the identity;
  //    one broadcast of L[q][t] serves both. The chain from one pivot to the
  //    next is a broadcast, a reciprocal square root and one broadcast-FMA; the
  //    pivot thresholds are read before it starts and the checks stay off it.
  //    d[q] is left with what entry q of this lane's row (INV: column) of the
  //    new diagonal block is to be: both chain waves read the old one.
  auto chain = [&](int kb, double (&d)[16]) {
    const int c = 16 * kb;
    const int s = lane & 15;
    const int npan = D - c - 16;            // panel rows
    const int e = 64 * wave + lane;         // this lane's row of the panel, then of I
    const bool pan = e < npan, idn = INV && e >= npan && e < npan + 16;
    const int prow = pan ? c + 16 + e : c;  // (a row that exists)
    double a[16], x[16], thr[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const double v = A[lidx(c + s, c + q)];  // the diagonal block is stored whole
      a[q] = (q <= s) ? v : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const double v = A[lidx(prow, c + q)];
      x[q] = pan ? v : (idn && q == e - npan ? 1.0 : 0.0);
    }
    // A pivot that has lost all but piv_rel of its diagonal entry is within
    // the rounding noise of A: A is numerically singular at the working
    // precision (or the caller's fail condition holds).
#pragma unroll
    for (int t = 0; t < 16; ++t) thr[t] = piv_rel * dg[c + t];
    // No early exit: after a failed pivot the rest is computed on whatever it
    // produced and discarded; the flag is the first failure's kind.
    bool failed = false, nonfinite = false;
    double piv = row_bcast_f64<0>(a[0]);  // A[t][t], from lane t of the row
    double y = rsqrt_f64<FULL>(piv);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const bool ok = piv > thr[t] && piv > 0.0;
      if (!ok && !failed) nonfinite = !isfinite(piv);
      failed = failed || !ok;
      a[t] = a[t] * y;  // column t of L (lane t: piv y; rows s < t: unused)
      x[t] = x[t] * y;
      // a[q] -= L[s][t] L[q][t] for q > t; L[q][t] is lane q's a[t]. Entries
      // with q > s are outside row s's lower part and never stored. Row
      // t + 1 goes first, and the next pivot's reciprocal square root is
      // issued before the other rows' updates, which then fill its latency.
      if (t + 1 < 16) {
        const double l = row_bcast_f64_at(a[t], t + 1);
        a[t + 1] = fma(-a[t], l, a[t + 1]);
        x[t + 1] = fma(-x[t], l, x[t + 1]);
        piv = row_bcast_f64_at(a[t + 1], t + 1);
        y = rsqrt_f64<FULL>(piv);
      }
#pragma unroll
      for (int q = t + 2; q < 16; ++q) {
        const double l = row_bcast_f64_at(a[t], q);
        a[q] = fma(-a[t], l, a[q]);
        x[q] = fma(-x[t], l, x[q]);
      }
      __builtin_amdgcn_sched_barrier(0);  // later steps' broadcasts held back: they would spill
    }
    // The rows of x exist here, on every path: moved into the branches below, their
    // updates would keep all 120 broadcasts live.
#pragma unroll
    for (int q = 0; q < 16; ++q) asm volatile("" : "+v"(x[q]));
    const int code = failed ? (nonfinite ? (int)kUnitNonfinite : fail) : 0;
    if (code) {  // the same in both chain waves
      if (wave == 0 && lane == 0) *bad = code;
      return;
    }
    if (pan) {
#pragma unroll
      for (int q = 0; q < 16; ++q) A[lidx(prow, c + q)] = x[q];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) d[q] = INV ? x[q] : a[q];
  };
  // The diagonal block, once every chain wave has read the old one; no step of
  // the factorisation reads it again.
  auto store_diag = [&](int kb, const double (&d)[16]) {
    const int c = 16 * kb, s = lane & 15;
    const int r = 64 * wave + lane - (D - c - 16);
    if (INV && r >= 0 && r < 16) {  // row r of L_kk^{-T}: column r of X_kk
#pragma unroll
      for (int q = 0; q < 16; ++q) A[lidx(c + q, c + r)] = d[q];
    }
    if (!INV && wave == 0 && lane < 16) {
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (q <= s) A[lidx(c + s, c + q)] = d[q];
    }
  };
  // 2. Trailing update A_IJ -= L_Ik L_Jk^T of one 16x16 block (I >= J > k) by
  //    one wave on the fp64 MFMA (K = 16 in four slices). Diagonal blocks also
  //    update their upper half, which nothing reads.
  auto update = [&](int kb, int bi, int bj) {
    const int c = 16 * kb, r16 = lane & 15, q4 = lane >> 4;
    const int I = 16 * bi, J = 16 * bj;
    // two chains: half the latency of four dependent MFMAs
    f64x4 acc, acc2 = {0.0, 0.0, 0.0, 0.0};
    double l[4], r[4];
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) {
      const int t = c + 4 * kq + q4;
      l[kq] = A[lidx((I + r16), t)];
      r[kq] = A[lidx((J + r16), t)];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = A[lidx((I + 4 * i + q4), J + r16)];
    acc2 = mfma64(-l[0], r[0], acc2);
    acc = mfma64(-l[1], r[1], acc);
    acc2 = mfma64(-l[2], r[2], acc2);
    acc = mfma64(-l[3], r[3], acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) A[lidx((I + 4 * i + q4), J + r16)] = acc[i] + acc2[i];
  };
  for (int kb = 0; kb < NB; ++kb) {
    const int m = NB - 1 - kb;  // block columns to the right
    const bool chains = wave < CW && 64 * wave < 16 * m + (INV || wave == 0 ? 16 : 0);
    double d[16];
    if (chains) {
      chain(kb, d);
    } else if (wave >= CW && kb > 0) {
      // the previous column's update of the blocks right of column kb
      for (int e = wave - CW; e < m * (m + 1) / 2; e += NW - CW) {
        int bi, bj;
        tri_index(e, bi, bj);
        update(kb - 1, kb + 1 + bi, kb + 1 + bj);
      }
    }
    __syncthreads();
    if (*bad) return *bad;
    if (chains) store_diag(kb, d);
    for (int e = wave; e < m; e += NW) update(kb, kb + 1 + e, kb + 1);
    __syncthreads();
  }
  return 0;
}

// The units that the first factorisation of bf16 inputs marks for the fp64
// path: their count and list (any order), beside the per-unit flag.
struct Marked {
  uint32_t* count;
  int32_t* list;
  __device__ __forceinline__ void add(int u, uint32_t* uflags) const {
    atomicOr(uflags + u, kUnitRefine);
    list[atomicAdd(count, 1u)] = u;
  }
};

// One unit. Its Gram: PASS 0 (all units) reads the reduced Gram `red` if the
// reduce kernel ran (`reduced`), else sums here, in chunk order, in fp64, the
// fp32 MFMA partials `part32` (bf16 inputs; gchunks per unit of gchunk tokens)
// or the unit's nch64 fp64 partials `part` (fp32 inputs) -- the reduce kernel's
// arithmetic; PASS 1 (the units of bf16 inputs that pass 0 marked) sums its
// fp64 partials. FRAGS: bf16 inputs.
template <int D, bool FRAGS, int NT, int PASS>
__device__ __forceinline__ void factor_unit(const Geo& g, int u, double* __restrict__ red,
                                            const double* __restrict__ part, int nch64,
                                            const float* __restrict__ part32, int gchunks,
                                            int gchunk, bool reduced, double ridge,
                                            const double* __restrict__ wscale,
                                            uint16_t* __restrict__ lfrag, uint32_t* status,
                                            uint32_t* uflags, const Marked& marked) {
  constexpr int NB = D / 16;
  constexpr int NPAIR = NB * (NB + 1) / 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Unit un = decode_unit(g, u);
  if (un.n == 0) return;
  // The fp32-accumulated Gram of bf16 inputs may be redone in fp64 later;
  // singularity is decided on an fp64 Gram only (pass 1, or fp32 inputs).
  constexpr bool may_refine = FRAGS && PASS == 0;
  constexpr double piv_rel =
      may_refine ? kPivRelRefine : (FRAGS ? kPivRelSingularBf16 : kPivRelSingularFp32);

  __shared__ double A[NB * (NB + 1) / 2 * kBlk];  // lower 16x16 blocks, see lidx
  __shared__ double dg[D];   // diagonal of A before factorisation
  __shared__ double red_sh[NT / 64];
  __shared__ double red_sh2[NT / 64];
  __shared__ double red_sh3[NT / 64];
  __shared__ int bad;        // 0, or the unit flag that stops the factorisation

  // Lower triangle of A = ridge I + M from the upper blocks of M. Entries
  // (2 e', 2 e' + 1) share a block pair and a lane: each thread loads its
  // pairs first (all loads in flight), then places them.
  constexpr int NE2 = NPAIR * 128;  // entry pairs
  constexpr int PER = (NE2 + NT - 1) / NT;
  double2 rv[PER];
  // Fixed-order sum of the unit's partials (the chunk loop unrolled so that
  // about 18 of a thread's loads are in flight; more spills registers).
  constexpr int CHU = PER <= 9 ? 2 : 1;
#pragma unroll
  for (int k = 0; k < PER; ++k) rv[k] = make_double2(0.0, 0.0);
  if (PASS == 0 && reduced) {
    const double2* R = reinterpret_cast<const double2*>(red + (int64_t)u * (NPAIR * 256));
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e2 = tid + k * NT;
      if (e2 < NE2) rv[k] = R[e2];
    }
  } else if (may_refine) {  // fp32 MFMA partials
    const int nch = (un.n + gchunk - 1) / gchunk;
    const float2* P = reinterpret_cast<const float2*>(part32 + (int64_t)u * gchunks * (NPAIR * 256));
#pragma unroll CHU
    for (int c = 0; c < nch; ++c) {
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e2 = tid + k * NT;
        if (e2 < NE2) {
          const float2 x = P[(int64_t)c * NE2 + e2];
          rv[k].x += (double)x.x;
          rv[k].y += (double)x.y;
        }
      }
    }
  } else {  // fp64 partials
    const double2* P = reinterpret_cast<const double2*>(part);
#pragma unroll CHU
    for (int c = 0; c < nch64; ++c) {
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e2 = tid + k * NT;
        if (e2 < NE2) {
          const double2 x = P[(int64_t)c * NE2 + e2];
          rv[k].x += x.x;
          rv[k].y += x.y;
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int e2 = tid + k * NT;
    if (e2 < NE2) {
      const int e = 2 * e2;
      // block pair p -> block (bi, bj), bi <= bj, row-major; two waves per pair
      const int p = (wave >> 1) + k * (NT / 128);
      int bi = 0;
#pragma unroll
      for (int q = 1; q < NB; ++q) bi += p >= q * NB - q * (q - 1) / 2;
      const int bj = p - (bi * NB - bi * (bi - 1) / 2) + bi;
      if (may_refine) {  // block-lane layout
        const int ln = (e & 255) / 4, r = e % 4;  // r even: entries r and r + 1 of lane ln
        const int row = bi * 16 + (ln >> 4) * 4 + r;
        const int col = bj * 16 + (ln & 15);
        if (row <= col) A[lidx(col, row)] = rv[k].x;  // diagonal block: upper half only
        if (row + 1 <= col) A[lidx(col, row + 1)] = rv[k].y;
      } else {  // the fp64 pass's layout: channels NB (4 i + l / 16) + bi, NB (l % 16) + bj
        const int i = (e >> 6) & 3, l = e & 63;  // l even: entries of lanes l and l + 1
        const int ra = NB * (4 * i + (l >> 4)) + bi, cb = NB * (l & 15) + bj;
        // bi == bj: an entry and its mirror image, the upper one left out
        if (bi != bj || ra >= cb) A[lidx(max(ra, cb), min(ra, cb))] = rv[k].x;
        const int cb1 = cb + NB;
        if (bi != bj || ra >= cb1) A[lidx(max(ra, cb1), min(ra, cb1))] = rv[k].y;
      }
    }
  }
  if (tid == 0) bad = 0;
  __syncthreads();
  // The weights of a saturated softmax are stored times a power of two (the
  // weight pass's scale); the ridge term takes the same factor, so that A is
  // the capacity matrix times it and every score is unchanged.
  const double sc = wscale[u];
  if (g.ridge_mat) {  // output-projection variant: A = R + M
    const double* Rm = g.ridge_mat + ((int64_t)un.l * g.H + un.h) * D * D;
    for (int e = tid; e < D * D; e += NT) {
      const int r = e / D, cc = e % D;
      if (cc <= r) A[lidx(r, cc)] += Rm[e] * sc;
    }
    __syncthreads();
  }
  for (int a = tid; a < D; a += NT) {
    if (!g.ridge_mat) A[lidx(a, a)] += ridge * sc;
    dg[a] = A[lidx(a, a)];
    if (!isfinite(dg[a])) atomicOr(&bad, (int)kUnitNonfinite);
  }
  __syncthreads();
  if (bad) {
    if (tid == 0) raise_flags(status, uflags, u, kUnitNonfinite);
    return;
  }

  // Largest sum of |.| over the rows (COLS: columns) of blocks that `entry`
  // reads: block row I of a wave (I, and NB-1-I where the waves are fewer), lane
  // (r16, q4) taking four entries 4 kq + q4 of row r16 per block, independent
  // reads of constant stride; then the four lanes of a row and the rows.
  constexpr int NW = NT / 64;
  const int r16 = lane & 15, q4 = lane >> 4;
  auto wave_rows_max = [&](auto entry) {
    double best = 0.0;
#pragma unroll
    for (int p = 0; p < (NB + NW - 1) / NW; ++p) {
      const int I = p == 0 ? wave : NB - 1 - wave;
      if (I < NB && (p == 0 || I != wave)) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        entry(I, s);
        double sr = (s[0] + s[1]) + (s[2] + s[3]);
        sr += __shfl_xor(sr, 16);
        sr += __shfl_xor(sr, 32);
        best = fmax(best, sr);
      }
    }
    best = fmax(best, dpp_f64<kDppQuadXor1>(best));
    best = fmax(best, dpp_f64<kDppQuadXor2>(best));
    best = fmax(best, dpp_f64<kDppHalfMirror>(best));
    return fmax(best, dpp_f64<kDppMirror>(best));
  };

  // max over rows of sum_c |A[r][c]| (>= lambda_max(A)), A symmetric with its
  // lower triangle stored: row r of block row I is the blocks J < I, the
  // diagonal block's own lower half mirrored, and column r of the blocks K > I.
  if constexpr (may_refine) {
    const double wm = wave_rows_max([&](int I, double (&s)[4]) {
      // every block of the row read (the diagonal one apart), whichever side of
      // the diagonal it is on: NB x 4 independent reads
#pragma unroll
      for (int K = 0; K < NB; ++K)
#pragma unroll
        for (int kq = 0; kq < 4; ++kq) {
          const int t = 4 * kq + q4;
          const int lo = K == I ? min(r16, t) : K < I ? t : r16, hi = K == I ? max(r16, t) : K < I ? r16 : t;
          s[kq] += fabs(A[lidx(16 * max(I, K) + hi, 16 * min(I, K) + lo)]);
        }
    });
    if (lane == 0) red_sh3[wave] = wm;  // read with the inverse's norms
  }

  // ---------------- Cholesky A = L L^T (L overwrites the lower triangle) ----
  // The first factorisation of bf16 inputs ends in two-term bf16 fragments
  // of L^{-1}; the fp64 paths keep full precision.
  const int code =
      may_refine ? cholesky_lds<D, NT, false, true>(A, dg, &bad, piv_rel, (int)kUnitRefine)
                 : cholesky_lds<D, NT, true, true>(A, dg, &bad, piv_rel, (int)kUnitSingular);
  if (code) {
    if (tid == 0) {
      if (code == (int)kUnitRefine) marked.add(u, uflags);
      else raise_flags(status, uflags, u, (uint32_t)code);
    }
    return;
  }

  // ---------------- Inverse X = L^{-1} --------------------------------------
  // The diagonal blocks hold X_kk. By doubling, for halves of h blocks: with
  // rows I of the lower half and columns J of the upper half of a diagonal pair,
  //   T_IJ = sum_{M >= J} L_IM X_MJ,  X_IJ = -sum_{M <= I} X_IM T_MJ,
  // each in place: the sums stay in registers until every wave has read its
  // operands. The output blocks go over the waves so that every SIMD has as
  // many products of both stages (mirrored for every second pair or row pair).
  {
    // D += P Q of two blocks: P = block (I, M), Q = block (M, J)
    auto product = [&](int I, int M, int J, f64x4 acc) {
      double pa[4], qb[4];
#pragma unroll
      for (int kq = 0; kq < 4; ++kq) {
        const int t = 4 * kq + q4;
        pa[kq] = A[lidx(16 * I + r16, 16 * M + t)];
        qb[kq] = A[lidx(16 * M + t, 16 * J + r16)];
      }
#pragma unroll
      for (int kq = 0; kq < 4; ++kq) acc = mfma64(pa[kq], qb[kq], acc);
      return acc;
    };
    auto level = [&](auto hc) {
      constexpr int h = decltype(hc)::value;
      constexpr int NOUT = NB * h / 2;               // output blocks
      constexpr int PW = (NOUT + NW - 1) / NW;       // ... per wave, at most
      auto place = [&](int o, int& base, int& i, int& j) {
        int r = o % (h * h);
        const int pr = o / (h * h);
        if (h == 2 && (pr & 1)) r = h * h - 1 - r;
        i = r / h;
        j = r % h;
        if (h == 4 && ((o / NW) & 1)) j = h - 1 - j;
        base = 2 * h * pr;
      };
#pragma unroll
      for (int stage = 0; stage < 2; ++stage) {
        f64x4 acc[PW];
#pragma unroll
        for (int p = 0; p < PW; ++p) {
          acc[p] = f64x4{0.0, 0.0, 0.0, 0.0};
          const int o = wave + NW * p;
          int base, i, j;
          place(o, base, i, j);
          if (o < NOUT) {
            if (stage == 0)
              for (int M = j; M < h; ++M) acc[p] = product(base + h + i, base + M, base + j, acc[p]);
            else
              for (int M = 0; M <= i; ++M) acc[p] = product(base + h + i, base + h + M, base + j, acc[p]);
          }
        }
        __syncthreads();  // every wave's operands read
#pragma unroll
        for (int p = 0; p < PW; ++p) {
          const int o = wave + NW * p;
          int base, i, j;
          place(o, base, i, j);
          if (o < NOUT)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              A[lidx(16 * (base + h + i) + 4 * q + q4, 16 * (base + j) + r16)] =
                  stage == 0 ? acc[p][q] : -acc[p][q];
        }
        __syncthreads();
      }
    };
    level(std::integral_constant<int, 1>{});
    level(std::integral_constant<int, 2>{});
    if constexpr (NB == 8) level(std::integral_constant<int, 4>{});
    static_assert(NB == 4 || NB == 8, "head_dim 64 or 128");
  }
  // X[r][c], r >= c (entries above the diagonal are not used).
  auto xinv = [&](int r, int cc) -> double { return A[lidx(r, cc)]; };

  // cond(A) <= ||A||_inf ||L^{-1}||_1 ||L^{-1}||_inf (lambda_max <= ||A||_inf,
  // 1 / lambda_min = ||L^{-1}||_2^2 <= ||L^{-1}||_1 ||L^{-1}||_inf): a bound,
  // so no ill-conditioned unit escapes the refinement.
  if constexpr (may_refine) {
    // the diagonal blocks hold zeros above the diagonal
    const double wr = wave_rows_max([&](int I, double (&s)[4]) {
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int kq = 0; kq < 4; ++kq) {
          const double v = A[lidx(16 * I + r16, 16 * min(J, I) + 4 * kq + q4)];
          s[kq] += J <= I ? fabs(v) : 0.0;
        }
    });
    const double wc = wave_rows_max([&](int J, double (&s)[4]) {
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int kq = 0; kq < 4; ++kq) {
          const double v = A[lidx(16 * max(I, J) + 4 * kq + q4, 16 * J + r16)];
          s[kq] += I >= J ? fabs(v) : 0.0;
        }
    });
    if (lane == 0) { red_sh[wave] = wr; red_sh2[wave] = wc; }
    __syncthreads();
    double xinf = red_sh[0], x1 = red_sh2[0], anorm = red_sh3[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) {
      xinf = fmax(xinf, red_sh[w]);
      x1 = fmax(x1, red_sh2[w]);
      anorm = fmax(anorm, red_sh3[w]);
    }
    if (anorm * x1 * xinf > kRefineCond) {
      if (tid == 0) marked.add(u, uflags);
      return;  // pass 1 writes this unit's L^{-1}
    }
  }

  // Store L^{-1}.
  if (!may_refine) {  // fp64, over the unit's slot of the reduced-Gram buffer
    store_lower_f64<D>(red + (int64_t)u * (NPAIR * 256), xinv);
  } else {
    store_lower_frags<D>(lfrag + (int64_t)u * lower_frag_elems(D), xinv);
  }
}

// PASS 0: one workgroup per unit. PASS 1: a grid-stride walk over the marked
// units' list. NT threads: 512 (eight waves)
// when the units fit the compute units in one round; 256 (bounded to 256
// VGPRs, so that two workgroups share a compute unit and one's sequential
// steps overlap the other's) when there are more.
template <int D, bool FRAGS, int NT, int PASS>
__global__ __launch_bounds__(NT, 512 / NT) void factor_kernel(
    Geo g, double* __restrict__ red, const double* __restrict__ part, int pchunks, int pchunk,
    int pslots, const float* __restrict__ part32, int gchunks, int gchunk, int reduced,
    double ridge, const double* __restrict__ wscale, uint16_t* __restrict__ lfrag,
    uint32_t* status, uint32_t* uflags, Marked marked) {
  constexpr int64_t SZ = (D / 16) * (D / 16 + 1) / 2 * 256;
  auto unit = [&](int u, const double* P, int tok) {
    const int nch64 = (decode_unit(g, u).n + tok - 1) / tok;
    factor_unit<D, FRAGS, NT, PASS>(g, u, red, P, nch64, part32, gchunks, gchunk, reduced != 0,
                                    ridge, wscale, lfrag, status, uflags, marked);
  };
  if constexpr (PASS == 0) {
    const int u = blockIdx.x;
    unit(u, part + (int64_t)u * pchunks * SZ, pchunk);
  } else {
    const int nu = (int)*marked.count;
    const RefineCut rc = refine_cut(nu, g.maxn, pslots);
    for (int li = blockIdx.x; li < nu; li += gridDim.x) {
      unit(marked.list[li], part + (int64_t)li * rc.nch * SZ, rc.tok);
      __syncthreads();  // LDS of this unit fully consumed before the next one's loads
    }
  }
}

hipError_t launch_factor(const Launch& L, bool refine) {
  if (refine && !L.ws.mfma) return hipSuccess;
  const Geo& g = L.geo;
  double* red = ws_ptr<double>(L.wsp, L.ws.gram_red);
  uint16_t* lf = ws_ptr<uint16_t>(L.wsp, L.ws.lfrag);
  uint32_t* st = ws_ptr<uint32_t>(L.wsp, L.ws.status);
  uint32_t* uf = ws_ptr<uint32_t>(L.wsp, L.ws.uflags);
  const double* wsc = ws_ptr<double>(L.wsp, L.ws.wscale);
  const double ridge = (double)L.cfg->ridge;
  // the Gram partials: fp64 (fp32 inputs, and the refine pass), fp32 (the
  // first pass of bf16 inputs); both in the Gram buffer
  const double* part = ws_ptr<double>(L.wsp, L.ws.gram);
  const float* part32 = ws_ptr<float>(L.wsp, L.ws.gram);
  const Marked marked{st + 1, ws_ptr<int32_t>(L.wsp, L.ws.rlist)};
  const int blocks = refine ? std::min(g.U, kComputeUnits) : g.U;
  const bool pairs = !refine && g.U > kComputeUnits;  // two workgroups per compute unit
  auto go = [&](auto kern, int nt) {
    kern<<<blocks, nt, 0, L.stream>>>(g, red, part, L.ws.pchunks, L.ws.pchunk, L.ws.pslots, part32,
                                      L.ws.gchunks, L.ws.gchunk, gram_reduced(L) ? 1 : 0, ridge,
                                      wsc, lf, st, uf, marked);
  };
  if (refine) {
    if (g.D == 128) go(factor_kernel<128, true, 512, 1>, 512);
    else go(factor_kernel<64, true, 512, 1>, 512);
  } else if (L.ws.mfma) {
    if (g.D == 128) pairs ? go(factor_kernel<128, true, 256, 0>, 256) : go(factor_kernel<128, true, 512, 0>, 512);
    else pairs ? go(factor_kernel<64, true, 256, 0>, 256) : go(factor_kernel<64, true, 512, 0>, 512);
  } else {
    if (g.D == 128) pairs ? go(factor_kernel<128, false, 256, 0>, 256) : go(factor_kernel<128, false, 512, 0>, 512);
    else pairs ? go(factor_kernel<64, false, 256, 0>, 256) : go(factor_kernel<64, false, 512, 0>, 512);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FULL covariance, triangular K pass (full_kpass_tri): per unit, Lambda_Q of
// the pooled window in fp64 and a factor Lambda_Q = X^T X with X lower
// triangular, stored as two-term bf16 B fragments (store_lower_frags) in the
// L^{-1} fragment buffer, which is free until the capacity matrix is factored.
// Then kappa_i = k_i^T Lambda_Q k_i = ||X k_i||^2 (Sec. 3.4, full query
// covariance) takes the leverage pass's triangular MFMA product.
//
// X comes from the Cholesky factorisation of the order-reversed matrix:
// P Lambda_Q P = C C^T (P reverses the channel order, C lower triangular)
// gives Lambda_Q = (P C P)(P C P)^T with P C P upper triangular, so
// X = (P C P)^T, X[i][j] = C[d-1-j][d-1-i].
//
// Lambda_Q = (1/N_s) sum_r (q_r - mu)(q_r - mu)^T: the window (raw bf16, all
// of it in LDS) goes through the fp64 MFMA, each row centred in fp64 as it is
// read, each wave accumulating its share of the 16x16 lower blocks in
// registers; the blocks are then written to the factor's LDS layout already
// reversed.
//
// The unit is marked kUnitKTile (the K pass takes the window tile) if it has
// fewer than kTriMinTokens tokens, non-finite window statistics, or a pivot at
// most kPivRelTri of its diagonal entry: a numerically rank-deficient
// Lambda_Q, whose factor would not carry kappa to the tolerance in two bf16
// terms.
// ---------------------------------------------------------------------------
constexpr double kPivRelTri = 1e-3;

template <int D>
__device__ __forceinline__ void qfactor_unit(const Geo& g, int u, const uint16_t* __restrict__ q,
                                             const double* __restrict__ mu,
                                             uint16_t* __restrict__ xfrag,
                                             uint32_t* __restrict__ uflags) {
  constexpr int NB = D / 16;
  constexpr int NPAIR = NB * (NB + 1) / 2;
  constexpr int NW = kFactorThreads / 64;
  constexpr int PW = (NPAIR + NW - 1) / NW;  // lower 16x16 blocks of Lambda_Q per wave
  constexpr int QPB = D + 8;  // u16 per staged window row
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;
  const Unit un = decode_unit(g, u);
  if (un.n == 0) return;
  if (un.n < kTriMinTokens || (uflags[u] & kUnitNonfinite)) {
    if (tid == 0) atomicOr(uflags + u, kUnitKTile);
    return;
  }
  __shared__ double A[NPAIR * kBlk];  // lower 16x16 blocks, see lidx
  __shared__ double dg[D];
  __shared__ double smu[D];
  __shared__ __attribute__((aligned(16))) uint16_t qs[kFullMaxQ * QPB];  // the window, raw bf16
  __shared__ int bad;

  const int Ns = g.G * g.w;
  const uint16_t* qb =
      q + un.b * g.qss + un.l * g.qsl + (int64_t)(un.h * g.V + un.s) * g.G * g.qsh;
  for (int c = tid; c < D; c += kFactorThreads) smu[c] = mu[(int64_t)u * D + c];
  if (tid == 0) bad = 0;
  // The whole window in one round of 16-byte loads (N_s <= kFullMaxQ rows),
  // then the products over it with no further barrier. Rows N_s .. N_s4 - 1
  // are padding and masked.
  const int Ns4 = (Ns + 3) & ~3;
  for (int e = tid; e < Ns4 * (D / 8); e += kFactorThreads) {
    const int r = e / (D / 8), pc = e - r * (D / 8);
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (r < Ns) {
      const int gq = r / g.w, p = r - gq * g.w;
      x = *reinterpret_cast<const uint4*>(qb + gq * g.qsh + p * g.qsp + pc * 8);
    }
    *reinterpret_cast<uint4*>(qs + r * QPB + pc * 8) = x;
  }
  __syncthreads();  // window and smu visible
  // block (bi, bj), bi >= bj: sum_r (q_r - mu)[16 bi + i] (q_r - mu)[16 bj + j],
  // four rows per MFMA (lane (r16, q4) supplies row 4 s + q4, column r16 of
  // each), centred in fp64 as they are read; the wave's blocks take turns so
  // that their accumulation chains interleave.
  f64x4 acc[PW];
  int cbi[PW], cbj[PW];
  double mbi[PW], mbj[PW];
  // A wave's slots past the last block repeat that block (no branch in the
  // loop below); their sums are not stored.
#pragma unroll
  for (int p = 0; p < PW; ++p) {
    acc[p] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int e = min(wave + NW * p, NPAIR - 1);
    int bi, bj;
    tri_index(e, bi, bj);
    cbi[p] = 16 * bi + r16;
    cbj[p] = 16 * bj + r16;
    mbi[p] = smu[cbi[p]];
    mbj[p] = smu[cbj[p]];
  }
  // Each row group's raw values are read while the previous group's MFMAs
  // run (the last read repeats the last group and is not used).
  uint16_t na[PW], nb[PW];
#pragma unroll
  for (int p = 0; p < PW; ++p) {
    na[p] = qs[q4 * QPB + cbi[p]];
    nb[p] = qs[q4 * QPB + cbj[p]];
  }
  for (int r = q4; r < Ns4; r += 4) {
    uint16_t ca[PW], cb[PW];
#pragma unroll
    for (int p = 0; p < PW; ++p) { ca[p] = na[p]; cb[p] = nb[p]; }
    const uint16_t* nrow = qs + min(r + 4, Ns4 - 4 + q4) * QPB;
#pragma unroll
    for (int p = 0; p < PW; ++p) {
      na[p] = nrow[cbi[p]];
      nb[p] = nrow[cbj[p]];
    }
    __builtin_amdgcn_sched_barrier(0);  // the next group's reads stay ahead of these MFMAs
    const double live = r < Ns ? 1.0 : 0.0;  // a factor, not a branch
#pragma unroll
    for (int p = 0; p < PW; ++p) {
      const double xa = ((double)bf16_to_f32(ca[p]) - mbi[p]) * live;
      const double xb = (double)bf16_to_f32(cb[p]) - mbj[p];
      acc[p] = mfma64(xa, xb, acc[p]);
    }
  }
  // Lambda_Q[row][col] (row >= col) goes to the reversed matrix at
  // (d-1-col, d-1-row), a lower entry; diagonal blocks are written whole.
  const double invn = 1.0 / (double)Ns;
#pragma unroll
  for (int p = 0; p < PW; ++p) {
    const int e = wave + NW * p;
    if (e < NPAIR) {
      int bi, bj;
      tri_index(e, bi, bj);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * bi + 4 * i + q4, col = 16 * bj + r16;
        A[lidx(D - 1 - col, D - 1 - row)] = acc[p][i] * invn;
      }
    }
  }
  __syncthreads();
  for (int a = tid; a < D; a += kFactorThreads) dg[a] = A[lidx(a, a)];
  __syncthreads();
  if (cholesky_lds<D, kFactorThreads, false, false>(A, dg, &bad, kPivRelTri, (int)kUnitKTile) != 0) {
    if (tid == 0) atomicOr(uflags + u, kUnitKTile);
    return;
  }
  store_lower_frags<D>(xfrag + (int64_t)u * lower_frag_elems(D),
                       [&](int a, int b) { return A[lidx(D - 1 - b, D - 1 - a)]; });
}

// One workgroup per unit (a grid-stride walk if the grid is smaller).
template <int D>
__global__ __launch_bounds__(kFactorThreads) void qfactor_kernel(Geo g, const uint16_t* __restrict__ q,
                                                                 const double* __restrict__ mu,
                                                                 uint16_t* __restrict__ xfrag,
                                                                 uint32_t* __restrict__ uflags) {
  for (int u = blockIdx.x; u < g.U; u += gridDim.x) {
    qfactor_unit<D>(g, u, q, mu, xfrag, uflags);
    __syncthreads();  // LDS of this unit fully consumed before the next one's
  }
}

hipError_t launch_qfactor(const Launch& L, const void* q) {
  const Geo& g = L.geo;
  if (g.U == 0) return hipSuccess;
  // The fragments go to the L^{-1} fragment section, which every layout that
  // can take this path reserves (offset 0 is the status word's).
  if (L.ws.lfrag == 0) return hipErrorInvalidValue;
  auto go = [&](auto kern) {
    kern<<<g.U, kFactorThreads, 0, L.stream>>>(g, (const uint16_t*)q,
                                                ws_ptr<double>(L.wsp, L.ws.mu),
                                                ws_ptr<uint16_t>(L.wsp, L.ws.lfrag),
                                                ws_ptr<uint32_t>(L.wsp, L.ws.uflags));
  };
  if (g.D == 128) go(qfactor_kernel<128>);
  else go(qfactor_kernel<64>);
  return hipGetLastError();
}

}  // namespace jacap
