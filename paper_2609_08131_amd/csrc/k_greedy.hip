// Exact greedy log-det selection (App. B.1): the sequential maximisation that
// the one-shot leverage ranking of Eq. 10 approximates, kept as a quality
// comparator for TOP-B.
//
// Per unit, with the Eq. 8 weights w_i and u_i = v_i, the greedy adds B times
// the token with the largest gain w_i c_i, c_i = u_i^T A_C^{-1} u_i, where
// A_C = ridge I + sum_{j in C} w_j u_j u_j^T (by the matrix determinant lemma
// the log-det increase is log(1 + w_i c_i), increasing in w_i c_i); ties go to
// the lowest position. After a pick s, Sherman-Morrison gives
// A^{-1} <- A^{-1} - g g^T with g = A^{-1} u_s sqrt(w_s / (1 + w_s c_s)).
//
// GPU design (one workgroup of 256 threads per unit):
// * A^{-1} (d x d, fp64) is held in registers: thread t owns row t / TPR and a
//   contiguous run of d / TPR columns (TPR = 256 / d). c = u^T A^{-1} u and
//   A^{-1} u cost d^2 FMA spread over the workgroup.
// * Gains never grow as C grows (each pick lowers c_i by (u_i . g)^2), so a
//   c_i computed after fewer picks bounds the current one from above (lazy
//   greedy, after Minoux). Per token the workspace keeps c_i and the number of
//   picks made when it was computed (its stamp; -1 = taken); per block of 256
//   positions an LDS entry keeps the block's best (key w_i c_i, c_i, position,
//   stamp). Each round wave 0 finds the best entry: if its stamp is current
//   the token is taken, else its c is recomputed and the block rescanned. The
//   token taken is the eager greedy's: every other token's current gain is at
//   most its key, and equal keys resolve by position.
// * Token i's workspace state is read and written only by lane i % 64 of wave
//   0 inside the kernel (the initial values come from the previous launch), so
//   every read sees that lane's own earlier writes.
// * The initial pass (c_i = ||u_i||^2 / ridge, stamp 0, and the block
//   entries) streams V once with many workgroups per unit.
// * Units whose keys w_i c_i fit in LDS take greedy_lds_kernel (below), the
//   same lazy search with a shorter round.
#include <float.h>

#include "jacap_internal.hpp"

namespace jacap {

namespace {

constexpr int kGBlock = 256;            // positions per tournament block
constexpr int kGMaxBlocks = kGreedyMaxLen / kGBlock;
constexpr int kGMaxWords = kGreedyMaxLen / 32;
constexpr int kGSlots = kGBlock / 64;   // positions per lane in a block scan

constexpr int kOpStop = 0, kOpRefresh = 1, kOpPick = 2;

// Ordering key of a gain; NaN and -inf (untaken) sort just above a taken
// token's -inf, so the search never returns a taken token while one is left.
__device__ __forceinline__ double gain_key(float w, double c) {
  const double x = (double)w * c;
  return x >= -DBL_MAX ? x : -DBL_MAX;
}

// (key, position) lexicographic: larger key first, then lower position.
__device__ __forceinline__ void take_better(double& k, int& p, double k2, int p2) {
  if (k2 > k || (k2 == k && p2 < p)) {
    k = k2;
    p = p2;
  }
}

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

// Wave64 arg-max of (key, position); every lane ends with the same result.
__device__ __forceinline__ void wave_argmax(double& k, int& p) {
  take_better(k, p, dpp_f64<kDppQuadXor1>(k), dpp_i32<kDppQuadXor1>(p));
  take_better(k, p, dpp_f64<kDppQuadXor2>(k), dpp_i32<kDppQuadXor2>(p));
  take_better(k, p, dpp_f64<kDppHalfMirror>(k), dpp_i32<kDppHalfMirror>(p));
  take_better(k, p, dpp_f64<kDppMirror>(k), dpp_i32<kDppMirror>(p));
  take_better(k, p, __shfl_xor(k, 16), __shfl_xor(p, 16));
  take_better(k, p, __shfl_xor(k, 32), __shfl_xor(p, 32));
}

// Sum over each 16-lane row (every lane of the row ends with the same value).
__device__ __forceinline__ double row_sum16(double v) {
  v += dpp_f64<kDppQuadXor1>(v);
  v += dpp_f64<kDppQuadXor2>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  v += dpp_f64<kDppMirror>(v);
  return v;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
  v = row_sum16(v);
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

template <typename X>
__device__ __forceinline__ X pick4(const X (&a)[kGSlots], int m) {
  return m == 0 ? a[0] : m == 1 ? a[1] : m == 2 ? a[2] : a[3];
}

// N consecutive elements (16-byte aligned for N * sizeof(T) == 16) as floats.
template <typename T, int N>
__device__ __forceinline__ void load_elems(const T* p, float (&x)[N]) {
  if constexpr (sizeof(T) == 2) {
    static_assert(N == 4 || N == 8, "bf16 chunk");
    if constexpr (N == 8) {
      const uint4 r = *reinterpret_cast<const uint4*>(p);
      const uint32_t wd[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[2 * i] = bf16_to_f32((uint16_t)(wd[i] & 0xFFFFu));
        x[2 * i + 1] = bf16_to_f32((uint16_t)(wd[i] >> 16));
      }
    } else {
      const uint2 r = *reinterpret_cast<const uint2*>(p);
      const uint32_t wd[2] = {r.x, r.y};
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x[2 * i] = bf16_to_f32((uint16_t)(wd[i] & 0xFFFFu));
        x[2 * i + 1] = bf16_to_f32((uint16_t)(wd[i] >> 16));
      }
    }
  } else {
    static_assert(N % 4 == 0, "fp32 chunk");
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
      const float4 r = reinterpret_cast<const float4*>(p)[i];
      x[4 * i] = r.x;
      x[4 * i + 1] = r.y;
      x[4 * i + 2] = r.z;
      x[4 * i + 3] = r.w;
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Initial pass: c_i = ||v_i||^2 / ridge (A_0 = ridge I), stamp 0, and each
// block's best entry. One workgroup per (block of 256 positions, unit); 16
// lanes per token, each summing d/16 squares.
// ---------------------------------------------------------------------------
template <int D, typename T>
__global__ __launch_bounds__(kThreads) void greedy_init_kernel(
    Geo g, const T* __restrict__ v, const float* __restrict__ wgt, float ridge,
    const double* __restrict__ wscale, int budget,
    int protect, double* __restrict__ gc, int32_t* __restrict__ gst,
    GreedyEntry* __restrict__ entries, int nblk_max) {
  constexpr int EPL = D / 16;
  __shared__ double rk[4], rc[4];
  __shared__ int rp[4];
  const int u = blockIdx.y, blk = blockIdx.x;
  const Unit un = decode_unit(g, u);
  const int i0 = blk * kGBlock;
  if (i0 >= un.n) return;
  const int kk = min(budget, un.n), p = min(protect, kk), nfree = un.n - p;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = lane >> 4, rl = lane & 15;
  const T* vb = v + (int64_t)un.l * g.vsl + (int64_t)un.h * g.vsh + un.t0 * g.vst;
  const int64_t trow = token_row(g, un);

  // Iteration it handles positions i0 + 64 wave + 4 it + row; lane rl == it
  // keeps that sum, so lane (row, rl) ends with position i0 + 64 wave + 4 rl + row.
  float x[16][EPL];
#pragma unroll
  for (int it = 0; it < 16; ++it) {
    const int i = min(i0 + wave * 64 + it * 4 + row, un.n - 1);
    load_elems<T, EPL>(vb + (int64_t)i * g.vst + rl * EPL, x[it]);
  }
  double mine = 0.0;
#pragma unroll
  for (int it = 0; it < 16; ++it) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < EPL; ++e) s = fma((double)x[it][e], (double)x[it][e], s);
    s = row_sum16(s);
    if (rl == it) mine = s;
  }
  const int i = i0 + wave * 64 + rl * 4 + row;
  const double c = mine / ((double)ridge * wscale[u]);  // the stored weights' scale
  double key = -__builtin_inf();
  int pos = INT32_MAX;
  if (i < un.n) {
    gc[trow + i] = c;
    gst[trow + i] = 0;
    if (i < nfree) {
      key = gain_key(wgt[trow + i], c);
      pos = i;
    }
  }
  const double mykey = key;
  const int mypos = pos;
  wave_argmax(key, pos);
  if (pos == INT32_MAX) {
    if (lane == 0) { rk[wave] = key; rc[wave] = 0.0; rp[wave] = INT32_MAX; }
  } else if (mypos == pos && mykey == key) {
    rk[wave] = key; rc[wave] = c; rp[wave] = pos;
  }
  __syncthreads();
  if (tid == 0) {
    double bk = rk[0], bc = rc[0];
    int bp = rp[0];
    for (int j = 1; j < 4; ++j)
      if (rk[j] > bk || (rk[j] == bk && rp[j] < bp)) { bk = rk[j]; bc = rc[j]; bp = rp[j]; }
    GreedyEntry e;
    e.key = bk; e.c = bc; e.pos = bp; e.stamp = 0;
    entries[(int64_t)u * nblk_max + blk] = e;
  }
}

// ---------------------------------------------------------------------------
// The greedy itself: one workgroup per unit.
// ---------------------------------------------------------------------------
struct GreedyShared {
  GreedyEntry ent[kGMaxBlocks];
  uint32_t bits[kGMaxWords];  // taken positions
  double us[kGreedyMaxD];     // the current token's u (fp64)
  double gs[kGreedyMaxD];     // g of the last pick
  double red[4];
  double f;                   // sqrt(w / (1 + w c)) of a pick (or w of a forced pick)
  int op, pos;
  uint32_t scan[5];
};

template <int D, typename T>
__global__ __launch_bounds__(kThreads) void greedy_kernel(
    Geo g, const T* __restrict__ v, const float* __restrict__ wgt, float ridge_f,
    const double* __restrict__ wscale, int budget,
    int protect, double* __restrict__ gc, int32_t* __restrict__ gst,
    const GreedyEntry* __restrict__ entries, int nblk_max, int32_t* __restrict__ idx_out,
    int32_t* __restrict__ order_out, double* __restrict__ logdet_out) {
  constexpr int TPR = kThreads / D;     // threads per row of A^{-1}
  constexpr int NA = D / TPR;           // entries of A^{-1} per thread
  constexpr int EPL = 16 / sizeof(T);   // elements per 16-byte row piece
  constexpr int ROWL = D / EPL;         // lanes fetching one row
  static_assert(TPR == 2 || TPR == 4, "head_dim 64 or 128");
  __shared__ __align__(16) GreedyShared sh;

  const int u = blockIdx.x;
  const Unit un = decode_unit(g, u);
  const int n = un.n;
  const int kk = min(budget, n), p = min(protect, kk), nfree = n - p;
  const int nblk = (n + kGBlock - 1) / kGBlock, words = (n + 31) / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = tid / TPR, q = tid % TPR;
  // A_0 = ridge I times the stored weights' scale (gains are unchanged by it)
  const double ridge = (double)ridge_f * (n > 0 ? wscale[u] : 1.0);
  const T* vb = v + (int64_t)un.l * g.vsl + (int64_t)un.h * g.vsh + un.t0 * g.vst;
  const int64_t trow = token_row(g, un);

  double ainv[NA];
#pragma unroll
  for (int m = 0; m < NA; ++m) ainv[m] = (q * NA + m == r) ? 1.0 / ridge : 0.0;
  for (int j = tid; j < nblk; j += kThreads) sh.ent[j] = entries[(int64_t)u * nblk_max + j];
  for (int j = tid; j < words; j += kThreads) sh.bits[j] = 0u;

  // Row i of V into sh.us (wave 0, lanes < ROWL).
  auto fetch_row = [&](int i) {
    if (lane < ROWL) {
      float x[EPL];
      load_elems<T, EPL>(vb + (int64_t)i * g.vst + lane * EPL, x);
#pragma unroll
      for (int e = 0; e < EPL; ++e) sh.us[lane * EPL + e] = (double)x[e];
    }
  };
  // (A^{-1} u)_r restricted to this thread's columns.
  auto row_partial = [&]() {
    const double2* u2 = reinterpret_cast<const double2*>(sh.us + q * NA);
    double a = 0.0;
#pragma unroll
    for (int m = 0; m < NA / 2; ++m) {
      const double2 x = u2[m];
      a = fma(ainv[2 * m], x.x, a);
      a = fma(ainv[2 * m + 1], x.y, a);
    }
    return a;
  };
  // c = u^T A^{-1} u over the workgroup (one barrier).
  auto quad_form = [&](double partial) {
    const double s = wave_sum_f64(sh.us[r] * partial);
    if (lane == 0) sh.red[wave] = s;
    __syncthreads();
    return ((sh.red[0] + sh.red[1]) + sh.red[2]) + sh.red[3];
  };
  // A^{-1} <- A^{-1} - g g^T, g = (A^{-1} u) f (one barrier).
  auto downdate = [&](double partial, double f) {
    double h = partial + dpp_f64<kDppQuadXor1>(partial);
    if constexpr (TPR == 4) h += dpp_f64<kDppQuadXor2>(h);
    const double gr = h * f;
    if (q == 0) sh.gs[r] = gr;
    __syncthreads();
    const double2* g2 = reinterpret_cast<const double2*>(sh.gs + q * NA);
#pragma unroll
    for (int m = 0; m < NA / 2; ++m) {
      const double2 x = g2[m];
      ainv[2 * m] = fma(-gr, x.x, ainv[2 * m]);
      ainv[2 * m + 1] = fma(-gr, x.y, ainv[2 * m + 1]);
    }
  };

  int32_t* order = order_out ? order_out + (int64_t)u * budget : nullptr;
  double logdet = 0.0;  // sum of log(1 + w c) over the picks (wave 0)
  int t = 0;
  __syncthreads();

  // Protected positions: taken first, in position order (outside the search).
  for (; t < p; ++t) {
    const int s = nfree + t;
    if (wave == 0) {
      fetch_row(s);
      if (lane == 0) sh.f = (double)wgt[trow + s];
    }
    __syncthreads();
    const double partial = row_partial();
    const double w = sh.f;
    const double c = quad_form(partial);
    downdate(partial, sqrt(w / (1.0 + w * c)));
    if (tid == 0) {
      logdet += log1p(w * c);
      sh.bits[s >> 5] |= 1u << (s & 31);
      if (order) order[t] = s;
    }
  }

  // Lazy greedy over positions [0, nfree).
  int cblk = -1, utok = -1;
  double bc[kGSlots];
  int bst[kGSlots];
  float bw[kGSlots];
#pragma unroll
  for (int j = 0; j < kGSlots; ++j) { bc[j] = 0.0; bst[j] = -1; bw[j] = 0.0f; }
  double pick_gain = 0.0;

  // Best entry of block cblk from the registers (wave 0).
  auto rescan = [&]() {
    double bk = -__builtin_inf();
    int bp = INT32_MAX;
#pragma unroll
    for (int j = 0; j < kGSlots; ++j) {
      const int i = cblk * kGBlock + j * 64 + lane;
      if (i < nfree && bst[j] >= 0) take_better(bk, bp, gain_key(bw[j], bc[j]), i);
    }
    wave_argmax(bk, bp);
    if (bp == INT32_MAX) {
      if (lane == 0) {
        GreedyEntry e;
        e.key = bk; e.c = 0.0; e.pos = INT32_MAX; e.stamp = 0;
        sh.ent[cblk] = e;
      }
    } else if (lane == (bp & 63)) {
      const int j = (bp & (kGBlock - 1)) >> 6;
      GreedyEntry e;
      e.key = bk; e.c = pick4(bc, j); e.pos = bp; e.stamp = pick4(bst, j);
      sh.ent[cblk] = e;
    }
  };

  while (t < kk) {
    if (wave == 0) {
      double bk = -__builtin_inf();
      int bp = INT32_MAX;
      for (int j = lane; j < nblk; j += 64) take_better(bk, bp, sh.ent[j].key, sh.ent[j].pos);
      wave_argmax(bk, bp);
      int op = kOpStop;
      if (bp < nfree) {
        const int b = bp / kGBlock;
        const GreedyEntry e = sh.ent[b];
        op = e.stamp == t ? kOpPick : kOpRefresh;
        if (b != cblk) {
#pragma unroll
          for (int j = 0; j < kGSlots; ++j) {
            const int i = b * kGBlock + j * 64 + lane;
            if (i < n) {
              bc[j] = gc[trow + i];
              bst[j] = gst[trow + i];
              bw[j] = wgt[trow + i];
            } else {
              bc[j] = 0.0; bst[j] = -1; bw[j] = 0.0f;
            }
          }
          cblk = b;
        }
        if (bp != utok) {
          fetch_row(bp);
          utok = bp;
        }
        if (op == kOpPick) {
          const int j = (bp & (kGBlock - 1)) >> 6;
          const double w = (double)__shfl(pick4(bw, j), bp & 63);
          pick_gain = w * e.c;
          if (lane == 0) sh.f = sqrt(w / (1.0 + pick_gain));
        }
      }
      if (lane == 0) { sh.op = op; sh.pos = bp; }
    }
    __syncthreads();
    const int op = sh.op, s = sh.pos;
    if (op == kOpStop) break;  // unreachable: an untaken position always remains
    const double partial = row_partial();
    if (op == kOpRefresh) {
      const double c = quad_form(partial);
      if (wave == 0) {
        const int j = (s & (kGBlock - 1)) >> 6;
        if (lane == (s & 63)) {
#pragma unroll
          for (int jj = 0; jj < kGSlots; ++jj)
            if (jj == j) { bc[jj] = c; bst[jj] = t; }
          gc[trow + s] = c;
          gst[trow + s] = t;
        }
        rescan();
      }
    } else {
      downdate(partial, sh.f);
      if (wave == 0) {
        const int j = (s & (kGBlock - 1)) >> 6;
        if (lane == (s & 63)) {
#pragma unroll
          for (int jj = 0; jj < kGSlots; ++jj)
            if (jj == j) bst[jj] = -1;
          gst[trow + s] = -1;
        }
        rescan();
        if (lane == 0) {
          logdet += log1p(pick_gain);
          sh.bits[s >> 5] |= 1u << (s & 31);
          if (order) order[t] = s;
        }
      }
      ++t;
    }
  }
  __syncthreads();

  // Kept positions in ascending order from the bitmap.
  const int per = (words + kThreads - 1) / kThreads;
  const int w0 = min(tid * per, words), w1 = min(w0 + per, words);
  uint32_t cnt = 0;
  for (int j = w0; j < w1; ++j) cnt += __popc(sh.bits[j]);
  uint32_t incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) sh.scan[wave] = incl;
  __syncthreads();
  uint32_t off = incl - cnt;
  for (int j = 0; j < wave; ++j) off += sh.scan[j];
  int32_t* out = idx_out + (int64_t)u * budget;
  for (int j = w0; j < w1; ++j) {
    uint32_t x = sh.bits[j];
    while (x) {
      const int bit = __ffs(x) - 1;
      out[off++] = j * 32 + bit;
      x &= x - 1u;
    }
  }
  for (int j = t + tid; j < budget; j += kThreads) {
    out[j] = -1;
    if (order) order[j] = -1;
  }
  if (logdet_out && tid == 0) logdet_out[u] = (double)D * log((double)ridge_f) + logdet;
}

// ---------------------------------------------------------------------------
// The same search with the unit's keys w_i c_i and weights in LDS (12 bytes per
// token and one row per block: up to 12032 tokens of bf16 rows at d = 128). What bounds it is the latency of
// one round -- find the best entry, form u^T A^{-1} u, rank the block again --
// times B picks of about two refreshes each, so a round is made of as few
// dependent steps as possible:
// * Every wave finds the best entry, re-ranks the block and updates its own copy of
//   the search state (the block entries, lane b holding block b's, and the
//   tokens refreshed since the last pick, in registers); only the quadratic
//   form (or the pick's g) crosses the waves, at one LDS-only barrier per round.
//   The keys in LDS are written by every wave, with the same values: a wave's
//   writes of a round precede its arrival at the next barrier, and no wave
//   writes the next round's values before that barrier, so a late wave repeats
//   a value and never restores an old one. What crosses the barrier is
//   double-buffered.
// * Four waves, one per SIMD (with eight, the steps that every wave repeats
//   take twice the issue slots: 2.20 against 2.05 ms).
// * A thread owns RPT rows x 4 columns of A^{-1}: it needs RPT + 4 elements of u
//   (against 1 + d / 2 for a piece of one row), taken straight from V's row.
// * The rows of V of every block's best token are kept in LDS: when a block's
//   best changes its row is requested at once, by the waves in turn, and written
//   kRowDelay rounds later, so that no round waits for it; a row needed
//   before that is read directly. A token picked right after its refresh
//   reuses A^{-1} u.
// * Keys are kept as order-preserving integers: maxima are taken on their high
//   words (one DPP instruction per level, scalar ones across the rows), the low
//   words only if several lanes hold that maximum.
// * Gains are kept (over the unit's c_i, which the LDS keys replace; 64 of them in
//   registers before a store) and their logarithms summed at the end by all
//   threads.
//
// Measured (MI355X, one layer of 8 units x 8192 tokens, d = 128, B = 512): 5.54
// ms with the keys in global memory and three barriers per round, 2.05 ms
// here. Longer units, whose keys do not fit, keep the kernel above.
// ---------------------------------------------------------------------------
constexpr size_t kGLdsMax = 156 * 1024;  // of the 160 KB; the kernel's fixed arrays take the rest
constexpr int kRowDelay = 3;             // rounds from a row's request to its place in LDS

// Bytes of LDS per block of 256 tokens: keys, weights, the bitmap of taken
// tokens, the row of the block's best token.
__host__ __device__ constexpr size_t greedy_lds_bytes(int row_bytes) {
  return (size_t)kGBlock * 12 + kGBlock / 8 + row_bytes;
}

// A gain as an integer of the same order (larger gain, larger integer); -0 as +0.
// kTakenKey lies below every gain.
constexpr int64_t kTakenKey = INT64_MIN;
__device__ __forceinline__ int64_t order_key(double x) {
  const int64_t b = __builtin_bit_cast(int64_t, x + 0.0);
  return b ^ ((b >> 63) & INT64_MAX);
}
__device__ __forceinline__ double key_gain(int64_t k) {
  return __builtin_bit_cast(double, k ^ ((k >> 63) & INT64_MAX));
}

// Maximum over the wave, the same in every lane: each row by DPP, then the rows.
template <typename I>
__device__ __forceinline__ I wave_max_int(I v) {
  v = max(v, (I)dpp_i32<kDppQuadXor1>((int)v));
  v = max(v, (I)dpp_i32<kDppQuadXor2>((int)v));
  v = max(v, (I)dpp_i32<kDppHalfMirror>((int)v));
  v = max(v, (I)dpp_i32<kDppMirror>((int)v));
  auto at = [&](int l) { return (I)__builtin_amdgcn_readlane((int)v, l); };
  return max(max(at(0), at(16)), max(at(32), at(48)));
}
// The lanes holding the wave's largest key, and that key.
__device__ __forceinline__ uint64_t wave_max_lanes(int64_t k, int64_t& best) {
  const int hi = (int)(k >> 32);
  const uint32_t lo = (uint32_t)k;
  const int mh = wave_max_int(hi);
  uint64_t bm = __ballot(hi == mh);
  uint32_t ml;
  if (bm & (bm - 1)) {  // uniform
    ml = wave_max_int(hi == mh ? lo : 0u);
    bm &= __ballot(lo == ml);
  } else {
    ml = (uint32_t)__builtin_amdgcn_readlane((int)lo, __builtin_ctzll(bm));
  }
  best = (int64_t)(((uint64_t)(uint32_t)mh << 32) | ml);
  return bm;
}
__device__ __forceinline__ double row_lane_f64(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_rows(double v) {
  v = row_sum16(v);
  return ((row_lane_f64(v, 0) + row_lane_f64(v, 16)) + row_lane_f64(v, 32)) + row_lane_f64(v, 48);
}

// Workgroup barrier that orders LDS only (global stores stay in flight).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kGLdsThreads = 256;

template <int D, typename T>
__global__ __launch_bounds__(kGLdsThreads) void greedy_lds_kernel(
    Geo g, const T* __restrict__ v, const float* __restrict__ wgt, float ridge_f,
    const double* __restrict__ wscale, int budget, int protect, double* __restrict__ gc,
    const GreedyEntry* __restrict__ entries, int nblk_max, int32_t* __restrict__ idx_out,
    int32_t* __restrict__ order_out, double* __restrict__ logdet_out) {
  constexpr int NT = kGLdsThreads, NW = NT / 64;
  constexpr int CPT = 4;                      // columns of A^{-1} per thread
  constexpr int CG = D / CPT;                 // threads along a row of blocks (lanes)
  constexpr int RPT = D * D / NT / CPT;       // rows per thread: 16 (d = 128) or 4
  static_assert(RPT * CPT * NT == D * D && 64 % CG == 0, "whole tiles");
  extern __shared__ __align__(16) char lds[];
  int64_t* key = reinterpret_cast<int64_t*>(lds);
  float* ws = reinterpret_cast<float*>(lds + (size_t)nblk_max * kGBlock * 8);
  uint32_t* bits = reinterpret_cast<uint32_t*>(lds + (size_t)nblk_max * kGBlock * 12);
  T* rows = reinterpret_cast<T*>(bits + nblk_max * (kGBlock / 32));  // [block][D]
  __shared__ __align__(16) double gs[2][D];
  __shared__ __align__(16) double red[2][NW];
  __shared__ uint32_t scan[NW];

  const int u = blockIdx.x;
  const Unit un = decode_unit(g, u);
  const int n = un.n;
  const int kk = min(budget, n), p = min(protect, kk), nfree = n - p;
  const int nblk = (n + kGBlock - 1) / kGBlock, words = nblk * (kGBlock / 32);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = tid / CG * RPT, c0 = lane % CG * CPT;
  // A_0 = ridge I times the stored weights' scale (gains are unchanged by it)
  const double ridge = (double)ridge_f * (n > 0 ? wscale[u] : 1.0);
  const T* vb = v + (int64_t)un.l * g.vsl + (int64_t)un.h * g.vsh + un.t0 * g.vst;
  const int64_t trow = token_row(g, un);
  double* gain_out = gc + trow;   // gain of pick t (after the keys are in LDS)

  for (int i = tid; i < nblk * kGBlock; i += NT) {
    const float w = i < n ? wgt[trow + i] : 0.0f;
    ws[i] = w;
    key[i] = i < nfree ? order_key(gain_key(w, gc[trow + i])) : kTakenKey;
  }
  for (int j = tid; j < words; j += NT) bits[j] = 0u;
  // Lane b: block b's best key, its position, and the number of picks when it was
  // computed if that is known (every c_i is current before the first pick).
  int64_t ek = kTakenKey;
  int ep = INT32_MAX, es = -1;
  if (lane < nblk) {
    const GreedyEntry e = entries[(int64_t)u * nblk_max + lane];
    if (e.pos != INT32_MAX) ek = order_key(e.key);
    ep = e.pos;
    es = p == 0 ? 0 : -1;
  }
  constexpr int PIECES = D * sizeof(T) / 16;  // 16-byte pieces of a row
  for (int e = tid; e < nblk * PIECES; e += NT) {
    const int b = e / PIECES, pc = e % PIECES;
    const int s = entries[(int64_t)u * nblk_max + b].pos;
    if ((unsigned)s < (unsigned)n)
      reinterpret_cast<uint4*>(rows)[e] =
          *(reinterpret_cast<const uint4*>(vb + (int64_t)s * g.vst) + pc);
  }
  double ainv[RPT][CPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int j = 0; j < CPT; ++j) ainv[i][j] = r0 + i == c0 + j ? 1.0 / ridge : 0.0;
  __syncthreads();

  // This thread's elements of a row of V (columns c0 .., rows r0 ..).
  struct Row { double c[CPT], r[RPT]; };
  auto load_rows = [&](const T* p, float (&r)[RPT]) {
    constexpr int STEP = RPT > 8 ? 8 : RPT;
#pragma unroll
    for (int i = 0; i < RPT; i += STEP) {
      float y[STEP];
      load_elems<T, STEP>(p + i, y);
#pragma unroll
      for (int j = 0; j < STEP; ++j) r[i + j] = y[j];
    }
  };
  auto row = [&](const T* vr) {
    float c[CPT], r[RPT];
    load_elems<T, CPT>(vr + c0, c);
    load_rows(vr + r0, r);
    Row x;
#pragma unroll
    for (int j = 0; j < CPT; ++j) x.c[j] = (double)c[j];
#pragma unroll
    for (int i = 0; i < RPT; ++i) x.r[i] = (double)r[i];
    return x;
  };
  // (A^{-1} u) restricted to this thread's columns, for its rows.
  auto partial = [&](const Row& x, double (&h)[RPT]) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) h[i] = ainv[i][0] * x.c[0];
#pragma unroll
    for (int j = 1; j < CPT; ++j)
#pragma unroll
      for (int i = 0; i < RPT; ++i) h[i] = fma(ainv[i][j], x.c[j], h[i]);
  };
  int par = 0;
  // u^T A^{-1} u over the workgroup (one barrier).
  auto quad_form = [&](const Row& x, const double (&h)[RPT]) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < RPT; i += 2) {
      s0 = fma(x.r[i], h[i], s0);
      s1 = fma(x.r[i + 1], h[i + 1], s1);
    }
    const double s = wave_sum_rows(s0 + s1);
    if (lane == 0) red[par][wave] = s;
    lds_barrier();
    double c[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) c[i] = red[par][i];
#pragma unroll
    for (int o = NW / 2; o > 0; o /= 2)
#pragma unroll
      for (int i = 0; i < o; ++i) c[i] += c[i + o];
    par ^= 1;
    return c[0];
  };
  // A^{-1} <- A^{-1} - g g^T, g = (A^{-1} u) f (one barrier).
  auto downdate = [&](const double (&h)[RPT], double f) {
    // Sum of h over the CG lanes of a row group: transposing steps (the row
    // mirror, the half-row mirror, a quad swap) leave one row per lane, plain
    // steps finish.
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
    double hv;
    int rl;
    if constexpr (RPT == 16) {
      const bool b0 = lane & 1;
      double a[8], b[4], c[2];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        a[i] = (b3 ? h[8 + i] : h[i]) + dpp_f64<kDppMirror>(b3 ? h[i] : h[8 + i]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        b[i] = (b2 ? a[4 + i] : a[i]) + dpp_f64<kDppHalfMirror>(b2 ? a[i] : a[4 + i]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        c[i] = (b1 ? b[2 + i] : b[i]) + dpp_f64<kDppQuadXor2>(b1 ? b[i] : b[2 + i]);
      hv = (b0 ? c[1] : c[0]) + dpp_f64<kDppQuadXor1>(b0 ? c[0] : c[1]);
      hv += __shfl_xor(hv, 16);  // CG = 32
      rl = (b3 ? 8 : 0) + (b2 ? 4 : 0) + (b1 ? 2 : 0) + (b0 ? 1 : 0);
    } else {
      double a[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        a[i] = (b3 ? h[2 + i] : h[i]) + dpp_f64<kDppMirror>(b3 ? h[i] : h[2 + i]);
      hv = (b2 ? a[1] : a[0]) + dpp_f64<kDppHalfMirror>(b2 ? a[0] : a[1]);
      hv += dpp_f64<kDppQuadXor2>(hv);
      hv += dpp_f64<kDppQuadXor1>(hv);  // CG = 16
      rl = (b3 ? 2 : 0) + (b2 ? 1 : 0);
    }
    gs[par][r0 + rl] = hv * f;  // lanes of one row write the same value
    lds_barrier();
    double gr[RPT], gcol[CPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) gr[i] = gs[par][r0 + i];
#pragma unroll
    for (int j = 0; j < CPT; ++j) gcol[j] = gs[par][c0 + j];
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int j = 0; j < CPT; ++j) ainv[i][j] = fma(-gr[i], gcol[j], ainv[i][j]);
    par ^= 1;
  };

  int32_t* order = order_out ? order_out + (int64_t)u * budget : nullptr;
  int t = 0;
  // Wave 0 records pick t: lane t % 64 holds it until 64 are stored together.
  double held_gain = 0.0;
  int held_pos = 0;
  auto store_held = [&](int first, int count) {
    if (lane < count) {
      gain_out[first + lane] = held_gain;
      if (order) order[first + lane] = held_pos;
    }
  };
  auto took = [&](int s, double gain) {
    if (wave != 0) return;
    if (lane == (t & 63)) { held_gain = gain; held_pos = s; }
    if (lane == 0) bits[s >> 5] |= 1u << (s & 31);
    if ((t & 63) == 63) store_held(t - 63, 64);
  };
  // Protected positions: taken first, in position order (outside the search).
  for (; t < p; ++t) {
    const int s = nfree + t;
    const Row x = row(vb + (int64_t)s * g.vst);
    double h[RPT];
    partial(x, h);
    const double w = (double)ws[s];
    const double c = quad_form(x, h);
    downdate(h, sqrt(w / (1.0 + w * c)));
    took(s, w * c);
  }

  // Lazy greedy over positions [0, nfree).
  Row x{};
  double h[RPT];
  int last = -1;            // the token of x and h, while they hold
  int asked = -2 * kRowDelay;  // lane b: the round in which block b's row was last requested
  uint4 pend{};             // a requested row (16 bytes per lane), its block and round
  int pend_b = 0, pend_at = -2 * kRowDelay;
  // The tokens refreshed since the last pick, one per lane, the oldest
  // overwritten: a forgotten one is refreshed again (to the same key) and is then
  // known, so the search still ends.
  int fresh = -1, nfresh = 0;
  drain_vmem();  // no prologue load is waited for (with the requested rows) in the loop
  for (int round = 0; t < kk; ++round) {
    int64_t top;
    // entries are in position order: the first one holding the maximum
    const int b = __builtin_ctzll(wave_max_lanes(ek, top));
    const int s = __builtin_amdgcn_readlane(ep, b);
    const int stamp = __builtin_amdgcn_readlane(es, b);
    if ((unsigned)s >= (unsigned)nfree) break;  // unreachable: an untaken position always remains
    const double w = (double)ws[s];
    int64_t k4[kGSlots];
    const int i0 = b * kGBlock;
#pragma unroll
    for (int j = 0; j < kGSlots; ++j) k4[j] = key[i0 + j * 64 + lane];
    if (s != last) {
      // in LDS since the barrier of round asked + kRowDelay
      if (__builtin_amdgcn_readlane(asked, b) + kRowDelay < round) {
        x = row(rows + b * D);
      } else {
        x = row(vb + (int64_t)s * g.vst);
        drain_vmem();  // waited for here: the other branch leaves requested rows in flight
      }
      partial(x, h);
    }
    if (pend_at + kRowDelay == round && lane < PIECES)
      reinterpret_cast<uint4*>(rows)[pend_b * PIECES + lane] = pend;
    int64_t nk;  // the token's new key
    const bool pick = stamp == t;
    last = pick ? -1 : s;
    if (pick) {
      const double gain = key_gain(top);  // w c
      downdate(h, sqrt(w / (1.0 + gain)));
      took(s, gain);
      nk = kTakenKey;
      ++t;
      fresh = -1;  // no c is current any more
      nfresh = 0;
    } else {
      nk = order_key(gain_key((float)w, quad_form(x, h)));
      if (lane == (nfresh & 63)) fresh = s;
      ++nfresh;
    }
    // The block's best: the token's key replaced, the lowest position of the
    // largest key.
    int64_t m = kTakenKey;
    int mj = 0;
#pragma unroll
    for (int j = 0; j < kGSlots; ++j) {
      const int64_t kj = i0 + j * 64 + lane == s ? nk : k4[j];
      const bool gt = kj > m;
      m = gt ? kj : m;
      mj = gt ? j : mj;
    }
    if (lane == 0) key[s] = nk;
    int64_t mk;
    const uint64_t hit = wave_max_lanes(m, mk);
    int at = INT32_MAX;
    if (mk != kTakenKey) {
      const int mp = i0 + mj * 64 + lane;
      at = hit & (hit - 1) ? INT32_MAX - wave_max_int(hit >> lane & 1 ? INT32_MAX - mp : 0)
                           : __builtin_amdgcn_readlane(mp, __builtin_ctzll(hit));
    }
    const bool known = __ballot(fresh == at) != 0;
    if (lane == b) {
      ek = mk;
      ep = at;
      es = known ? t : -1;
    }
    if (at != s && at != INT32_MAX) {  // another token's row
      if (lane == b) asked = round;
      if (wave == round % NW) {
        pend_b = b;
        pend_at = round;
        if (lane < PIECES) pend = *(reinterpret_cast<const uint4*>(vb + (int64_t)at * g.vst) + lane);
      }
    }
    // this round's keys before the next round's reads of them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  }
  if (wave == 0) store_held(t & ~63, t & 63);
  __syncthreads();

  // Kept positions in ascending order from the bitmap.
  const int per = (words + NT - 1) / NT;
  const int w0 = min(tid * per, words), w1 = min(w0 + per, words);
  uint32_t cnt = 0;
  for (int j = w0; j < w1; ++j) cnt += __popc(bits[j]);
  uint32_t incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) scan[wave] = incl;
  double lg = 0.0;  // log(1 + w c) of the picks
  for (int j = tid; j < t; j += NT) lg += log1p(gain_out[j]);
  lg = wave_sum_rows(lg);
  if (lane == 0) red[0][wave] = lg;
  __syncthreads();
  uint32_t off = incl - cnt;
  for (int j = 0; j < wave; ++j) off += scan[j];
  int32_t* out = idx_out + (int64_t)u * budget;
  for (int j = w0; j < w1; ++j) {
    uint32_t x = bits[j];
    while (x) {
      const int bit = __ffs(x) - 1;
      out[off++] = j * 32 + bit;
      x &= x - 1u;
    }
  }
  for (int j = t + tid; j < budget; j += NT) {
    out[j] = -1;
    if (order) order[j] = -1;
  }
  if (logdet_out && tid == 0) {
    double s = red[0][0];
    for (int i = 1; i < NW; ++i) s += red[0][i];
    logdet_out[u] = (double)D * log((double)ridge_f) + s;
  }
}

hipError_t launch_greedy(const Launch& L, const void* v, int32_t* idx, int32_t* order,
                         double* logdet) {
  const Geo& g = L.geo;
  const int budget = L.cfg->budget_k;
  const int nblk_max = (g.maxn + kGBlock - 1) / kGBlock;
  const float* wb = ws_ptr<float>(L.wsp, L.ws.wgt);
  double* gc = ws_ptr<double>(L.wsp, L.ws.gc);
  int32_t* gst = ws_ptr<int32_t>(L.wsp, L.ws.gst);
  GreedyEntry* ent = ws_ptr<GreedyEntry>(L.wsp, L.ws.gent);
  const float ridge = L.cfg->ridge;
  const double* wsc = ws_ptr<double>(L.wsp, L.ws.wscale);
  const int protect = L.cfg->protect_last;
  const bool bf16 = L.cfg->dtype == JACAP_DTYPE_BF16;
  {
    TimedPhase tp(L.stream, JACAP_PHASE_GREEDY_INIT);
    if (nblk_max > 0) {
      const dim3 grid(nblk_max, g.U);
      auto go = [&](auto kern, auto vp) {
        kern<<<grid, kThreads, 0, L.stream>>>(g, vp, wb, ridge, wsc, budget, protect, gc, gst,
                                              ent, nblk_max);
      };
      if (bf16) {
        if (g.D == 128) go(greedy_init_kernel<128, uint16_t>, (const uint16_t*)v);
        else go(greedy_init_kernel<64, uint16_t>, (const uint16_t*)v);
      } else {
        if (g.D == 128) go(greedy_init_kernel<128, float>, (const float*)v);
        else go(greedy_init_kernel<64, float>, (const float*)v);
      }
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  TimedPhase tp(L.stream, JACAP_PHASE_GREEDY);
  // Units whose keys fit in LDS: 2.7 times faster there (see the kernel).
  const size_t bytes = greedy_lds_bytes(g.D * (bf16 ? 2 : 4)) * nblk_max;
  if (bytes <= kGLdsMax) {
    static_assert(kGLdsMax / greedy_lds_bytes(128) <= 64, "a wave holds one block entry per lane");
    auto lds = [&](auto kern, auto vp) {
      // The limit is state of the function that every host thread shares, so it is the same
      // for every batch: between another thread's setting and its launch, a
      // shorter batch's own need would be too small for it.
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGLdsMax);
      if (e != hipSuccess) return e;
      kern<<<g.U, kGLdsThreads, bytes, L.stream>>>(g, vp, wb, ridge, wsc, budget, protect, gc, ent, nblk_max,
                                         idx, order, logdet);
      return hipGetLastError();
    };
    if (bf16)
      return g.D == 128 ? lds(greedy_lds_kernel<128, uint16_t>, (const uint16_t*)v)
                        : lds(greedy_lds_kernel<64, uint16_t>, (const uint16_t*)v);
    return g.D == 128 ? lds(greedy_lds_kernel<128, float>, (const float*)v)
                      : lds(greedy_lds_kernel<64, float>, (const float*)v);
  }
  auto go = [&](auto kern, auto vp) {
    kern<<<g.U, kThreads, 0, L.stream>>>(g, vp, wb, ridge, wsc, budget, protect, gc, gst, ent,
                                         nblk_max, idx, order, logdet);
  };
  if (bf16) {
    if (g.D == 128) go(greedy_kernel<128, uint16_t>, (const uint16_t*)v);
    else go(greedy_kernel<64, uint16_t>, (const uint16_t*)v);
  } else {
    if (g.D == 128) go(greedy_kernel<128, float>, (const float*)v);
    else go(greedy_kernel<64, float>, (const float*)v);
  }
  return hipGetLastError();
}

}  // namespace jacap
