// TOP-B selection (Algorithm 1, last step), its complement (the evicted
// positions, for caches refilled in place) and the retained-cache gather
// Z_C = {(k_i, v_i)}_{i in C} (Sec. 3.1).
//
// Selection is exact integer work on order-preserving 32-bit keys of the fp32
// scores (NaN -> 0, the lowest key; -0 -> +0): the budget-th largest key T,
// then every token with key > T and the lowest-position tokens with key == T,
// written in ascending position order. One workgroup per unit, in one of two
// shapes (1024 threads with 8192-entry lists, or 256 threads with 1024-entry
// lists for batches of many units with small effective budgets).
//
// Three paths (sel_wide_path has the wide shape's rule):
// * direct: units whose keys fit a thread's registers are ranked and emitted
//   from there;
// * sampled (wide shape): a lower bound lo <= T from a small sample, one ordered
//   pass that collects the candidates, key >= lo, in position order into LDS,
//   their ranking and emission -- as long as the candidates a sample leaves are few;
// * staged: a larger sample brackets lo <= T <= hi, so that large budgets too leave
//   few candidates: the pass collects the tokens with key > hi (kept for sure) and
//   those of the band, in a list of 8192 each (the first is full from about 10000
//   kept of 131072 on).
// The pass checks that the bounds hold (fewer than budget tokens above hi, at
// least budget at or above lo) and that the lists fit; otherwise the unit takes
// the general path: a three-pass radix select over the scores (11 + 11 + 10
// bits, MSB first) and an ordered emission pass, several times slower. All paths
// give the same, deterministic result.
//
// The first two count with wave ballots: a wave takes 64 consecutive positions per
// step, so popcounts of the lanes below give every position's place, and the waves
// exchange one word each at one barrier; ranks among keys held in registers are
// found two bits at a time (rank_search), without the LDS atomics of a histogram
// (radix_rank), whose conflicts on the few exponents of the scores cost more
// while the keys per thread are few.
//
// Measured (MI355X, jacap_select calls; histogram ranks and staged chunks
// everywhere, and now): 8 units of 32768 tokens keeping 512 32.6 and 22.9 us; 256
// units of 131072 keeping 1024 68.7 and 48.2, keeping 8192 80.3 and 77.1; 64 units
// of 262144 keeping 4096 118 and 110; 1024 units of 16512 keeping 16384 85 and 50;
// 4096 units of 2176 tokens, evicted slots, 167 and 65; 8 units of 8192 tokens 16.2
// and 16.3.
#include <algorithm>
#include <type_traits>

#include "jacap_internal.hpp"
#include "select_plan.hpp"

namespace jacap {

// Launch shape of the selection: THREADS per workgroup, CAP entries in each
// LDS list. The wide shape (one unit per CU) serves few long units; the
// narrow one fits several workgroups per CU for many units with small
// effective budgets.
template <int THREADS, int CAP>
struct SelCfg {
  static constexpr int kThreads = THREADS;
  static constexpr int kWaves = THREADS / 64;
  static constexpr int kPer = 8;                   // tokens per thread per chunk of the ordered pass
  static constexpr int kChunk = kPer * THREADS;    // scores per chunk
  static constexpr int kCand = CAP;                // candidate band capacity
  static constexpr int kSure = CAP;                // kept-for-sure list capacity
  static constexpr int kCandPer = CAP / THREADS;   // candidates per thread
  static constexpr bool kWide = THREADS == 1024;
  // Longest unit of the direct path. Its search costs 16 steps of three counts per
  // key and thread; in the wide shape two keys are where a histogram costs less.
  static constexpr int kDirect = kWide ? kSelWideDirect : 4096;
  static constexpr int kSample = kChunk / 64;      // sample of the staged path: <= kSample blocks
};
using SelWide = SelCfg<1024, kSelWideCand>;   // 141 KB of LDS: one workgroup per CU
using SelNarrow = SelCfg<256, 1024>;          // 29 KB: five per CU
// Batches of at least this many units take the narrow shape when no unit
// ranks more than half its list capacity.
constexpr int kSelNarrowUnits = 1024;

__device__ __forceinline__ uint32_t score_key(float f) {
  const float g = f + 0.0f;       // -0 == +0
  const uint32_t b = __float_as_uint(g);
  const uint32_t k = b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);  // ~b, or b with its top bit set
  return g == g ? k : 0u;         // NaN ranks lowest
}

// The n scores that a unit ranks: kForward, or kReverse: in reverse, by their
// complemented keys (to find the tokens at the end of the order instead), or either
// of them as the launch finds (kEither: one kernel body for both).
enum { kForward = 0, kReverse = 1, kEither = 2 };
template <int DIR>
struct RankedScores {
  const float* s;
  int n;
  bool reversed;
  __device__ __forceinline__ uint32_t flip() const {
    return DIR == kEither ? (reversed ? ~0u : 0u) : DIR == kReverse ? ~0u : 0u;
  }
  __device__ __forceinline__ float raw(int i) const {
    return s[(int)((uint32_t)i ^ flip()) + (n & (int)flip())];  // s[i], or s[n - 1 - i]
  }
  __device__ __forceinline__ uint32_t conv(float f) const { return score_key(f) ^ flip(); }
  __device__ __forceinline__ uint32_t key(int i) const { return conv(raw(i)); }
};
// The list of selected positions: a unit's kept ones in global memory, or (of
// reversed scores) the evicted ones in LDS.
template <int DIR>
struct SelOut {
  int32_t* global;
  int32_t* lds;
  bool reversed;
  __device__ __forceinline__ void put(int place, int32_t pos) const {
    if (DIR == kReverse || (DIR == kEither && reversed)) lds[place] = pos;
    else global[place] = pos;
  }
};

template <class C>
struct SelShared {
  uint32_t ckey[C::kCand];    // candidate keys (position order)
  int32_t cpos[C::kCand];     // candidate positions
  int32_t gpos[C::kSure];     // kept-for-sure positions (position order)
  // kept candidates (position order) / evicted positions; in the staged path also
  // the chunk's keys (one pad word per 8: the per-thread reads of 8 consecutive
  // keys are then bank-conflict free) and the sample's
  int32_t kept[C::kChunk + C::kChunk / 8];
  uint32_t hist[2048];
  uint32_t scan[C::kWaves + 1];
  uint32_t bc[2];
  uint2 cnt[2][C::kWaves];    // counts of the waves, one of the two sets per exchange
};

// Per-wave words a and b (uniform in each wave, every 16-bit field's sum below
// 65536): their sums over the workgroup's waves, and over the waves before this
// one. One barrier; `par` alternates the exchange buffer.
template <class C>
__device__ __forceinline__ uint2 wave_exchange(uint2 v, SelShared<C>& sh, int& par, uint2& before) {
  static_assert(C::kWaves <= 16, "one DPP row of wave words");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (lane == 0) sh.cnt[par][wave] = v;
  __syncthreads();
  uint2 w = make_uint2(0u, 0u);
  if ((lane & 15) < C::kWaves) w = sh.cnt[par][lane & 15];
  uint2 b = (lane & 15) < wave ? w : make_uint2(0u, 0u);
  auto row_sum = [](uint32_t x) {
    auto d = [](uint32_t y, auto c) {
      return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, decltype(c)::value, 0xF, 0xF, true);
    };
    x += d(x, std::integral_constant<int, kDppQuadXor1>{});
    x += d(x, std::integral_constant<int, kDppQuadXor2>{});
    x += d(x, std::integral_constant<int, kDppHalfMirror>{});
    x += d(x, std::integral_constant<int, kDppMirror>{});
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
  };
  before = make_uint2(row_sum(b.x), row_sum(b.y));
  par ^= 1;
  return make_uint2(row_sum(w.x), row_sum(w.y));
}

// Bitwise and of v.x and or of v.y over the workgroup's threads (the exchange of
// wave_exchange).
template <class C>
__device__ __forceinline__ uint2 block_and_or(uint2 v, SelShared<C>& sh, int& par) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto rows = [](uint2 x) {
    auto d = [](uint32_t y, auto c) {
      return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, decltype(c)::value, 0xF, 0xF, true);
    };
    auto step = [&](auto c) { x = make_uint2(x.x & d(x.x, c), x.y | d(x.y, c)); };
    step(std::integral_constant<int, kDppQuadXor1>{});
    step(std::integral_constant<int, kDppQuadXor2>{});
    step(std::integral_constant<int, kDppHalfMirror>{});
    step(std::integral_constant<int, kDppMirror>{});
    return x;
  };
  auto at = [](uint32_t x, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)x, l); };
  v = rows(v);
  const uint2 w = make_uint2(at(v.x, 0) & at(v.x, 16) & at(v.x, 32) & at(v.x, 48),
                             at(v.y, 0) | at(v.y, 16) | at(v.y, 32) | at(v.y, 48));
  if (lane == 0) sh.cnt[par][wave] = w;
  __syncthreads();
  uint2 r = make_uint2(~0u, 0u);
  if ((lane & 15) < C::kWaves) r = sh.cnt[par][lane & 15];
  r = rows(r);
  par ^= 1;
  return make_uint2(at(r.x, 0), at(r.y, 0));
}

// A threshold for the rank `rank` (1 = largest) among the keys k[0 .. PER) of every
// thread (0 in unused places): the largest T with at least `rank` keys >= T,
// found two bits at a time from the top -- or, as soon as some prefix c has
// rank .. rank + slack keys >= c, T = c - 1, whose lower bits do not matter. `above`
// = the number of keys > T: with slack 0 the top `rank` keys are those > T and
// the first rank - above of those == T. Where many keys share T's prefix after six
// steps, the bits in which none of them differs are not searched, which ends the
// search where many scores are equal (8 units of 512 scores of 15 values 13.5 to 7.9 us).
constexpr int kTieBit = 20;
template <class C, int PER>
__device__ __forceinline__ uint32_t rank_search(const uint32_t (&k)[PER], uint32_t rank,
                                                uint32_t slack, SelShared<C>& sh, int& par,
                                                uint32_t& above) {
  static_assert(PER * C::kThreads < 65536, "counts in 16-bit fields");
  uint32_t T = 0u, reach = PER * C::kThreads;  // reach: keys >= T (at most)
  above = 0u;
#pragma unroll 1
  for (int bit = 30; bit >= 0; bit -= 2) {
    uint32_t c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const uint32_t cand = T | (uint32_t)(d + 1) << bit;
      c[d] = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) c[d] += __popcll(__ballot(k[j] >= cand));
    }
    uint2 before;
    const uint2 s = wave_exchange<C>(make_uint2(c[0] | c[1] << 16, c[2]), sh, par, before);
    const uint32_t n1 = s.x & 0xFFFFu, n2 = s.x >> 16, n3 = s.y;
    const uint32_t d = n3 >= rank ? 3u : n2 >= rank ? 2u : n1 >= rank ? 1u : 0u;
    const uint32_t nd = d == 3 ? n3 : d == 2 ? n2 : n1;  // keys >= the digit's prefix (d > 0)
    T |= d << bit;
    if (d > 0 && nd <= rank + slack) {
      above = nd;
      return T - 1u;
    }
    above = d == 3 ? above : d == 2 ? n3 : d == 1 ? n2 : n1;
    reach = d > 0 ? nd : reach;
    if (bit == kTieBit && reach - above > PER * C::kThreads / 32) {
      uint2 ao = make_uint2(~0u, 0u);  // and / or of the keys with T's prefix (one at least)
#pragma unroll
      for (int j = 0; j < PER; ++j)
        if (k[j] >> kTieBit == T >> kTieBit) ao = make_uint2(ao.x & k[j], ao.y | k[j]);
      ao = block_and_or<C>(ao, sh, par);
      const uint32_t differ = ao.x ^ ao.y;
      if (differ == 0u) return ao.x;
      bit = ((31 - __clz(differ)) & ~1) + 2;  // the next step is two bits below
      T = ao.x & ~((1u << bit) - 1u);
    }
  }
  return T;
}

// Places of the kept keys among k[0 .. PER) of every thread, in the order (wave,
// j, lane): keys > T, and the first `need` of those == T. f(j, place) for each
// kept key of this thread. (Unused places hold key 0 and come last, so none of them
// is among the first `need`.)
template <class C, int PER, class F>
__device__ __forceinline__ void emit_kept(const uint32_t (&k)[PER], uint32_t T, uint32_t need,
                                          SelShared<C>& sh, int& par, F f) {
  const uint64_t below = ((uint64_t)1 << (threadIdx.x & 63)) - 1;
  uint32_t ng = 0, ne = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    ng += __popcll(__ballot(k[j] > T));
    ne += __popcll(__ballot(k[j] == T));
  }
  uint2 before;
  wave_exchange<C>(make_uint2(ng, ne), sh, par, before);
  uint32_t g = before.x, e = before.y;  // keys > T, keys == T so far
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    uint32_t kj = k[j];
    if constexpr (PER > 4) asm volatile("" : "+v"(kj));  // the ballots above again: kept, they would spill
    const bool gt = kj > T, eq = kj == T;
    const uint64_t bg = __ballot(gt), be = __ballot(eq);
    const uint32_t gb = g + __popcll(bg & below), eb = e + __popcll(be & below);
    if (gt || (eq && eb < need)) f(j, gb + min(eb, need));
    g += __popcll(bg);
    e += __popcll(be);
  }
}

// Exclusive prefix sum over C::kThreads values (one per thread), fixed order:
// a wave scan, then every thread adds the totals of the waves before its own
// (broadcast LDS reads, no serial pass).
template <class C>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* sh, uint32_t& total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t incl = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  __syncthreads();
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < C::kThreads / 64; ++w) {
    const uint32_t t = sh[w];
    before += w < wave ? t : 0u;
    all += t;
  }
  total = all;
  return before + incl - x;
}

// Radix select (11 + 11 + 10 bits, MSB first): the key of rank `rank`
// (1 = largest, rank <= cnt) among key_at(0 .. cnt-1); `need` = how many keys
// equal to it fall within the top `rank`.
template <class C, class KeyAt>
__device__ __forceinline__ uint32_t radix_rank(KeyAt key_at, int cnt, uint32_t rank,
                                               SelShared<C>& sh, uint32_t& need) {
  const int tid = threadIdx.x;
  uint32_t prefix = 0u, pmask = 0u, remaining = rank;
  const int shifts[3] = {21, 10, 0};
  const int widths[3] = {11, 11, 10};
  for (int pass = 0; pass < 3; ++pass) {
    const int shf = shifts[pass];
    const uint32_t nb = 1u << widths[pass];
    const uint32_t dmask = nb - 1u;
    for (uint32_t i = tid; i < nb; i += C::kThreads) sh.hist[i] = 0u;
    if (tid == 0) { sh.bc[0] = 0u; sh.bc[1] = 0u; }
    __syncthreads();
    for (int i = tid; i < cnt; i += C::kThreads) {
      const uint32_t key = key_at(i);
      if ((key & pmask) == prefix) atomicAdd(&sh.hist[(key >> shf) & dmask], 1u);
    }
    __syncthreads();
    // Suffix counts from the top digit down: each thread owns a contiguous run
    // of bins (descending digit order), then a block scan.
    const uint32_t per = nb / C::kThreads;  // bins per thread
    uint32_t local = 0;
    for (uint32_t q = 0; q < per; ++q) local += sh.hist[nb - 1 - (tid * per + q)];
    uint32_t tot;
    uint32_t above = block_exclusive_scan<C>(local, sh.scan, tot);
    for (uint32_t q = 0; q < per; ++q) {
      const uint32_t d = nb - 1 - (tid * per + q);
      const uint32_t c = sh.hist[d];
      if (above < remaining && remaining <= above + c) {
        sh.bc[0] = d;
        sh.bc[1] = above;
      }
      above += c;
    }
    __syncthreads();
    prefix |= sh.bc[0] << shf;
    pmask |= dmask << shf;
    remaining -= sh.bc[1];
    __syncthreads();
  }
  need = remaining;
  return prefix;
}

// General path: radix select over the scores, then an ordered emission pass
// over contiguous per-thread segments.
template <class C, int DIR>
__device__ __forceinline__ void select_general(const RankedScores<DIR>& rs, int kk,
                                               const SelOut<DIR>& out, SelShared<C>& sh) {
  const int tid = threadIdx.x, n = rs.n;
  auto key_at = [&](int i) { return rs.key(i); };
  uint32_t need;
  const uint32_t T = radix_rank<C>(key_at, n, (uint32_t)kk, sh, need);
  const int seg = (n + C::kThreads - 1) / C::kThreads;
  const int lo = min(n, tid * seg), hi = min(n, lo + seg);
  uint32_t cgt = 0, ceq = 0;
  for (int i = lo; i < hi; ++i) {
    const uint32_t key = key_at(i);
    cgt += key > T;
    ceq += key == T;
  }
  uint32_t tot;
  uint32_t gt_before = block_exclusive_scan<C>(cgt, sh.scan, tot);
  uint32_t eq_before = block_exclusive_scan<C>(ceq, sh.scan, tot);
  for (int i = lo; i < hi; ++i) {
    const uint32_t key = key_at(i);
    if (key > T) {
      const uint32_t pos = gt_before + min(eq_before, need);
      if (pos < (uint32_t)kk) out.put((int)pos, i);
      ++gt_before;
    } else if (key == T) {
      const uint32_t pos = gt_before + eq_before;
      if (eq_before < need && pos < (uint32_t)kk) out.put((int)pos, i);
      ++eq_before;
    }
  }
}

// Number of entries of the ascending list a[0 .. cnt) that are < p.
__device__ __forceinline__ int lower_bound_lds(const int32_t* a, int cnt, int32_t p) {
  int lo = 0, hi = cnt;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (a[mid] < p) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// The top r of the ccnt candidates, PER keys per thread (C::kThreads * PER >= ccnt):
// their positions, ascending, to out.
template <class C, int PER, int DIR>
__device__ __forceinline__ void keep_candidates(uint32_t ccnt, uint32_t r, const SelOut<DIR>& out,
                                                SelShared<C>& sh, int& par) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t k[PER];
  auto index = [&](int j) { return (uint32_t)((wave * PER + j) * 64 + lane); };
#pragma unroll
  for (int j = 0; j < PER; ++j) k[j] = index(j) < ccnt ? sh.ckey[index(j)] : 0u;
  uint32_t above;  // (the search's barriers come before the list that may replace ckey)
  const uint32_t T = rank_search<C, PER>(k, r, 0u, sh, par, above);
  emit_kept<C, PER>(k, T, r - above, sh, par,
                    [&](int j, uint32_t place) { out.put((int)place, sh.cpos[index(j)]); });
}

// Every key in a register: PER per thread (n <= C::kThreads * PER).
template <class C, int PER, int DIR>
__device__ __forceinline__ void select_direct(const RankedScores<DIR>& rs, int kk,
                                              const SelOut<DIR>& out, SelShared<C>& sh) {
  const int n = rs.n;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int par = 0;
  uint32_t k[PER];
  auto pos = [&](int j) { return (wave * PER + j) * 64 + lane; };
  float raw[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) raw[j] = rs.raw(min(pos(j), n - 1));
#pragma unroll
  for (int j = 0; j < PER; ++j) k[j] = pos(j) < n ? rs.conv(raw[j]) : 0u;
  uint32_t above;
  const uint32_t T = rank_search<C, PER>(k, (uint32_t)kk, 0u, sh, par, above);
  emit_kept<C, PER>(k, T, (uint32_t)kk - above, sh, par,
                    [&](int j, uint32_t place) { out.put((int)place, pos(j)); });
}

// Long units of the wide shape, where a small sample leaves few enough candidates:
// sample select, counted with ballots. The sample's rank search costs a step of
// every wave per two bits, so the sample is small, and its segments short, so that
// they still meet every run of high scores that a larger sample of 64-token blocks
// would; an upper bound, whose kept-for-sure tokens shorten the candidates' list,
// costs a second search and a merge, and is left to select_staged.
template <class C, int DIR>
__device__ __forceinline__ bool select_sampled(const RankedScores<DIR>& rs, int kk,
                                               const SelOut<DIR>& out, SelShared<C>& sh) {
  const int lane = threadIdx.x & 63, n = rs.n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int par = 0;
  // A lower bound of T from a sample of PER keys per thread.
  uint32_t lo = 0u;
  const SelBracket b = sel_sampled_bracket(n, kk);
  auto bound = [&](auto perc) {
    constexpr int PER = decltype(perc)::value;
    uint32_t k[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = (wave * PER + j) * 64 + lane;   // of the sample
      const int p = e / kSelSeg * b.q * kSelSeg + e % kSelSeg;
      k[j] = e < b.S ? rs.key(p) : 0u;
    }
    uint32_t dummy;
    lo = rank_search<C, PER>(k, (uint32_t)b.r_lo, (uint32_t)sel_slack(b), sh, par, dummy);
  };
  if (sel_sample_per(n) == 1) bound(std::integral_constant<int, 1>{});
  else bound(std::integral_constant<int, 2>{});

  // One ordered pass: the candidates, key >= lo; a chunk's scores loaded one chunk
  // ahead (kept raw until used, so that no conversion waits on the loads early).
  const uint64_t below = ((uint64_t)1 << lane) - 1;
  float nxt[C::kPer];
  auto pos = [&](int base, int j) { return base + (wave * C::kPer + j) * 64 + lane; };
  auto load_chunk = [&](int base) {
#pragma unroll
    for (int j = 0; j < C::kPer; ++j) nxt[j] = rs.raw(min(pos(base, j), n - 1));
  };
  load_chunk(0);
  uint32_t ccnt = 0;
  for (int base = 0; base < n; base += C::kChunk) {
    uint32_t k[C::kPer];
#pragma unroll
    for (int j = 0; j < C::kPer; ++j) k[j] = rs.conv(nxt[j]);
    if (base + C::kChunk < n) load_chunk(base + C::kChunk);  // uniform
    uint64_t cand[C::kPer];
    uint32_t nc = 0;
#pragma unroll
    for (int j = 0; j < C::kPer; ++j) {
      cand[j] = __ballot(pos(base, j) < n && k[j] >= lo);
      nc += __popcll(cand[j]);
    }
    uint2 before;
    const uint2 tot = wave_exchange<C>(make_uint2(nc, 0u), sh, par, before);
    uint32_t co = ccnt + before.x;
#pragma unroll
    for (int j = 0; j < C::kPer; ++j) {
      const uint32_t at = co + __popcll(cand[j] & below);
      if ((cand[j] >> lane & 1) && at < (uint32_t)C::kCand) {
        sh.ckey[at] = k[j];
        sh.cpos[at] = pos(base, j);
      }
      co += __popcll(cand[j]);
    }
    ccnt += tot.x;
  }
  __syncthreads();
  // uniform: the same count in every thread
  if (ccnt < (uint32_t)kk || ccnt > (uint32_t)C::kCand) return false;
  // T among the candidates; fewer keys per thread cost less.
  if (ccnt <= (uint32_t)C::kThreads) keep_candidates<C, 1>(ccnt, (uint32_t)kk, out, sh, par);
  else if (ccnt <= 2u * C::kThreads) keep_candidates<C, 2>(ccnt, (uint32_t)kk, out, sh, par);
  else if (ccnt <= 4u * C::kThreads) keep_candidates<C, 4>(ccnt, (uint32_t)kk, out, sh, par);
  else keep_candidates<C, 8>(ccnt, (uint32_t)kk, out, sh, par);
  static_assert(C::kCandPer <= 8, "candidates per thread");
  return true;
}

// Long units otherwise: the same with a larger sample of 64-token blocks, histogram
// ranks (radix_rank) and the chunk's keys staged in LDS, 8 consecutive per thread.
// In the narrow shape several workgroups share a compute unit and its one scalar
// unit, which the ballots of select_sampled keep busy (4096 units of 4096 to 32768
// tokens 178 us, 326 us with ballots); in the wide one the larger sample keeps the
// candidates of large budgets within their list, and histogram ranks cost less
// than ballots on that many.
template <class C, int DIR>
__device__ __forceinline__ bool select_staged(const RankedScores<DIR>& rs, int kk,
                                              const SelOut<DIR>& out, SelShared<C>& sh) {
  static_assert(C::kCand <= C::kChunk + C::kChunk / 8, "kept candidates are merged from stage");
  uint32_t* stage = reinterpret_cast<uint32_t*>(sh.kept);
  static_assert(C::kSample * 64 <= C::kChunk, "the sample is staged in stage");
  const int tid = threadIdx.x, n = rs.n;
  // Bracket [lo, hi] of T from the sample (the whole unit if it fits the band).
  uint32_t lo = 0u, hi = 0xFFFFFFFFu;
  if (n > C::kCand) {
    const SelBracket b = sel_bracket(n, kk, 64, C::kSample);
    for (int j = tid; j < b.S; j += C::kThreads)
      stage[j] = rs.key((j >> 6) * b.q * 64 + (j & 63));
    __syncthreads();
    uint32_t dummy;
    // When the band reaches the top of the sample there is no upper bound:
    // tokens above the sample maximum are candidates too.
    if (b.r_hi >= 1)
      hi = radix_rank<C>([&](int i) { return stage[i]; }, b.S, (uint32_t)b.r_hi, sh, dummy);
    lo = radix_rank<C>([&](int i) { return stage[i]; }, b.S, (uint32_t)b.r_lo, sh, dummy);
  }

  // One ordered pass: kept-for-sure (key > hi) and candidates (lo <= key <= hi).
  // Chunks (2048 scores, 8192 in the wide shape) are loaded coalesced one chunk ahead (kept raw until
  // staged, so that no conversion waits on the loads early), staged in LDS
  // with a pad word per 8 keys, and read back as 8 consecutive keys per
  // thread (bank-conflict free); the block scan orders the threads' lists.
  auto pad = [](int e) { return e + (e >> 3); };
  float nxt[C::kPer];
  auto load_chunk = [&](int base) {
#pragma unroll
    for (int j = 0; j < C::kPer; ++j) nxt[j] = rs.raw(min(base + j * C::kThreads + tid, n - 1));
  };
  load_chunk(0);
  uint32_t gcnt = 0, ccnt = 0;
  for (int base = 0; base < n; base += C::kChunk) {
#pragma unroll
    for (int j = 0; j < C::kPer; ++j) {
      const int p = base + j * C::kThreads + tid;
      stage[pad(j * C::kThreads + tid)] = p < n ? rs.conv(nxt[j]) : 0u;
    }
    if (base + C::kChunk < n) load_chunk(base + C::kChunk);  // uniform
    __syncthreads();
    uint32_t k8[C::kPer];
    uint32_t ng = 0, nc = 0;
#pragma unroll
    for (int qd = 0; qd < C::kPer; ++qd) {
      const int p = base + C::kPer * tid + qd;
      k8[qd] = stage[pad(C::kPer * tid + qd)];
      const bool valid = p < n;
      ng += valid && k8[qd] > hi;
      nc += valid && k8[qd] >= lo && k8[qd] <= hi;
    }
    uint32_t tot;
    const uint32_t off = block_exclusive_scan<C>((ng << 16) | nc, sh.scan, tot);
    uint32_t go = gcnt + (off >> 16), co = ccnt + (off & 0xFFFFu);
#pragma unroll
    for (int qd = 0; qd < C::kPer; ++qd) {
      const int p = base + C::kPer * tid + qd;
      if (p >= n) continue;
      if (k8[qd] > hi) {
        if (go < (uint32_t)C::kSure) sh.gpos[go] = p;
        ++go;
      } else if (k8[qd] >= lo) {
        if (co < (uint32_t)C::kCand) { sh.ckey[co] = k8[qd]; sh.cpos[co] = p; }
        ++co;
      }
    }
    gcnt += tot >> 16;
    ccnt += tot & 0xFFFFu;
    __syncthreads();
  }
  const bool ok = gcnt < (uint32_t)kk && gcnt + ccnt >= (uint32_t)kk &&
                  gcnt <= (uint32_t)C::kSure && ccnt <= (uint32_t)C::kCand;
  if (!ok) return false;  // uniform: every thread holds the same counts

  // T among the candidates: rank kk - gcnt.
  const uint32_t r = (uint32_t)kk - gcnt;
  uint32_t need;
  const uint32_t T = radix_rank<C>([&](int i) { return sh.ckey[i]; }, (int)ccnt, r, sh, need);
  // Kept candidates, in position order, into stage[0 .. r).
  const int per = ((int)ccnt + C::kThreads - 1) / C::kThreads;
  const int c0 = min((int)ccnt, tid * per), c1 = min((int)ccnt, c0 + per);
  uint32_t ceq = 0;
  for (int i = c0; i < c1; ++i) ceq += sh.ckey[i] == T;
  uint32_t tot;
  uint32_t eq_before = block_exclusive_scan<C>(ceq, sh.scan, tot);
  uint32_t csel = 0;
  for (int i = c0, e = eq_before; i < c1; ++i) {
    const uint32_t key = sh.ckey[i];
    if (key > T) ++csel;
    else if (key == T) { csel += (uint32_t)e < need; ++e; }
  }
  uint32_t sel_before = block_exclusive_scan<C>(csel, sh.scan, tot);
  for (int i = c0, e = eq_before; i < c1; ++i) {
    const uint32_t key = sh.ckey[i];
    bool keep = false;
    if (key > T) keep = true;
    else if (key == T) { keep = (uint32_t)e < need; ++e; }
    if (keep) stage[sel_before++] = (uint32_t)sh.cpos[i];
  }
  __syncthreads();
  // Merge the two position-ordered lists into out[0 .. kk).
  const int32_t* kept_c = reinterpret_cast<const int32_t*>(stage);
  for (int a = tid; a < (int)gcnt; a += C::kThreads) {
    const int32_t p = sh.gpos[a];
    out.put(a + lower_bound_lds(kept_c, (int)r, p), p);
  }
  for (int e = tid; e < (int)r; e += C::kThreads) {
    const int32_t p = kept_c[e];
    out.put(e + lower_bound_lds(sh.gpos, (int)gcnt, p), p);
  }
  return true;
}

// TOP-kk of the ranked scores by (key desc, position asc), written to out at
// 0 .. kk in ascending position order (0 < kk < n).
template <class C, int DIR>
__device__ __forceinline__ void select_unit(const RankedScores<DIR>& rs, int kk,
                                            const SelOut<DIR>& out, SelShared<C>& sh) {
  if (rs.n <= C::kDirect / 2) {
    select_direct<C, C::kDirect / 2 / C::kThreads>(rs, kk, out, sh);
  } else if (rs.n <= C::kDirect) {
    select_direct<C, C::kDirect / C::kThreads>(rs, kk, out, sh);
  } else {
    bool done;
    if (C::kWide && sel_wide_path(rs.n, kk) == SelPath::kSampled) {
      if constexpr (C::kWide) done = select_sampled(rs, kk, out, sh);
    } else {
      done = select_staged(rs, kk, out, sh);
    }
    if (!done) select_general(rs, kk, out, sh);
  }
}

// The complement is ranked instead of the kept tokens when it is the smaller
// part of the n ranked positions and fits the lists.
template <class C>
__device__ __forceinline__ bool ranks_evicted(int n, int kk) {
  return kk > 0 && kk < n && n - kk < kk && n - kk <= C::kCand;
}

// slots != null: the evicted-slot lists are wanted (capacity cap per unit); a unit
// whose evicted tokens are the ranked part writes its list here, and no kept
// positions, the others leave theirs in idx for evicted_kernel.
template <class C>
__global__ __launch_bounds__(C::kThreads) void select_kernel(Geo g, const float* __restrict__ scores,
                                                             int32_t* __restrict__ idx, int budget,
                                                             int protect,
                                                             int32_t* __restrict__ slots, int cap) {
  __shared__ SelShared<C> sh;
  const int u = blockIdx.x, tid = threadIdx.x;
  const Unit un = decode_unit(g, u);
  int32_t* out = idx + (int64_t)u * budget;
  const int kk_all = min(budget, un.n);
  const float* s = scores + token_row(g, un);
  // Protected tail: the last p positions are kept; the ranking fills the
  // remaining kk slots from positions 0 .. n-1 (n = n_b - p), whose indices
  // all precede the tail, so the tail simply follows them in idx.
  const int npro = min(protect, kk_all);
  const int n = un.n - npro, kk = kk_all - npro;

  // Keeping more than half: select the n - kk tokens to evict instead (the
  // last n - kk of the order (key desc, position asc) are the first n - kk of
  // (~key desc, reversed position asc)), then emit every other position.
  const bool evicts = ranks_evicted<C>(n, kk);
  const int m = n - kk;
  if (!evicts) {
    for (int j = kk_all + tid; j < budget; j += C::kThreads) out[j] = -1;
    for (int j = tid; j < npro; j += C::kThreads) out[kk + j] = n + j;
    if (kk == 0) return;
    if (kk == n) {
      for (int j = tid; j < n; j += C::kThreads) out[j] = j;
      return;
    }
  }
  // evicted: as reversed positions, ascending (the candidates' keys are no
  // longer read when they are written)
  int32_t* rev = reinterpret_cast<int32_t*>(sh.ckey);
  if constexpr (!C::kWide) {  // (16 keys per thread: 30 spilled scalar registers, 57 if compiled twice)
    select_unit(RankedScores<kEither>{s, n, evicts}, evicts ? m : kk, SelOut<kEither>{out, rev, evicts}, sh);
  } else if (evicts) {
    select_unit(RankedScores<kReverse>{s, n, true}, m, SelOut<kReverse>{out, rev, true}, sh);
  } else {
    select_unit(RankedScores<kForward>{s, n, false}, kk, SelOut<kForward>{out, rev, false}, sh);
  }
  if (evicts) {
    __syncthreads();
    auto evicted = [&](int j) { return n - 1 - rev[m - 1 - j]; };  // ascending
    if (slots) {
      int32_t* so = slots + (int64_t)u * cap;
      for (int j = tid; j < cap; j += C::kThreads) so[j] = j < m ? evicted(j) : -1;
      return;
    }
    for (int j = kk_all + tid; j < budget; j += C::kThreads) out[j] = -1;
    for (int j = tid; j < npro; j += C::kThreads) out[kk + j] = n + j;
    if (n <= 2048 * 32) {
      // a bitmap of the evicted; each wave walks a run of 64-position blocks with
      // a running count
      const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      const int nb64 = (n + 63) / 64, run = (nb64 + C::kWaves - 1) / C::kWaves;
      for (int j = tid; j < 2 * nb64; j += C::kThreads) sh.hist[j] = 0u;
      __syncthreads();
      for (int j = tid; j < m; j += C::kThreads) {
        const int p = evicted(j);
        atomicOr(&sh.hist[p >> 5], 1u << (p & 31));
        sh.kept[j] = p;
      }
      __syncthreads();
      const int b0 = min(nb64, wave * run), b1 = min(nb64, b0 + run);
      int gone = lower_bound_lds(sh.kept, m, b0 * 64);  // evicted before the block
      const uint64_t below = ((uint64_t)1 << lane) - 1;
      for (int b = b0; b < b1; ++b) {
        const uint64_t ev = (uint64_t)sh.hist[2 * b] | (uint64_t)sh.hist[2 * b + 1] << 32;
        const int p = 64 * b + lane;
        if (p < n && !(ev >> lane & 1)) out[p - gone - __popcll(ev & below)] = p;
        gone += __popcll(ev);
      }
      return;
    }
    for (int j = tid; j < m; j += C::kThreads) sh.kept[j] = evicted(j);
    __syncthreads();
    for (int i = tid; i < n; i += C::kThreads) {
      const int c = lower_bound_lds(sh.kept, m, i);
      if (c == m || sh.kept[c] != i) out[i - c] = i;
    }
  }
}

// The narrow shape: many units, each ranking at most half of its lists (the
// largest number of tokens any unit ranks is min(B, n - B) at the longest n).
static bool select_narrow(const Launch& L) {
  const int budget = L.cfg->budget_k;
  const int kmax = std::min(budget, std::max(0, L.geo.maxn - budget));
  return L.geo.U >= kSelNarrowUnits && kmax <= SelNarrow::kCand / 2;
}

static hipError_t select_launch(const Launch& L, const float* scores, int32_t* idx, int32_t* slots,
                                int cap) {
  const Geo& g = L.geo;
  auto go = [&](auto kern, int threads) {
    kern<<<g.U, threads, 0, L.stream>>>(g, scores, idx, L.cfg->budget_k, L.cfg->protect_last, slots,
                                        cap);
  };
  if (select_narrow(L)) go(select_kernel<SelNarrow>, SelNarrow::kThreads);
  else go(select_kernel<SelWide>, SelWide::kThreads);
  return hipGetLastError();
}

hipError_t launch_select(const Launch& L, const float* scores, int32_t* idx) {
  return select_launch(L, scores, idx, nullptr, 0);
}

// ---------------------------------------------------------------------------
// Evicted slots: the positions of each unit that the selection does not keep,
// ascending, then -1 up to the list's capacity. The kept positions come
// ascending from select_kernel; an evicted position i goes to slot i - r,
// r = the number of kept positions below i. Workgroup (tile, unit) takes the
// positions [p0, p0 + kEvTile): two binary searches of the kept list bound the
// kept positions inside the tile, which are staged in LDS, and each thread
// places the positions p0 + tid, p0 + tid + kThreads, ... (consecutive
// threads write consecutive slots between kept positions). The tile also
// writes the -1 padding of the slots [p0, p0 + kEvTile) at or past n - kept,
// and the last tile every padding slot beyond. Units whose list select_kernel has
// written already are skipped.
// ---------------------------------------------------------------------------
constexpr int kEvTile = 4096;

template <class C>
__global__ __launch_bounds__(kThreads) void evicted_kernel(Geo g, const int32_t* __restrict__ kept,
                                                           int budget, int protect,
                                                           int32_t* __restrict__ slots, int cap) {
  const int u = blockIdx.y, tile = blockIdx.x, tid = threadIdx.x;
  const Unit un = decode_unit(g, u);
  const int n = un.n, kk = min(budget, n), ne = n - kk;
  const int npro = min(protect, kk);
  if (ranks_evicted<C>(n - npro, kk - npro)) return;
  const int32_t* kp = kept + (int64_t)u * budget;
  int32_t* out = slots + (int64_t)u * cap;
  const int p0 = tile * kEvTile;
  const int pad_hi = tile == (int)gridDim.x - 1 ? cap : min(cap, p0 + kEvTile);
  for (int j = max(ne, p0) + tid; j < pad_hi; j += kThreads) out[j] = -1;
  if (p0 >= n) return;
  const int p1 = min(n, p0 + kEvTile);
  __shared__ int32_t ks[kEvTile];
  __shared__ int bounds[2];
  if (tid < 2) bounds[tid] = lower_bound_lds(kp, kk, tid == 0 ? p0 : p1);
  __syncthreads();
  const int lo = bounds[0], cnt = bounds[1] - bounds[0];  // distinct positions: cnt <= kEvTile
  for (int j = tid; j < cnt; j += kThreads) ks[j] = kp[lo + j];
  __syncthreads();
  for (int i = p0 + tid; i < p1; i += kThreads) {
    const int r = lower_bound_lds(ks, cnt, i);
    if (r < cnt && ks[r] == i) continue;  // kept
    out[i - (lo + r)] = i;                // i - (lo + r) < ne for an evicted i
  }
}

hipError_t launch_select_evicted(const Launch& L, const float* scores, int32_t* slots, int cap) {
  const int budget = L.cfg->budget_k;
  int32_t* kept = ws_ptr<int32_t>(L.wsp, L.ws.kept);
  if (budget > 0) {
    const hipError_t e = select_launch(L, scores, kept, slots, cap);
    if (e != hipSuccess) return e;
  }
  const int tiles = std::max(1, (L.geo.maxn + kEvTile - 1) / kEvTile);
  auto go = [&](auto kern) {
    kern<<<dim3(tiles, L.geo.U), kThreads, 0, L.stream>>>(L.geo, kept, budget, L.cfg->protect_last,
                                                          slots, cap);
  };
  if (select_narrow(L)) go(evicted_kernel<SelNarrow>);
  else go(evicted_kernel<SelWide>);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gather: a workgroup copies `rows` consecutive kept rows of one unit; each
// thread moves one 16-byte piece of UNR rows of K and of V per trip (all
// loads issued before the stores). STREAM: non-temporal loads and stores, for
// copies much larger than the caches.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool STREAM>
__device__ __forceinline__ u32x4 copy_load(const char* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  else return *reinterpret_cast<const u32x4*>(p);
}

template <bool STREAM>
__device__ __forceinline__ void copy_store(char* p, u32x4 x) {
  if constexpr (STREAM) __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(p));
  else *reinterpret_cast<u32x4*>(p) = x;
}

template <int ROWBYTES, bool STREAM>
__global__ __launch_bounds__(kThreads) void compact_kernel(Geo g, const int32_t* __restrict__ idx,
                                                           int budget, int rows, int esize,
                                                           const char* __restrict__ k,
                                                           const char* __restrict__ v,
                                                           char* __restrict__ ko,
                                                           char* __restrict__ vo) {
  constexpr int PIECES = ROWBYTES / 16;
  constexpr int RPT = kThreads / PIECES;  // rows per trip slice
  constexpr int UNR = 4;
  const int u = blockIdx.y;
  const int j0 = blockIdx.x * rows;
  const int jend = min(budget, j0 + rows);
  if (j0 >= jend) return;
  const Unit un = decode_unit(g, u);
  const int rr = threadIdx.x / PIECES, off = (threadIdx.x % PIECES) * 16;
  const char* kb = k + ((int64_t)un.l * g.ksl + (int64_t)un.h * g.ksh + un.t0 * g.kst) * esize + off;
  const char* vb = v + ((int64_t)un.l * g.vsl + (int64_t)un.h * g.vsh + un.t0 * g.vst) * esize + off;
  char* kob = ko + ((int64_t)un.b * g.oss + (int64_t)un.l * g.osl + (int64_t)un.h * g.osh) * esize + off;
  char* vob = vo + ((int64_t)un.b * g.oss + (int64_t)un.l * g.osl + (int64_t)un.h * g.osh) * esize + off;
  const int32_t* ix = idx + (int64_t)u * budget;
  const int64_t kst = g.kst * esize, vst = g.vst * esize, ost = g.osr * esize;
  for (int jb = j0; jb < jend; jb += UNR * RPT) {
    int32_t t[UNR];
#pragma unroll
    for (int q = 0; q < UNR; ++q) {
      const int j = jb + q * RPT + rr;
      t[q] = j < jend ? ix[j] : -1;
      if (t[q] >= un.n) t[q] = -1;  // a position outside the sequence
    }
    u32x4 a[UNR], b[UNR];
#pragma unroll
    for (int q = 0; q < UNR; ++q)
      if (t[q] >= 0) {
        a[q] = copy_load<STREAM>(kb + t[q] * kst);
        b[q] = copy_load<STREAM>(vb + t[q] * vst);
      }
#pragma unroll
    for (int q = 0; q < UNR; ++q)
      if (t[q] >= 0) {
        const int64_t j = jb + q * RPT + rr;
        copy_store<STREAM>(kob + j * ost, a[q]);
        copy_store<STREAM>(vob + j * ost, b[q]);
      }
  }
}

hipError_t launch_compact(const Launch& L, const int32_t* idx, const void* k, const void* v,
                          void* ko, void* vo) {
  const Geo& g = L.geo;
  const int budget = L.cfg->budget_k;
  if (budget == 0) return hipSuccess;
  const int esize = L.cfg->dtype == JACAP_DTYPE_BF16 ? 2 : 4;
  const int rowbytes = g.D * esize;
  // Rows per workgroup: 64 .. 1024, the most that keep >= 8192 workgroups.
  int rows = 64;
  while (rows < 1024 && (int64_t)g.U * ((budget + 2 * rows - 1) / (2 * rows)) >= 8192) rows *= 2;
  const dim3 grid((unsigned)((budget + rows - 1) / rows), g.U);
  auto go = [&](auto kern) {
    kern<<<grid, kThreads, 0, L.stream>>>(g, idx, budget, rows, esize, (const char*)k,
                                          (const char*)v, (char*)ko, (char*)vo);
  };
  // Non-temporal above 1 GiB of kept rows (K and V), far beyond L2 and MALL.
  const bool stream = 2 * (int64_t)g.U * budget * rowbytes > (int64_t(1) << 30);
  switch (rowbytes * 2 + (stream ? 1 : 0)) {
    case 256: go(compact_kernel<128, false>); break;
    case 257: go(compact_kernel<128, true>); break;
    case 512: go(compact_kernel<256, false>); break;
    case 513: go(compact_kernel<256, true>); break;
    case 1024: go(compact_kernel<512, false>); break;
    case 1025: go(compact_kernel<512, true>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace jacap
