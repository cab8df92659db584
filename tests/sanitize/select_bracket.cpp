// Counts, on the CPU, how often a unit of the selection's wide shape would fall
// through to the general path: the bracket of select_plan.hpp on random scores,
// with the sample, the ranks and the capacities that the kernel takes from it.
// Prints "tokens budget path share" per size; exits non-zero above the allowed share.
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <vector>

#include "select_plan.hpp"

using namespace jacap;

// The kernel's search: the top `rank` keys' threshold two bits at a time, stopping
// at a prefix that rank .. rank + slack keys reach.
static uint32_t rank_search(const std::vector<uint32_t>& k, uint32_t rank, uint32_t slack) {
  uint32_t T = 0;
  for (int bit = 30; bit >= 0; bit -= 2) {
    uint32_t n[4] = {0, 0, 0, 0};
    for (uint32_t d = 1; d <= 3; ++d)
      for (uint32_t x : k) n[d] += x >= (T | d << bit);
    const uint32_t d = n[3] >= rank ? 3 : n[2] >= rank ? 2 : n[1] >= rank ? 1 : 0;
    T |= d << bit;
    if (d > 0 && n[d] <= rank + slack) return T - 1;
  }
  return T;
}
static uint32_t at_rank(std::vector<uint32_t> k, int rank) {
  std::nth_element(k.begin(), k.begin() + (rank - 1), k.end(), std::greater<uint32_t>());
  return k[rank - 1];
}
static uint32_t key_of(float f) {
  uint32_t b;
  memcpy(&b, &f, 4);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}

// True: the unit's lists are enough.
static bool fits(const std::vector<uint32_t>& key, int kk) {
  const int n = (int)key.size();
  const SelPath path = sel_wide_path(n, kk);
  if (path == SelPath::kDirect || n <= kSelWideCand) return true;
  const int seg = path == SelPath::kSampled ? kSelSeg : 64;
  const SelBracket b = path == SelPath::kSampled ? sel_sampled_bracket(n, kk) : sel_bracket(n, kk, 64, 128);
  std::vector<uint32_t> sample;
  for (int e = 0; e < b.S; ++e) {
    const int p = e / seg * b.q * seg + e % seg;
    if (p >= n) { fprintf(stderr, "sample past the end\n"); return false; }
    sample.push_back(key[p]);
  }
  uint32_t lo, hi = 0xFFFFFFFFu;
  if (path == SelPath::kSampled) {
    lo = rank_search(sample, b.r_lo, sel_slack(b));
  } else {
    lo = at_rank(sample, b.r_lo);
    if (b.r_hi >= 1) hi = at_rank(sample, b.r_hi);
  }
  int64_t sure = 0, cand = 0;
  for (uint32_t k : key) {
    sure += k > hi;
    cand += k >= lo && k <= hi;
  }
  return sure < kk && sure + cand >= kk && sure <= kSelWideCand && cand <= kSelWideCand;
}

int main() {
  const int sizes[][2] = {{2049, 700}, {8192, 4096}, {8193, 1024}, {16384, 1024}, {16385, 8000}, {32768, 512},
                          {32768, 8192}, {65536, 4096}, {131072, 1024}, {131072, 4096}, {131072, 8192},
                          {200000, 4096}, {262144, 2048}, {262144, 4096}, {393216, 2048}, {524288, 2048},
                          {1048576, 1024}};
  std::mt19937 gen(11);
  std::normal_distribution<float> normal;
  int bad = 0;
  for (const auto& s : sizes) {
    const int n = s[0], kk = s[1], sets = n > 300000 ? 12 : 30;
    for (int kind = 0; kind < 2; ++kind) {   // independent scores; runs of 256 positions alike
      if (kind == 1 && n > 131072) continue;
      if (kind == 1 && kk > 1024) continue;  // (a larger sample too misses too many of the runs)
      int through = 0;
      for (int r = 0; r < sets; ++r) {
        std::vector<uint32_t> key(n);
        float run = 0.0f;
        for (int i = 0; i < n; ++i) {
          if (i % 256 == 0) run = kind ? 2.0f * normal(gen) : 0.0f;
          key[i] = key_of(expf(run + (kind ? 0.5f : 4.0f) * normal(gen)));
        }
        through += !fits(key, kk);
      }
      const char* names[] = {"direct", "sampled", "staged"};
      printf("%d %d %s kind %d: %d of %d through\n", n, kk, names[(int)sel_wide_path(n, kk)], kind, through, sets);
      if (through * 10 > sets * (kind ? 4 : 0)) ++bad;
    }
  }
  if (bad) return 1;
  printf("brackets ok\n");
  return 0;
}
