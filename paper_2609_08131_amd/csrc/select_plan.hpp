// How the selection brackets its threshold from a sample, and which path a unit's
// sizes take: arithmetic on sizes alone, shared with the host (a test counts on
// the CPU how often a bracket's candidates would not fit).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace jacap {

// A sample of segments of SEG contiguous tokens, every q-th segment, and the
// sample ranks (1 = largest) of the bracket lo <= T <= hi: four standard deviations
// of the kk-th key's rank in the sample, and 16, either way.
struct SelBracket {
  int q, nseg, S;   // stride and number of the segments; sampled tokens
  int r_lo, r_hi;   // ranks of lo and hi; r_hi < 1: the band reaches the top of the sample
};
__host__ __device__ inline SelBracket sel_bracket(int n, int kk, int seg, int most) {
  SelBracket b;
  const int all = (n + seg - 1) / seg;
  b.q = (all + most - 1) / most;
  b.nseg = (all + b.q - 1) / b.q;
  const int last = n - (b.nseg - 1) * b.q * seg;   // the valid samples form a prefix
  b.S = (b.nseg - 1) * seg + (last < seg ? last : seg);
  const double ks = (double)kk * (double)b.S / (double)n;
  const int delta = (int)(4.0 * sqrt(ks)) + 16;
  const int kr = (int)(ks + 0.5) > 1 ? (int)(ks + 0.5) : 1;
  b.r_lo = kr + delta < b.S ? kr + delta : b.S;
  b.r_hi = kr - delta;
  return b;
}

// The wide shape (1024 threads, lists of kSelWideCand entries).
constexpr int kSelWideCand = 8192;
constexpr int kSelWideDirect = 2048;   // longest unit ranked from registers
constexpr int kSelSeg = 16;            // tokens per sampled segment of the sampled path
// Sample keys per thread of the sampled path.
__host__ __device__ constexpr int sel_sample_per(int n) { return n <= 16384 ? 1 : 2; }
__host__ __device__ inline SelBracket sel_sampled_bracket(int n, int kk) {
  return sel_bracket(n, kk, kSelSeg, 1024 * sel_sample_per(n) / kSelSeg);
}
// lo may be any key that up to this many more sample keys reach (a looser bound is
// found sooner).
__host__ __device__ constexpr int sel_slack(const SelBracket& b) { return b.r_lo / 8; }
// Candidates (every key >= lo) that the sampled path expects, at most, and the most of them
// that it is taken for: four per thread, half of their list.
constexpr int kSelSampledMost = 4096;
__host__ __device__ inline int64_t sel_sampled_band(int n, int kk) {
  const SelBracket b = sel_sampled_bracket(n, kk);
  return (int64_t)(b.r_lo + sel_slack(b)) * n / b.S;
}

// The paths (k_select.hip). Measured, sampled against staged (jacap_select): 8 units of
// 16384 tokens keeping 1024 20 and 27 us, of 131072 keeping 1024 44 and 66; beyond
// the line 256 units of 32768 keeping 4096 44 (with an upper bound) and 38 us, of 8192
// keeping 4096 28 and 18, and at 131072 keeping 8192 two units of three
// overflowed their list, 399 and 80 us. Up to 8192 tokens staged takes no sample.
enum class SelPath { kDirect, kSampled, kStaged };
__host__ __device__ inline SelPath sel_wide_path(int n, int kk) {
  if (n <= kSelWideDirect) return SelPath::kDirect;
  if (n <= kSelWideCand) return SelPath::kStaged;
  return sel_sampled_band(n, kk) <= kSelSampledMost ? SelPath::kSampled : SelPath::kStaged;
}

}  // namespace jacap
