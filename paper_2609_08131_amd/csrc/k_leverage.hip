// Leverage score of Eq. 10: score_i = w_i v_i^T A^{-1} v_i = w_i ||L^{-1} v_i||^2.
//
// bf16 inputs: Y = V L^{-T} on MFMA 16x16x32 bf16. The token dimension is the
// MFMA row dimension. V rows are read whole (each wave load covers complete
// 128-byte lines, streamed non-temporally, or cached for per-head GQA) and pass through a small
// wave-private LDS tile into the operand layout. L^{-1} is split into bf16
// hi + lo and kept in registers; only the K-blocks with b <= a of the lower
// triangle are multiplied. The squared row norm is reduced across the 16
// lanes that share a token.
//
// fp64 pass (every unit of fp32 inputs; the units of bf16 inputs that the
// factorisation sent to the fp64 path): the same product on the fp64 MFMA.
#include <algorithm>

#include "jacap_internal.hpp"

namespace jacap {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// POL: cache policy of the V loads (streamed, or kept in L2 for the other
// query-head units of the same KV head).
template <int D, int POL>
__global__ __launch_bounds__(kThreads, 2) void leverage_mfma_kernel(
    Geo g, const uint16_t* __restrict__ v, const float* __restrict__ wbuf,
    const uint16_t* __restrict__ lfrag, const uint32_t* __restrict__ uflags,
    float* __restrict__ scores, int lchunks, int lchunk) {
  constexpr int NB = D / 16;                    // output blocks of 16 channels (a)
  constexpr int NK = D / 32;                    // K blocks of 32 channels (b)
  constexpr int NLP = (NB / 2) * (NB / 2 + 1);  // lower (j, kb) block pairs
  int u, chunk;
  if (!grid_unit_chunk<true>(g, lchunks, u, chunk)) return;
  const Unit un = decode_unit(g, u);
  const int base = chunk * lchunk;
  if (base >= un.n) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ch = lane & 15, kg = lane >> 4;
  const int rl = 2 * (ch >> 3) + ((ch >> 2) & 1);  // token (of 4) whose score this lane ends with
  const int64_t trow = token_row(g, un);
  const int end = min(un.n, base + lchunk);

  const uint32_t uf = uflags[u];
  if (uf & kUnitRefine) return;  // scored by the fp64 pass
  if (uf & kUnitFailed) {  // unit failed (non-finite input): NaN scores
    for (int t = base + threadIdx.x; t < end; t += kThreads) scores[trow + t] = __builtin_nanf("");
    return;
  }

  // B fragments, pre-split by the factor kernel in lane order.
  bf16x8 bh[NLP], bl[NLP];
  const uint16_t* lf = lfrag + (int64_t)u * NLP * 2 * 64 * 8;
#pragma unroll
  for (int q = 0; q < NLP; ++q) {
    bh[q] = *reinterpret_cast<const bf16x8*>(lf + ((int64_t)(q * 2 + 0) * 64 + lane) * 8);
    bl[q] = *reinterpret_cast<const bf16x8*>(lf + ((int64_t)(q * 2 + 1) * 64 + lane) * 8);
  }
  drain_vmem();

  const uint16_t* vb = v + un.l * g.vsl + un.h * g.vsh + un.t0 * g.vst;

  // A step is 16 tokens (one MFMA row tile). V rows are prefetched two
  // steps ahead into three rotating register buffers (the loop is unrolled
  // by three so the buffers stay in fixed registers). A step's 16 rows are
  // read whole: each wave load brings RPL consecutive rows (d / 8 lanes per
  // row, 1 KB of contiguous lines, cache policy), through a buffer range
  // that ends at the chunk's last row (rows past it load as zeros and are not
  // stored), so every load is unconditional with a fixed per-lane offset and
  // the compiler's wait counts stay static. The rows then pass through a
  // wave-private LDS tile into the MFMA operand layout (lane (ch, kg) of
  // K-block kb: row ch, channels 32 kb + 8 kg .. + 7). MFMAs are issued
  // kb-outer so that consecutive MFMAs update different output blocks.
  // One prefetched step: the lane's V row pieces and the weight of the token
  // whose score this lane writes.
  struct Buf { uint4 a[NK]; float w; };
  // bytes per tile row: a 32-byte pad leaves the operand reads free of bank
  // conflicts, measured (16 bytes: 25 %)
  constexpr int PITCH = D * 2 + 32;
  __shared__ __attribute__((aligned(16))) char tiles[kThreads / 64][16 * PITCH];
  char* tile = tiles[wave];
  const int32_t vstb = (int32_t)g.vst * 2;
  constexpr int LPR = D / 8;                    // lanes per whole row (16 bytes each)
  constexpr int RPL = 64 / LPR;                 // rows per wave load
  static_assert(RPL * NK == 16, "a step's 16 rows in NK whole-row loads");
  const int rrow = lane / LPR, rpc = lane % LPR;  // row (of RPL) and 16-byte piece of a load
  int32_t voff[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) voff[i] = (RPL * i + rrow) * vstb + rpc * 16;
  const int32_t woff = (4 * kg + rl) * 4;
  const float* wb = wbuf + trow;
  auto load = [&](int t0, Buf& b) {
    const int32_t rows = min(end - t0, 16);
    const auto vr = buffer_range(vb + (int64_t)t0 * g.vst, rows_bytes(rows, vstb, D * 2));
#pragma unroll
    for (int i = 0; i < NK; ++i) b.a[i] = buffer_load16<POL>(vr, voff[i]);
    b.w = buffer_load_f32(buffer_range(wb + t0, max(rows, 0) * 4), woff);
    __builtin_amdgcn_sched_barrier(0);  // issue here, ahead of the MFMAs that follow
  };
  auto step = [&](int t0, const Buf& b) {
    const int tw = t0 + 4 * kg + rl;
    const float wt = b.w;
#pragma unroll
    for (int i = 0; i < NK; ++i)
      *reinterpret_cast<uint4*>(tile + (RPL * i + rrow) * PITCH + rpc * 16) = b.a[i];
    bf16x8 cur[NK];
#pragma unroll
    for (int kb = 0; kb < NK; ++kb)
      cur[kb] = *reinterpret_cast<const bf16x8*>(tile + ch * PITCH + kb * 64 + kg * 16);
    // Output blocks j = 2 jp and 2 jp + 1 share the K-block range kb <= jp:
    // their two accumulation chains are interleaved.
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jp = 0; jp < NB / 2; ++jp) {
      floatx4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f};
      const int q0 = jp * (jp + 1);             // pair index of (2 jp, 0)
      const int q1 = jp * (jp + 1) + (jp + 1);  // pair index of (2 jp + 1, 0)
#pragma unroll
      for (int kb = 0; kb <= jp; ++kb) {
        y0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur[kb], bh[q0 + kb], y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur[kb], bh[q1 + kb], y1, 0, 0, 0);
        y0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur[kb], bl[q0 + kb], y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur[kb], bl[q1 + kb], y1, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) ss[r] += y0[r] * y0[r] + y1[r] * y1[r];
    }
    // ss[r] is this lane's channel's part of token 4 kg + r; sum over the 16
    // lanes (channels) of the row by a transposing reduction: the row mirror
    // (ch <-> 15 - ch) leaves tokens 0, 1 to the lower half and 2, 3 to the
    // upper, the half-row mirror (ch <-> 7 - ch) one token per lane, and two
    // quad swaps finish; lane ch then holds token rl.
    const bool hi8 = ch >= 8, hi4 = (ch & 4) != 0;
    const float m0 = (hi8 ? ss[2] : ss[0]) + dpp_f32<kDppMirror>(hi8 ? ss[0] : ss[2]);
    const float m1 = (hi8 ? ss[3] : ss[1]) + dpp_f32<kDppMirror>(hi8 ? ss[1] : ss[3]);
    float sv = (hi4 ? m1 : m0) + dpp_f32<kDppHalfMirror>(hi4 ? m0 : m1);
    sv += dpp_f32<kDppQuadXor1>(sv);
    sv += dpp_f32<kDppQuadXor2>(sv);
    if ((ch & 3) == 0 && tw < end) scores[trow + tw] = wt * sv;
  };
  constexpr int WSTRIDE = 16 * (kThreads / 64);
  const int t_first = base + wave * 16;
  if (t_first >= end) return;
  Buf b0, b1, b2;
  load(t_first, b0);
  load(t_first + WSTRIDE, b1);
  for (int t0 = t_first; t0 < end; t0 += 3 * WSTRIDE) {
    load(t0 + 2 * WSTRIDE, b2);
    step(t0, b0);
    if (t0 + WSTRIDE >= end) break;
    load(t0 + 3 * WSTRIDE, b0);
    step(t0 + WSTRIDE, b1);
    if (t0 + 2 * WSTRIDE >= end) break;
    load(t0 + 4 * WSTRIDE, b1);
    step(t0 + 2 * WSTRIDE, b2);
  }
}

// ---------------------------------------------------------------------------
// fp64 leverage: every unit (fp32 inputs), or (MARKED) the marked units of bf16
// inputs, from their list. Y = L^{-1} V^T on the fp64 MFMA 16x16x4: rows are 16
// channels of a block J of L^{-1}, columns 16 tokens, and only the blocks
// B <= J of the lower triangle are multiplied.
//
// Bound by the fp64 matrix rate (144 MFMAs of 64 cycles per 16 tokens at
// d = 128). L^{-1} lies in LDS in the operand order of store_lower_f64 (72 KB:
// two workgroups per compute unit), two K-steps per conflict-free 16-byte read;
// each wave runs two tiles of 16 tokens against every value read, which
// halves the reads and gives two independent accumulation chains. V goes
// straight from global memory into the operand: K-step s of a 16-channel block
// takes lane (token r, q)'s channel 4 q + s of the block, so a lane reads four
// consecutive channels of its token; the next tiles are read a trip ahead.
//
// Measured (MI355X): 241 marked units of 8192 tokens, d = 128, bf16: 8.85 ms
// with eight threads per token on the fp64 VALU, both operands from LDS,
// 0.63 ms here (0.54 ms at the measured fp64 matrix rate of 72 TFLOP/s);
// 14 marked units of 2176 tokens among 4096: 2036 us and 19 us.
// ---------------------------------------------------------------------------
template <typename T, int D, bool MARKED>
__global__ __launch_bounds__(kThreads, 2) void leverage_f64_kernel(
    Geo g, const T* __restrict__ v, const float* __restrict__ wbuf,
    const double* __restrict__ xred, const uint32_t* __restrict__ uflags,
    const uint32_t* __restrict__ rcount, const int32_t* __restrict__ rlist,
    float* __restrict__ scores, int lchunks, int lchunk) {
  constexpr int NB = D / 16;
  constexpr int NPAIR = NB * (NB + 1) / 2;
  constexpr int TT = 2;                        // 16-token tiles per wave
  constexpr int TRIP = TT * 16 * (kThreads / 64);  // tokens per workgroup trip
  constexpr int WORDS = 4 * sizeof(T) / 4;     // 32-bit words of four channels
  // fp32 tiles are read after the previous trip: a second set of them would spill
  // (the bf16 one does at d = 128, 10 registers)
  constexpr bool AHEAD = sizeof(T) == 2;
  static_assert(TRIP == kLChunkPreciseMin, "the smallest chunk is one trip");
  __shared__ __attribute__((aligned(16))) double X[NPAIR * 256];
  int nu = g.U, nch = lchunks, tok = lchunk;
  if constexpr (MARKED) {
    nu = (int)*rcount;
    if (nu == 0) return;
    // about kLRefineItems items, in whole trips
    nch = min(max(kLRefineItems / nu, 1), (g.maxn + TRIP - 1) / TRIP);
    tok = ((g.maxn + nch - 1) / nch + TRIP - 1) / TRIP * TRIP;
    nch = (g.maxn + tok - 1) / tok;
  }
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t items = (int64_t)nu * nch;
  for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const int li = (int)(item / nch), chunk = (int)(item % nch);
    const int u = MARKED ? rlist[li] : li;
    const Unit un = decode_unit(g, u);
    const int base = chunk * tok;
    if (base >= un.n) continue;
    const int end = min(un.n, base + tok);
    const int64_t trow = token_row(g, un);
    if (uflags[u] & kUnitFailed) {  // non-finite input or singular A: NaN scores
      for (int t = base + tid; t < end; t += kThreads) scores[trow + t] = __builtin_nanf("");
      continue;
    }
    const T* vb = v + un.l * g.vsl + un.h * g.vsh + un.t0 * g.vst;
    const int32_t vstb = (int32_t)g.vst * (int32_t)sizeof(T);
    const int32_t voff = r16 * vstb + q4 * (int32_t)(4 * sizeof(T));
    struct Tiles { uint32_t v[TT][NB][WORDS]; float w[TT]; };
    // Rows past the chunk's end load as zeros and are not stored.
    auto load = [&](int t0, Tiles& tl) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        const int ts = t0 + 16 * tt;
        const int32_t rows = min(end - ts, 16);
        const auto vr = buffer_range(vb + (int64_t)ts * g.vst,
                                     rows_bytes(rows, vstb, D * (int32_t)sizeof(T)));
#pragma unroll
        for (int B = 0; B < NB; ++B)
          buffer_load_words<WORDS>(vr, voff + B * (int32_t)(16 * sizeof(T)), tl.v[tt][B]);
        tl.w[tt] = buffer_load_f32(buffer_range(wbuf + trow + ts, max(rows, 0) * 4), r16 * 4);
      }
      __builtin_amdgcn_sched_barrier(0);  // issued here, a trip ahead of their use
    };
    const int t_first = base + wave * TT * 16;
    Tiles nxt;
    load(t_first, nxt);
    __syncthreads();  // the previous item's X is no longer read
    {
      const double2* src = reinterpret_cast<const double2*>(xred + (int64_t)u * (NPAIR * 256));
      double2* dst = reinterpret_cast<double2*>(X);
#pragma unroll 6
      for (int e = tid; e < NPAIR * 128; e += kThreads) dst[e] = src[e];
    }
    __syncthreads();
    for (int t0 = t_first; t0 < end; t0 += TRIP) {
      double x[TT][NB][4];
      float w[TT];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        w[tt] = nxt.w[tt];
#pragma unroll
        for (int B = 0; B < NB; ++B)
#pragma unroll
          for (int s = 0; s < 4; ++s) x[tt][B][s] = word_elem<T, WORDS>(nxt.v[tt][B], s);
      }
      if constexpr (AHEAD) load(t0 + TRIP, nxt);  // empty past the chunk's end
      double ss[TT];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) ss[tt] = 0.0;
#pragma unroll
      for (int J = 0; J < NB; ++J) {
        f64x4 y[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) y[tt] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int B = 0; B <= J; ++B) {
          const double2* xp =
              reinterpret_cast<const double2*>(X + (J * (J + 1) / 2 + B) * 256) + lane;
          const double2 x0 = xp[0], x1 = xp[64];  // K-steps 0, 1 and 2, 3
          const double a[4] = {x0.x, x0.y, x1.x, x1.y};
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) y[tt] = mfma64(a[s], x[tt][B][s], y[tt]);
        }
        // y[i]: channel 16 J + 4 i + q4 of token r16
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
          for (int i = 0; i < 4; ++i) ss[tt] = fma(y[tt][i], y[tt][i], ss[tt]);
      }
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        ss[tt] += __shfl_xor(ss[tt], 16);
        ss[tt] += __shfl_xor(ss[tt], 32);
        const int t = t0 + 16 * tt + r16;
        if (q4 == 0 && t < end) scores[trow + t] = (float)((double)w[tt] * ss[tt]);
      }
      if constexpr (!AHEAD) load(t0 + TRIP, nxt);
    }
  }
}

hipError_t launch_leverage(const Launch& L, const void* v, float* scores) {
  const Geo& g = L.geo;
  const dim3 grid((unsigned)chunked_grid(g, L.ws.lchunks));
  const float* wb = ws_ptr<float>(L.wsp, L.ws.wgt);
  const uint32_t* uf = ws_ptr<uint32_t>(L.wsp, L.ws.uflags);
  if (L.ws.mfma) {
    const uint16_t* lf = ws_ptr<uint16_t>(L.wsp, L.ws.lfrag);
    auto go = [&](auto kern) {
      kern<<<grid, kThreads, 0, L.stream>>>(g, (const uint16_t*)v, wb, lf, uf, scores, L.ws.lchunks,
                                            L.ws.lchunk);
    };
    if (g.D == 128) {
      if (g.V > 1) go(leverage_mfma_kernel<128, kPolicyShared>);
      else go(leverage_mfma_kernel<128, kPolicyStream>);
    } else {
      if (g.V > 1) go(leverage_mfma_kernel<64, kPolicyShared>);
      else go(leverage_mfma_kernel<64, kPolicyStream>);
    }
  } else {
    return launch_leverage_precise(L, v, scores);
  }
  return hipGetLastError();
}

// fp64 leverage: every unit of fp32 inputs, or the marked units of bf16 inputs.
hipError_t launch_leverage_precise(const Launch& L, const void* v, float* scores) {
  const Geo& g = L.geo;
  const int64_t items = (int64_t)g.U * L.ws.plchunks;
  const unsigned blocks =
      (unsigned)std::min<int64_t>(items, L.ws.mfma ? kRefineBlocks : (int64_t(1) << 20));
  if (blocks == 0) return hipSuccess;
  auto go = [&](auto kern, auto vv) {
    kern<<<blocks, kThreads, 0, L.stream>>>(
        g, vv, ws_ptr<float>(L.wsp, L.ws.wgt), ws_ptr<double>(L.wsp, L.ws.gram_red),
        ws_ptr<uint32_t>(L.wsp, L.ws.uflags), ws_ptr<uint32_t>(L.wsp, L.ws.status) + 1,
        ws_ptr<int32_t>(L.wsp, L.ws.rlist), scores, L.ws.plchunks, L.ws.plchunk);
  };
  if (L.ws.mfma) {
    if (g.D == 128) go(leverage_f64_kernel<uint16_t, 128, true>, (const uint16_t*)v);
    else go(leverage_f64_kernel<uint16_t, 64, true>, (const uint16_t*)v);
  } else {
    if (g.D == 128) go(leverage_f64_kernel<float, 128, false>, (const float*)v);
    else go(leverage_f64_kernel<float, 64, false>, (const float*)v);
  }
  return hipGetLastError();
}

}  // namespace jacap
