// The FP32 sweep of one stamp split over a workgroup of four waves, with the
// sums of the one-wave sweep bit for bit: for batches too small to fill the
// card, where a stamp's latency counts and not its instructions.
//
// A lane of the one-wave sweep sums its pixels in order, and its FP32 sums
// round in that order, so its pixels cannot be dealt out to several lanes.
// The sums can: every wave runs sweep() over the whole stamp for one of the
// four kinds of sums (kSumsShape ..), with the one wave's operations, and
// reduces its own.  The rendering of each pixel is repeated in every wave.
//
// Bound by instruction issue of one wave per SIMD, about 4.4 cycles each.
// Cycles per sweep (256 stamps; one wave / this): 48 x 48 19,600 / 14,400, 64 x 64
// 19,900 / 11,400, 128 x 128 115,700 / 78,600.  Handing the rendered quantities
// over in LDS instead of repeating the rendering took 9,300, 13,900 and 99,700
// with every wave rendering a quarter of the pixels, and 11,700, 12,800 and
// 82,800 with two waves rendering and two summing: the LDS traffic to the
// readers, a barrier per chunk and the start of the pipeline cost more on all
// but the smaller stamps.
#pragma once

#include "sweep.hpp"

namespace shape {

constexpr int kSplitWaves = 4;

// The sums of one wave, as indices into the reduced sums (0: chi^2, 1 + k:
// (J^T r)_k, 9 + tri(k, l): (J^T J)_kl), in the order it reduces them.
template <uint32_t EM, uint32_t SUMS>
struct SplitEntries {
  int n = 0;
  int at[16] = {};
  __host__ __device__ constexpr SplitEntries() {
    if (SUMS == kSumsGradient) {
      at[n++] = 0;
      for (int a = 0; a < 8; ++a)
        if (has(EM, a)) at[n++] = 1 + a;
    }
    for (int a = 0; a < 7; ++a)
      for (int c = a; c < 8; ++c)
        if (has(EM, a) && has(EM, c) && in_sums(SUMS, a, c)) at[n++] = 9 + tri(a, c);
  }
};

// Reduce a wave's sums over its lanes and store them at dst, with the
// reduction trees of reduce_store.
template <uint32_t EM, uint32_t SUMS>
__device__ __forceinline__ void reduce_split(const Acc<EM>& acc, double* dst, int lane) {
  using V = typename std::conditional<SUMS == kSumsGradient, double, float>::type;
  constexpr SplitEntries<EM, SUMS> E;
  auto value = [&](int i) -> V {
    if constexpr (SUMS == kSumsGradient)
      return i == 0 ? acc.c2 : acc.g[i - 1];
    else
      return acc.A[i - 9];
  };
  if constexpr (popcount(EM) >= 6) {
    // halving: row k of 16 lanes ends with entries k Q .. k Q + Q - 1
    constexpr int N = (E.n + 3) / 4 * 4, Q = N / 4;
    V v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = i < E.n ? value(E.at[i]) : (V)0;
#pragma unroll
    for (int j = 0; j < N / 2; ++j) swap_add32(v[j], v[j + N / 2]);
#pragma unroll
    for (int j = 0; j < Q; ++j) swap_add16(v[j], v[j + Q]);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      v[j] = dpp::add<dpp::kShr1, 0xf>(v[j]);
      v[j] = dpp::add<dpp::kShr2, 0xf>(v[j]);
      v[j] = dpp::add<dpp::kShr4, 0xf>(v[j]);
      v[j] = dpp::add<dpp::kShr8, 0xf>(v[j]);
    }
    const int row = lane >> 4;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      auto at = [&](int e) { return e < E.n ? E.at[e] : -1; };
      const int i = row == 0 ? at(j) : row == 1 ? at(Q + j) : row == 2 ? at(2 * Q + j) : at(3 * Q + j);
      if ((lane & 15) == 15 && i >= 0) dst[i] = (double)v[j];
    }
  } else {
#pragma unroll
    for (int i = 0; i < E.n; ++i) {
      const V v = wave_sum(value(E.at[i]));
      if (lane == 0) dst[E.at[i]] = (double)v;
    }
  }
}

// One sweep at trial t by the workgroup (LAYOUT: the one-wave sweep's); the
// reduced sums are left in S (LDS, kSums doubles, but for the pixel count).
// Callers synchronise the workgroup before and after.
template <int DT, int MODEL, uint32_t EM, int LAYOUT>
__device__ __forceinline__ void split_sweep(const shape_batch& b, const Stamp& st, const TrialF& t,
                                            double* S, int tid) {
  const int lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave);
  auto one = [&](auto sums) {
    constexpr uint32_t kSet = decltype(sums)::value;
    if constexpr (SplitEntries<EM, kSet>().n > 0) {
      Acc<EM> acc;
      sweep<DT, MODEL, EM, kWave, float, LAYOUT, true, kSet>(b, st, t, acc, lane);
      reduce_split<EM, kSet>(acc, S, lane);
    }
  };
  switch (w) {
    case 0: one(std::integral_constant<uint32_t, kSumsShape>()); break;
    case 1: one(std::integral_constant<uint32_t, kSumsCross>()); break;
    case 2: one(std::integral_constant<uint32_t, kSumsProfile>()); break;
    default: one(std::integral_constant<uint32_t, kSumsGradient>());
  }
}

}  // namespace shape
