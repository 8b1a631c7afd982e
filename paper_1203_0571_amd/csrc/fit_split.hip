// The fused profile fit with a workgroup of four waves per stamp, for batches
// that leave the card's SIMDs short of waves, and for the largest stamps of
// middling batches of mixed sides: the same LM trials as fit_kernel with the same
// sums (split_sweep.hpp), so the same results bit for bit.
#include "kernels.hpp"
#include "lm.hpp"

namespace shape {
namespace {

// Which batches take four waves per stamp: those that the card holds at two or
// three workgroups per CU; with more, the repeated rendering costs more than the
// latency gained.  One side, one wave / four (us): 64 x 64 FP32 64 stamps 330 / 214,
// 512 339 / 247, 640 344 / 280, 1,024 349 / 371; 48 x 48 64 stamps 233 / 178, 640
// 338 / 316, 1,024 342 / 400; 128 x 128 256 stamps 1,598 / 1,126, 640 1,667 / 1,449,
// 1,024 1,699 / 1,978; 32 x 32 with (Re, n, I0, sky) free 640 135 / 113, 1,024 138 /
// 134; small sides with all eight free 12 x 12 320 133 / 131, 640 139 / 151, 6 x 6
// 320 119 / 123.
constexpr int64_t kSplitUniform = 640;

// Mixed sides above that, up to kSplitMixed stamps: the few large stamps set the
// pace, so only stamps of a side above 1.5 times the root of the mean area are
// split, the others taken by one wave each (fit_uneven_kernel), and both models
// share one launch.  Stamps of nearly equal sides, of which none is split, must
// not lose by it: where the mean is so large that none could be
// (kSplitMost), and in short fits of small stamps, fit_kernel stays.  Against
// fit_kernel (us): log-uniform sides 16 to 128 1,024 stamps 2,134 / 912, 2,048 2,811 /
// 1,290, 8,192 3,338 / 2,180; all of side 24 1,024 195 / 161, 4,096 315 / 297, 8,192
// 454 / 460, 48 8,192 846 / 851, 64 8,192 1,340 / 1,390; with (Re, n, I0, sky) free
// log-uniform 8,192 1,997 / 1,354, side 24 2,048 152 / 146, 4,096 180 / 193, 48 8,192
// 494 / 510.
constexpr int64_t kSplitMixed = 8192;
constexpr int kSplitMost = 104;

// Pixels of a stamp on average (with a side array at most: the buffer may hold
// more than the stamps).
double mean_area(const shape_batch& b) {
  return b.side ? (double)b.n_pixels / (double)b.n : (double)b.side0 * b.side0;
}
bool split_all(const shape_batch& b, const KOpts& o) {
  const double area = mean_area(b);
  if (o.free_mask != kMaskAll || area >= 16 * 16) return b.n <= kSplitUniform;
  return area >= 8 * 8 && b.n <= kSplitUniform / 2;
}
// The side above which a stamp of a batch of mixed sides is split.
int split_side(const shape_batch& b) {
  return (int)fmin(fmax(1.5 * sqrt(mean_area(b)), kSegsMinSide - 1.0), kMaxSide);
}
bool split_some(const shape_batch& b, const KOpts& o) {
  const bool brief = o.free_mask != kMaskAll && mean_area(b) < 40 * 40;
  return b.side && b.n <= (brief ? kSplitMixed / 4 : kSplitMixed) && split_side(b) <= kSplitMost;
}

// A stamp that cannot be processed.
__device__ __forceinline__ void write_bad(uint32_t bad, int64_t s, float* p_out, float* chi2,
                                          float* perr, int32_t* iters, uint32_t* status,
                                          int32_t* sweeps, int tid) {
  if (tid < 8) {
    p_out[s * 8 + tid] = qnan();
    if (perr) perr[s * 8 + tid] = qnan();
  }
  if (tid == 0) {
    chi2[s] = qnan();
    iters[s] = 0;
    status[s] = bad;
    if (sweeps) sweeps[s] = 0;
  }
}

// Workgroup s fits stamp s, of either model.
template <int DT, uint32_t MASK, int LAYOUT, bool PROF>
__global__ __launch_bounds__(kWave * kSplitWaves) void fit_split_kernel(
    shape_batch b, KOpts o, const float* p_init, const float* rec, float* p_out, float* chi2,
    float* perr, int32_t* iters, uint32_t* status, int32_t* sweeps) {
  __shared__ LmShared W;
  const int tid = threadIdx.x;
  const int64_t s = blockIdx.x;   // the grid is b.n
  const Stamp st = stamp_info(b, s);
  if (st.bad) {
    write_bad(st.bad, s, p_out, chi2, perr, iters, status, sweeps, tid);
    return;
  }
  if (LAYOUT == kLayoutRows || !PROF || st.model == SHAPE_SERSIC) {
    lm_fit<DT, SHAPE_SERSIC, MASK, kSplit, LAYOUT, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2,
                                                         perr, iters, status, sweeps, tid);
  } else if constexpr (LAYOUT != kLayoutRows && PROF) {
    lm_fit<DT, SHAPE_MOFFAT, MASK, kSplit, LAYOUT, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2,
                                                         perr, iters, status, sweeps, tid);
  }
}

// The same for a batch of mixed sides that fills the card with one wave per
// stamp: only the stamps of a side above `big`, far larger than the others, are
// split, since the batch waits for them; the first wave takes the others alone.
template <int DT, uint32_t MASK, bool PROF>
__global__ __launch_bounds__(kWave * kSplitWaves, 4) void fit_uneven_kernel(
    shape_batch b, KOpts o, const float* p_init, const float* rec, float* p_out, float* chi2,
    float* perr, int32_t* iters, uint32_t* status, int32_t* sweeps, int big) {
  __shared__ LmShared W;
  const int tid = threadIdx.x;
  const int64_t s = blockIdx.x;   // the grid is b.n
  const Stamp st = stamp_info(b, s);
  if (st.bad) {
    write_bad(st.bad, s, p_out, chi2, perr, iters, status, sweeps, tid);
    return;
  }
  const bool split = st.side > big;
  if (!split && __builtin_amdgcn_readfirstlane(tid / kWave) > 0) return;
  auto fit = [&](auto model) {
    constexpr int M = decltype(model)::value;
    if (split)
      lm_fit<DT, M, MASK, kSplit, kLayoutSegsOnly, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2,
                                                         perr, iters, status, sweeps, tid);
    else if (st.side >= kSegsMinSide)
      lm_fit<DT, M, MASK, 1, kLayoutSegsOnly | kLayoutFloorFree, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2, perr,
                                                    iters, status, sweeps, tid);
    else
      lm_fit<DT, M, MASK, 1, kLayoutAny | kLayoutFloorFree, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2, perr,
                                               iters, status, sweeps, tid);
  };
  if (!PROF || st.model == SHAPE_SERSIC)
    fit(std::integral_constant<int, SHAPE_SERSIC>());
  else if constexpr (PROF)
    fit(std::integral_constant<int, SHAPE_MOFFAT>());
}

template <int DT, uint32_t MASK, bool PROF>
void launch_layout(const shape_batch& b, const KOpts& o, const float* p_init, const float* rec,
                   float* p_out, float* chi2, float* perr, int32_t* iters, uint32_t* status,
                   int32_t* sweeps, hipStream_t stream) {
  const dim3 g((unsigned)b.n), t(kWave * kSplitWaves);
  if (!split_all(b, o)) {
    const int big = split_side(b);
    hipLaunchKernelGGL((fit_uneven_kernel<DT, MASK, PROF>), g, t, 0, stream, b, o, p_init, rec,
                       p_out, chi2, perr, iters, status, sweeps, big);
    return;
  }
  // (with a model array both models take the same layout)
  switch (single_wave_layout(b, SHAPE_SERSIC)) {
    case kLayoutRows:
      hipLaunchKernelGGL((fit_split_kernel<DT, MASK, kLayoutRows, PROF>), g, t, 0, stream, b, o,
                         p_init, rec, p_out, chi2, perr, iters, status, sweeps);
      break;
    case kLayoutAny:
      hipLaunchKernelGGL((fit_split_kernel<DT, MASK, kLayoutAny, PROF>), g, t, 0, stream, b, o,
                         p_init, rec, p_out, chi2, perr, iters, status, sweeps);
      break;
    default:
      hipLaunchKernelGGL((fit_split_kernel<DT, MASK, kLayoutSegs, PROF>), g, t, 0, stream, b, o,
                         p_init, rec, p_out, chi2, perr, iters, status, sweeps);
  }
}

template <int DT>
hipError_t launch_dt(const shape_batch& b, const KOpts& o, const float* p_init, const float* rec,
                     float* p_out, float* chi2, float* perr, int32_t* iters, uint32_t* status,
                     int32_t* sweeps, hipStream_t stream) {
  if (!o.linear_init)
    launch_layout<DT, kMaskSize, false>(b, o, p_init, rec, p_out, chi2, perr, iters, status,
                                        sweeps, stream);
  else if (o.free_mask == kMaskAll)
    launch_layout<DT, kMaskAll, true>(b, o, p_init, rec, p_out, chi2, perr, iters, status, sweeps,
                                      stream);
  else
    launch_layout<DT, kMaskSize, true>(b, o, p_init, rec, p_out, chi2, perr, iters, status, sweeps,
                                       stream);
  return hipGetLastError();
}

}  // namespace

bool fit_takes_split(const shape_batch& b, const KOpts& o) {
  return split_all(b, o) || split_some(b, o);
}

hipError_t launch_fit_split(const shape_batch& b, const KOpts& o, const float* p_init,
                            const float* rec, float* p_out, float* chi2, float* perr,
                            int32_t* iters, uint32_t* status, int32_t* sweeps, hipStream_t stream) {
  if (b.dtype == SHAPE_F32)
    return launch_dt<SHAPE_F32>(b, o, p_init, rec, p_out, chi2, perr, iters, status, sweeps,
                                stream);
  return launch_dt<SHAPE_F16_SCALED>(b, o, p_init, rec, p_out, chi2, perr, iters, status, sweeps,
                                     stream);
}

}  // namespace shape
