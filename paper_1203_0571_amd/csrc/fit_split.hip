// The fused profile fit with a workgroup of four waves per stamp, for batches
// that leave the card's SIMDs short of waves: the same LM trials as fit_kernel
// with the same sums (split_sweep.hpp), so the same results bit for bit.
#include "kernels.hpp"
#include "lm.hpp"

namespace shape {
namespace {

// Up to which batch four waves per stamp are faster (us, one wave / four).  One
// side: while the card holds the batch at two or three workgroups per CU; with
// more, the repeated rendering costs more than the latency gained.  64 x 64 FP32:
// 64 stamps 330 / 214, 512 339 / 247, 768 348 / 302, 1,024 349 / 371; 48 x 48: 64
// stamps 233 / 178, 640 338 / 316, 768 341 / 345; 128 x 128: 256 stamps 1,598 /
// 1,126, 1,024 1,699 / 1,978.  Mixed sides: the pace is set by the few large
// stamps, and both models share one launch instead of two: 512 stamps 1,670 /
// 775, 2,048 2,364 / 1,063, 8,192 3,095 / 2,420, 12,000 3,330 / 3,324.
constexpr int64_t kSplitUniform = 640, kSplitMixed = 8192;

template <int DT, int MODEL, uint32_t MASK, int LAYOUT, bool PROF>
__device__ __forceinline__ void fit_split(const shape_batch& b, const KOpts& o, const Stamp& st,
                                          const float* p_init, const float* rec, int64_t s,
                                          LmShared& W, float* p_out, float* chi2,
                                          float* perr, int32_t* iters, uint32_t* status,
                                          int32_t* sweeps, int tid) {
  lm_start<DT, MODEL, MASK, kSplit, LAYOUT>(b, o, st, p_init, rec, s, W, nullptr, tid);
  while (!W.L.done && W.L.it < o.max_iter_lm)
    lm_iterate<DT, MODEL, MASK, kSplit, LAYOUT, PROF>(b, o, st, W, nullptr, tid);
  lm_finish<MODEL, MASK>(o, st, W.L, W.sums[W.cur], s, p_out, chi2, perr, iters, status, sweeps,
                         tid);
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
    if (tid < 8) {
      p_out[s * 8 + tid] = qnan();
      if (perr) perr[s * 8 + tid] = qnan();
    }
    if (tid == 0) {
      chi2[s] = qnan();
      iters[s] = 0;
      status[s] = st.bad;
      if (sweeps) sweeps[s] = 0;
    }
    return;
  }
  if (LAYOUT == kLayoutRows || !PROF || st.model == SHAPE_SERSIC) {
    fit_split<DT, SHAPE_SERSIC, MASK, LAYOUT, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2,
                                                    perr, iters, status, sweeps, tid);
  } else if constexpr (LAYOUT != kLayoutRows && PROF) {
    fit_split<DT, SHAPE_MOFFAT, MASK, LAYOUT, PROF>(b, o, st, p_init, rec, s, W, p_out, chi2,
                                                    perr, iters, status, sweeps, tid);
  }
}

template <int DT, uint32_t MASK, bool PROF>
void launch_layout(const shape_batch& b, const KOpts& o, const float* p_init, const float* rec,
                   float* p_out, float* chi2, float* perr, int32_t* iters, uint32_t* status,
                   int32_t* sweeps, hipStream_t stream) {
  const dim3 g((unsigned)b.n), t(kWave * kSplitWaves);
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

bool fit_takes_split(const shape_batch& b) { return b.n <= (b.side ? kSplitMixed : kSplitUniform); }

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
