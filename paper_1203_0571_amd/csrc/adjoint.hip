// chi^2 of given parameters (Sec. 4.1, eq. chi2) and its gradient by the
// adjoint of the render, one wave per stamp.
//
// With r_i = (d_i - m_i) / sigma the adjoint of pixel i is
//   dL/dm_i = -(2 / sigma) r_i dL/dchi2,
// and dL/dp_k = sum_i dL/dm_i dm_i/dp_k.  Render, Jacobian and sums are FP64
// (adjoint_sweep.hpp for the Sersic stamps of a batch of one larger side,
// sweep.hpp's FP64 instance for the others and for Moffat stamps, each a kernel
// of its own so that neither holds the other's registers): the FP32 rounding of
// the exponent b t is amplified where the gradient components cancel over the
// stamp, up to ~1e-4 of the largest component.  J^T J is summed only when it is
// asked for.
#include "kernels.hpp"
#include "adjoint_sweep.hpp"

namespace shape {
namespace {

// What the caller gets for a stamp that cannot be evaluated, by one thread.
template <bool GRAD>
__device__ __forceinline__ void write_nan(int64_t s, float* chi2, float* grad_p, float* jtj,
                                          float* jtr) {
  if (chi2) chi2[s] = qnan();
  if constexpr (GRAD) {
    for (int k = 0; k < 8; ++k) {
      grad_p[s * 8 + k] = qnan();
      if (jtr) jtr[s * 8 + k] = qnan();
    }
    if (jtj)
      for (int k = 0; k < 36; ++k) jtj[s * 36 + k] = qnan();
  }
}

// A stamp's parameters; false when one is not finite.
__device__ __forceinline__ bool read_params(const float* params, int64_t s, double (&p)[8]) {
  bool finite = true;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    p[k] = params[s * 8 + k];
    finite = finite && __builtin_isfinite(p[k]);
  }
  return finite;
}

// Reduce a wave's sums and write the stamp's outputs.
template <bool GRAD, bool JTJ>
__device__ __forceinline__ void write_sums(const Acc<GRAD ? 0xFFu : 0u, double>& acc,
                                           const Stamp& st, int64_t s, const float* grad_chi2,
                                           float* chi2, float* grad_p, float* jtj, float* jtr,
                                           int lane) {
  // chi^2 and J^T r: one pass of FP64 wave sums over 12 values (every lane
  // receives the totals)
  double u[12];
  u[0] = acc.c2;
  if constexpr (GRAD) {
#pragma unroll
    for (int k = 0; k < 8; ++k) u[1 + k] = acc.g[k];
    u[9] = u[10] = u[11] = 0.0;
    wave_sum_n(u);
  } else {
    // chi^2 alone, by the same tree of additions
    double v[4] = {acc.c2, 0.0, 0.0, 0.0};
    wave_sum_n(v);
    u[0] = v[0];
  }
  const double inv2 = 1.0 / (st.sigma * st.sigma);
  if (lane == 0) {
    if (chi2) chi2[s] = (float)(u[0] * inv2);
    if constexpr (GRAD) {
      const double up = grad_chi2 ? (double)grad_chi2[s] : 1.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        grad_p[s * 8 + k] = (float)(-2.0 * up * u[1 + k] * inv2);
        if (jtr) jtr[s * 8 + k] = (float)(u[1 + k] * inv2);
      }
    }
  }
  if constexpr (JTJ) {
    double v[36];
#pragma unroll
    for (int k = 0; k < 36; ++k) v[k] = acc.A[k];
    wave_sum_n(v);
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < 36; ++k)
        jtj[s * 36 + k] = (k == tri(7, 7)) ? (float)(st.npix * inv2) : (float)(v[k] * inv2);
    }
  }
}

// The Sersic stamps of a batch, `chunk` to a workgroup of one wave.  GRAD: also
// J^T r (the gradient); JTJ: also J^T J (the normal matrix).  Waves per SIMD:
// with the gradient 3 (64 x 64 FP32 660 us; 4 spill more per stamp: 695, and 16 x
// 16 314 -> 379; 2: 744), with J^T J 2, for chi^2 alone 5.
template <int DT, bool GRAD, bool JTJ>
__global__ __launch_bounds__(kWave, JTJ ? 2 : GRAD ? 3 : 5) void chi2_tables_kernel(
    shape_batch b, const float* params, const float* grad_chi2, float* chi2, float* grad_p,
    float* jtj, float* jtr, int chunk) {
  __shared__ SersicTables<kChi2Chunk<GRAD>> tab;
  const int lane = threadIdx.x;
  bool general = false;   // whether the general sweep's tables are filled
  sersic_tables_fill(tab, lane);
  for (int64_t s0 = (int64_t)blockIdx.x * chunk; s0 < b.n; s0 += (int64_t)gridDim.x * chunk) {
    const int n = (int)(b.n - s0 < chunk ? b.n - s0 : chunk);
    wave_sync();   // the previous chunk's constants have been read
    if (lane < n) {
      const int64_t s = s0 + lane;
      const Stamp st = stamp_info(b, s);
      int todo = kSkip;   // the other model's launch owns it
      if (st.bad || st.model == SHAPE_SERSIC) {
        double p[8];
        if (!read_params(params, s, p) || st.bad) {
          write_nan<GRAD>(s, chi2, grad_p, jtj, jtr);
        } else {
          tab.t[lane] = make_trial<double, false>(p, SHAPE_SERSIC, 0.0);
          todo = sersic_covered(p, st.side) ? kCovered : kGeneral;
        }
      }
      tab.todo[lane] = todo;
    }
    wave_sync();
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
      const int todo = __builtin_amdgcn_readfirstlane(tab.todo[i]);
      if (todo == kSkip) continue;
      const Stamp st = stamp_info(b, s0 + i);
      Acc<GRAD ? 0xFFu : 0u, double> acc;
      // (expected: else the general sweep's registers spill in the covered one)
      if (__builtin_expect(todo == kCovered, 1)) {
        sersic_sweep<DT, GRAD, JTJ>(b, st, tab, tab.t[i], lane, acc);
      } else {
        if (!general) f64_tables_fill(lane, kWave);
        general = true;
        wave_sync();
        sweep<DT, SHAPE_SERSIC, GRAD ? 0xFFu : 0u, kWave, double, kLayoutAny, JTJ>(b, st, tab.t[i],
                                                                                  acc);
      }
      write_sums<GRAD, JTJ>(acc, st, s0 + i, grad_chi2, chi2, grad_p, jtj, jtr, lane);
    }
  }
}

// The stamps of one model, one wave per stamp (sweep.hpp in FP64): Moffat
// stamps, and the Sersic stamps of batches that do not take the tables.  With
// J^T J, FP16 stamps' rolled loops fit three waves per SIMD.
template <int DT, int MODEL, bool GRAD, bool JTJ>
__global__ __launch_bounds__(kWave, JTJ ? (DT == SHAPE_F32 ? 2 : 3) : 5) void chi2_kernel(
    shape_batch b, const float* params, const float* grad_chi2, float* chi2, float* grad_p,
    float* jtj, float* jtr) {
  constexpr uint32_t EM = GRAD ? 0xFFu : 0u;
  const int lane = threadIdx.x;
  f64_tables_fill(lane, kWave);   // the FP64 log2 / exp2 tables
  wave_sync();
  for (int64_t s = blockIdx.x; s < b.n; s += gridDim.x) {
    const Stamp st = stamp_info(b, s);
    if (!st.bad && st.model != MODEL) continue;  // the other model's launch owns it
    if (st.bad && MODEL != SHAPE_SERSIC) continue;
    double p[8];
    if (!read_params(params, s, p) || st.bad) {
      if (lane == 0) write_nan<GRAD>(s, chi2, grad_p, jtj, jtr);
      continue;
    }
    Acc<EM, double> acc;
    // a side that divides 64 takes the column-per-lane layout (the geometry
    // as per-column quadratics), any other side the lane-stride walk
    const Trial<double> tr = make_trial<double>(p, MODEL, p[5]);
    if (rows_layout_fits(st.side))
      sweep<DT, MODEL, EM, kWave, double, kLayoutRows, JTJ>(b, st, tr, acc);
    else
      sweep<DT, MODEL, EM, kWave, double, kLayoutAny, JTJ>(b, st, tr, acc);
    write_sums<GRAD, JTJ>(acc, st, s, grad_chi2, chi2, grad_p, jtj, jtr, lane);
  }
}

// Whether the Sersic stamps of a batch take the tables: those of a batch of one
// side, from 48 on, however many, so that a stamp's results do not depend on its
// batch.  A stamp's own tables and a workgroup's cost 600 instructions, which
// small stamps earn back in large batches only.  Time against chi2_kernel's over
// 16 to 20,000 stamps (chi^2, gradient, normal matrix; FP32 and FP16): side 48
// 0.75-1.05, 0.70-0.86, 0.76-0.97; 52 to 64 0.73-1.06, 0.70-0.86, 0.76-0.95; 44
// 0.83-1.14, 0.79-0.99, 0.88-1.08; 36 0.93-1.28, 0.86-1.16, 0.94-1.18; 28 1.02-1.47,
// 0.90-1.27, 0.98-1.31.  Mixed sides would need both kernels, each passing over
// the other's stamps (100 stamps of side 24 11 -> 14 us, 20,000 46 -> 60), or one
// that holds both sweeps (20,000 46 -> 69).
constexpr int kTablesSide = 48;
bool takes_tables(const shape_batch& b) { return !b.side && b.side0 >= kTablesSide; }

template <int DT, bool GRAD, bool JTJ>
hipError_t launch_dt(const shape_batch& b, const float* params, const float* grad_chi2,
                     float* chi2, float* grad_p, float* jtj, float* jtr, hipStream_t stream) {
  const dim3 g((unsigned)(b.n < (1ll << 30) ? b.n : (1ll << 30))), t(kWave);
  if (takes_tables(b)) {
    // chunks of up to kChi2Chunk stamps that still make 8,192 workgroups, a few
    // rounds over the card
    constexpr int64_t most = kChi2Chunk<GRAD>;
    const int64_t fair = b.n / 8192, chunk = fair < 1 ? 1 : fair > most ? most : fair;
    const int64_t groups = (b.n + chunk - 1) / chunk, cap = 1ll << 25;
    hipLaunchKernelGGL((chi2_tables_kernel<DT, GRAD, JTJ>),
                       dim3((unsigned)(groups < cap ? groups : cap)), t, 0, stream, b, params,
                       grad_chi2, chi2, grad_p, jtj, jtr, (int)chunk);
  } else {
    hipLaunchKernelGGL((chi2_kernel<DT, SHAPE_SERSIC, GRAD, JTJ>), g, t, 0, stream, b, params,
                       grad_chi2, chi2, grad_p, jtj, jtr);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !b.model) return e;
  hipLaunchKernelGGL((chi2_kernel<DT, SHAPE_MOFFAT, GRAD, JTJ>), g, t, 0, stream, b, params,
                     grad_chi2, chi2, grad_p, jtj, jtr);
  return hipGetLastError();
}

template <int DT>
hipError_t launch_forms(const shape_batch& b, const float* params, const float* grad_chi2,
                        float* chi2, float* grad_p, float* jtj, float* jtr, bool grad,
                        hipStream_t stream) {
  if (!grad) return launch_dt<DT, false, false>(b, params, grad_chi2, chi2, grad_p, jtj, jtr, stream);
  if (jtj) return launch_dt<DT, true, true>(b, params, grad_chi2, chi2, grad_p, jtj, jtr, stream);
  return launch_dt<DT, true, false>(b, params, grad_chi2, chi2, grad_p, jtj, jtr, stream);
}

// grad_p = grad_chi2 (per stamp) x grad_unit, eight entries per stamp.
__global__ __launch_bounds__(256) void grad_scale_kernel(const float* grad_unit,
                                                        const float* grad_chi2, int64_t n,
                                                        float* grad_p) {
  const int64_t m = n * 8;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
       i += (int64_t)gridDim.x * blockDim.x)
    grad_p[i] = grad_chi2 ? grad_chi2[i >> 3] * grad_unit[i] : grad_unit[i];
}

}  // namespace

hipError_t launch_grad_scale(const float* grad_unit, const float* grad_chi2, int64_t n,
                             float* grad_p, hipStream_t stream) {
  const int64_t blocks = (n * 8 + 255) / 256;
  const unsigned grid = (unsigned)(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(grad_scale_kernel, dim3(grid), dim3(256), 0, stream, grad_unit, grad_chi2, n,
                     grad_p);
  return hipGetLastError();
}

hipError_t launch_chi2(const shape_batch& b, const float* params, const float* grad_chi2,
                       float* chi2, float* grad_p, float* jtj, float* jtr, bool grad,
                       hipStream_t stream) {
  if (b.dtype == SHAPE_F32)
    return launch_forms<SHAPE_F32>(b, params, grad_chi2, chi2, grad_p, jtj, jtr, grad, stream);
  return launch_forms<SHAPE_F16_SCALED>(b, params, grad_chi2, chi2, grad_p, jtj, jtr, grad, stream);
}

}  // namespace shape
