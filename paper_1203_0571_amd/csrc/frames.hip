// Front end on whole frames (Sec. 4.1, the paragraph on the starting point):
// the brightest pixel of each frame, r50 by summing the pixels outward from
// it until half the total flux, and the square of side 6 r50 around it cut
// out into a packed stamp batch.
//
// Detection without scratch memory runs one workgroup per frame
// (detect_kernel):
//   pass 0  border mean -> sky (FP64, fixed reduction order);
//   pass 1  one read of the frame: finiteness, brightest pixel (first index
//           among equals), total F = sum (I - sky) in FP64, max |I - sky|;
//   pass 2  ring sums about the peak over a square window of half-size R
//           (R = 16, 32, ... until the growth curve crosses F/2 or the window
//           covers the frame), in fixed point (int64 LDS atomics with a
//           power-of-two scale from max |I - sky|, so the sums do not depend
//           on the order of the atomics), rings r - 1 < d <= r, the peak
//           pixel counted with ring 1;
// then the crossing radius is interpolated and the box placed.  A frame is
// read about once: pass 2 touches only the window, typically a few r50.
//
// With scratch memory the read of the frames is a launch of its own
// (scan_kernel, any number of workgroups per frame, each leaving one partial
// record), and a workgroup per frame combines the records and runs pass 2
// (place_kernel).  One workgroup alone reads a frame at some 90 GB/s, so a
// few frames leave the card idle.
#include <type_traits>

#include "kernels.hpp"

namespace shape {
namespace {

constexpr int kFrameThreads = 256;
constexpr int kFrameWaves = kFrameThreads / kWave;
constexpr int kR0 = 16;

template <int DT>
__device__ __forceinline__ float frame_px(const shape_frames& f, int64_t base, int64_t k,
                                          float scale) {
  if constexpr (DT == SHAPE_F32) {
    return static_cast<const float*>(f.pixels)[base + k];
  } else {
    return static_cast<float>(static_cast<const _Float16*>(f.pixels)[base + k]) * scale;
  }
}

// Four consecutive pixels from a 4-aligned index (frames whose pixel count
// is a multiple of 4 on a 16-byte aligned buffer).
template <int DT>
__device__ __forceinline__ void load4(const shape_frames& f, int64_t base, int64_t k, float scale,
                                      float (&v)[4]) {
  if constexpr (DT == SHAPE_F32) {
    const float4 q = *reinterpret_cast<const float4*>(static_cast<const float*>(f.pixels) + base + k);
    v[0] = q.x;
    v[1] = q.y;
    v[2] = q.z;
    v[3] = q.w;
  } else {
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    const h4 q = *reinterpret_cast<const h4*>(static_cast<const _Float16*>(f.pixels) + base + k);
    v[0] = (float)q[0] * scale;
    v[1] = (float)q[1] * scale;
    v[2] = (float)q[2] * scale;
    v[3] = (float)q[3] * scale;
  }
}

// Sum over the workgroup in a fixed order (wave DPP sums, then waves 0..3).
__device__ __forceinline__ double block_sum(double v, double* red) {
  const int tid = threadIdx.x, w = tid / kWave;
  v = wave_sum(v);
  __syncthreads();
  if ((tid & (kWave - 1)) == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kFrameWaves; ++q) s += red[q];
  return s;
}

// Smallest r >= 0 with r^2 >= d2.
__device__ __forceinline__ int ceil_sqrt(int64_t d2) {
  int r = (int)ceil(sqrt((double)d2));
  while ((int64_t)r * r < d2) ++r;
  while (r > 0 && (int64_t)(r - 1) * (r - 1) >= d2) --r;
  return r;
}

// Where the growth curve crosses half the flux (LDS).
struct Crossing {
  int r;
  double prev, cum;
};

// Pass 2 and the box of frame fr, by one workgroup: sky, total F, largest
// |I - sky| and the brightest pixel (i0, j0) are known to every thread.
template <int DT>
__device__ __forceinline__ void place_box(const shape_frames& f, int64_t fr, float scale,
                                          double sky, double F, double mabs, int i0, int j0,
                                          int max_side, int nbins, long long* bins, Crossing& gc,
                                          float* info, int32_t* peak, int32_t* box,
                                          uint32_t* status) {
  uint32_t stt = 0;
  const int tid = threadIdx.x;
  const int H = f.height, W = f.width;
  const int64_t npix = (int64_t)H * W, base = fr * npix;
  const int mind = H < W ? H : W;
  double rr = 0.125 * mind;
  if (F > 0.0) {
    // fixed point: |sum| <= npix * mabs * scale < 2^62
    int ex;
    __builtin_frexp((double)npix * fmax(mabs, 1e-300), &ex);
    const double fs = __builtin_ldexp(1.0, 62 - ex);
    const double half = 0.5 * F;
    const int rmax = ceil_sqrt((int64_t)(H - 1) * (H - 1) + (int64_t)(W - 1) * (W - 1));
    int R = kR0;
    for (;;) {
      if (R > rmax) R = rmax;
      const int Rc = R + 1 < nbins ? R + 1 : nbins;
      for (int q = tid; q < Rc; q += kFrameThreads) bins[q] = 0;
      if (tid == 0) gc.r = -1;
      __syncthreads();
      const int ia = i0 - R > 0 ? i0 - R : 0, ib = i0 + R < H - 1 ? i0 + R : H - 1;
      const int ja = j0 - R > 0 ? j0 - R : 0, jb = j0 + R < W - 1 ? j0 + R : W - 1;
      const int ww = jb - ja + 1;
      const int nw = (ib - ia + 1) * ww;   // < 2^31 for sides up to 4096
      const int64_t R2 = (int64_t)R * R;
      for (int q = tid; q < nw; q += kFrameThreads) {
        const int i = ia + q / ww, j = ja + q % ww;
        const int64_t d2 = (int64_t)(i - i0) * (i - i0) + (int64_t)(j - j0) * (j - j0);
        if (d2 > R2) continue;
        const int r = ceil_sqrt(d2);
        const double d = (double)frame_px<DT>(f, base, (int64_t)i * W + j, scale) - sky;
        atomicAdd((unsigned long long*)&bins[r < 1 ? 1 : r],
                  (unsigned long long)__builtin_llrint(d * fs));
      }
      __syncthreads();
      // first crossing of F/2 by the growth curve C(r), r = 1..R (wave 0)
      if (tid < kWave) {
        long long carry = 0;
        for (int c0 = 1; c0 <= R; c0 += kWave) {
          const int r = c0 + tid;
          long long v = r <= R ? bins[r] : 0;
          // inclusive scan over the wave
          for (int o = 1; o < kWave; o <<= 1) {
            const long long u = __shfl_up(v, o);
            if (tid >= o) v += u;
          }
          const long long cum = carry + v;
          const bool hit = r <= R && (double)cum / fs >= half;
          const unsigned long long m = __ballot(hit);
          if (m) {
            const int l = __builtin_ctzll(m);
            if (tid == l) {
              const long long prev = cum - bins[r];
              gc.r = r;
              gc.prev = (r == 1) ? 0.0 : (double)prev / fs;
              gc.cum = (double)cum / fs;
            }
            break;
          }
          carry += __shfl(v, kWave - 1);
        }
      }
      __syncthreads();
      const int fr_r = gc.r;
      if (fr_r > 0) {
        rr = (fr_r - 1) + (half - gc.prev) / (gc.cum - gc.prev);
        break;
      }
      if (R >= rmax) {
        // rounding left the last ring a hair short of F/2: it crosses there
        rr = (double)rmax;
        break;
      }
      R *= 2;
      __syncthreads();
    }
  } else {
    stt |= SHAPE_ST_NONPOSITIVE_FLUX;
  }
  if (tid == 0) {
    int smax = max_side < mind ? max_side : mind;
    long long side = __builtin_llround(6.0 * rr);
    if (side < 4) side = 4;
    if (side > smax) side = smax;
    int ox = j0 - (int)side / 2, oy = i0 - (int)side / 2;
    if (ox > W - side) ox = W - (int)side;
    if (oy > H - side) oy = H - (int)side;
    if (ox < 0) ox = 0;
    if (oy < 0) oy = 0;
    info[fr * 3 + 0] = (float)sky;
    info[fr * 3 + 1] = (float)rr;
    info[fr * 3 + 2] = (float)F;
    peak[fr * 2 + 0] = j0;
    peak[fr * 2 + 1] = i0;
    box[fr * 3 + 0] = ox;
    box[fr * 3 + 1] = oy;
    box[fr * 3 + 2] = (int)side;
    status[fr] = stt;
  }
}

// A frame with a NaN or Inf pixel.
__device__ __forceinline__ void write_nonfinite(int64_t fr, float* info, int32_t* peak,
                                                int32_t* box, uint32_t* status) {
  info[fr * 3 + 0] = info[fr * 3 + 1] = info[fr * 3 + 2] = qnan();
  peak[fr * 2 + 0] = peak[fr * 2 + 1] = -1;
  box[fr * 3 + 0] = box[fr * 3 + 1] = box[fr * 3 + 2] = 0;
  status[fr] = SHAPE_ST_NONFINITE_INPUT;
}

template <int DT>
__global__ __launch_bounds__(kFrameThreads) void detect_kernel(shape_frames f, int max_side,
                                                               int nbins, bool vec4, float* info,
                                                               int32_t* peak, int32_t* box,
                                                               uint32_t* status) {
  extern __shared__ long long bins[];   // nbins
  __shared__ double red[kFrameWaves];
  __shared__ float bval[kFrameThreads];
  __shared__ int64_t bidx[kFrameThreads];
  __shared__ Crossing gc;
  const int tid = threadIdx.x;
  const int H = f.height, W = f.width;
  const int64_t npix = (int64_t)H * W;
  for (int64_t fr = blockIdx.x; fr < f.n; fr += gridDim.x) {
    const int64_t base = fr * npix;
    const float scale = (DT == SHAPE_F16_SCALED) ? f.scale[fr] : 1.0f;
    // pass 0: border mean
    const int nb = 2 * W + 2 * H - 4;
    double bs = 0.0;
    for (int q = tid; q < nb; q += kFrameThreads) {
      int64_t k;
      if (q < W) k = q;                                   // top row
      else if (q < 2 * W) k = (int64_t)(H - 1) * W + (q - W);   // bottom row
      else {
        const int r = q - 2 * W;                          // left, right columns
        const int row = 1 + (r >> 1);
        k = (int64_t)row * W + ((r & 1) ? W - 1 : 0);
      }
      bs += (double)frame_px<DT>(f, base, k, scale);
    }
    const double sky = block_sum(bs, red) / (double)nb;
    // pass 1: finiteness, brightest pixel, total, extent
    float best = -__builtin_inff();
    int64_t bk = npix;
    bool finite = true;
    double tot = 0.0, amax = 0.0;
    auto visit = [&](float v, int64_t k) {
      finite = finite && __builtin_isfinite(v);
      if (v > best) {  // each thread's k increases: ties keep the first index
        best = v;
        bk = k;
      }
      const double d = (double)v - sky;
      tot += d;
      amax = fmax(amax, fabs(d));
    };
    if (vec4) {
      // four pixels per load (16 B FP32 / 8 B FP16), four loads in flight
      const int64_t n4 = npix >> 2;
#pragma unroll 4
      for (int64_t q = tid; q < n4; q += kFrameThreads) {
        float v[4];
        load4<DT>(f, base, q * 4, scale, v);
#pragma unroll
        for (int c = 0; c < 4; ++c) visit(v[c], q * 4 + c);
      }
    } else {
      for (int64_t k = tid; k < npix; k += kFrameThreads) visit(frame_px<DT>(f, base, k, scale), k);
    }
    const bool all_finite = __syncthreads_and(finite);
    if (!all_finite) {
      if (tid == 0) write_nonfinite(fr, info, peak, box, status);
      __syncthreads();
      continue;
    }
    const double F = block_sum(tot, red);
    // max |I - sky| (exact: max is order independent)
    {
      double m = amax;
      for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o));
      if ((tid & (kWave - 1)) == 0) bins[tid / kWave] = __builtin_bit_cast(long long, m);
    }
    bval[tid] = best;
    bidx[tid] = bk;
    __syncthreads();
    for (int s = kFrameThreads / 2; s >= 1; s >>= 1) {
      if (tid < s) {
        const float v2 = bval[tid + s];
        const int64_t k2 = bidx[tid + s];
        if (v2 > bval[tid] || (v2 == bval[tid] && k2 < bidx[tid])) {
          bval[tid] = v2;
          bidx[tid] = k2;
        }
      }
      __syncthreads();
    }
    double mabs = 0.0;
#pragma unroll
    for (int q = 0; q < kFrameWaves; ++q)
      mabs = fmax(mabs, __builtin_bit_cast(double, bins[q]));
    const int64_t pk = bidx[0];
    const int i0 = (int)(pk / W), j0 = (int)(pk - (int64_t)i0 * W);
    __syncthreads();
    place_box<DT>(f, fr, scale, sky, F, mabs, i0, j0, max_side, nbins, bins, gc, info, peak, box,
                  status);
    __syncthreads();
  }
}

// ---- the read of the frames as a launch of its own -----------------------

// What one workgroup of scan_kernel found in its chunk of a frame.
struct FramePart {
  double sum, border;   // all pixels; those on the frame's border
  float vmax, vmin;
  int32_t imax;         // frame index of the first pixel equal to vmax
  int32_t pad;
};

// Vectors a thread of scan_kernel has in flight, and the pixels of the
// 16-byte vector of either storage.
constexpr int kScanDepth = 4;
template <int DT>
constexpr int kScanVec = DT == SHAPE_F32 ? 4 : 8;

// kScanVec pixels from any pixel on: the types ask for no more than the pixel's
// own alignment, and the vector is one load all the same.  FP32 frames of odd
// pixel counts lose nothing by it; FP16 vectors on odd addresses read slower
// (4,000 frames of 517 x 333 261 -> 311 us).
template <int DT>
__device__ __forceinline__ void load_vec(const void* p, float scale, float (&v)[kScanVec<DT>]) {
  if constexpr (DT == SHAPE_F32) {
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    const f4 q = *static_cast<const f4*>(p);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = q[c];
  } else {
    typedef _Float16 h8 __attribute__((ext_vector_type(8), aligned(2)));
    const h8 q = *static_cast<const h8*>(p);
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = (float)q[c] * scale;
  }
}

// Pass 1 of a chunk of a frame.  Bound by the read: per pixel it forms the
// FP64 sum (a convert and an add) and the FP32 extremes (half an instruction
// each), and nothing that needs the sky, which no chunk knows yet:
//   F = sum - npix sky, and the largest |I - sky| is that of an extreme;
//   a NaN or Inf pixel shows in the sum (finite FP32 pixels cannot overflow
//   an FP64 sum, and Inf - Inf is NaN).
// Of the brightest pixel a thread remembers only which of its batches first
// held it; the threads that hold the chunk's maximum look their batch up
// again.  The border is summed from the chunk's own rows, just read.
// Measured with place_kernel: 4,096 frames of 512 x 512 FP32 in 732 us (5.9
// TB/s; a 4 GiB device copy reaches 4.6), 797 us for detect_kernel; 4 frames of
// 2048 x 2048 in 22 us, 776 us for detect_kernel, whose four workgroups read 86
// GB/s.
template <int DT>
__global__ __launch_bounds__(kFrameThreads) void scan_kernel(shape_frames f, int64_t chunk,
                                                             int64_t chunks, FramePart* parts) {
  using E = typename std::conditional<DT == SHAPE_F32, float, _Float16>::type;
  constexpr int V = kScanVec<DT>;
  __shared__ double red[2][kFrameWaves];
  __shared__ float ext[2][kFrameWaves];
  __shared__ int first;
  const int tid = threadIdx.x, w = tid / kWave;
  const int W = f.width, H = f.height;
  const int64_t npix = (int64_t)H * W;
  for (int64_t id = blockIdx.x; id < f.n * chunks; id += gridDim.x) {
    const int64_t fr = id / chunks;
    const int a = (int)((id - fr * chunks) * chunk);
    const int e = (int)(a + chunk < npix ? a + chunk : npix);
    const float scale = (DT == SHAPE_F16_SCALED) ? f.scale[fr] : 1.0f;
    const E* fp = static_cast<const E*>(f.pixels) + fr * npix;
    // [a, vb) in vectors, wherever the frame lies in memory (its sums must not
    // depend on that), [vb, e) pixel by pixel
    const int nv = (e - a) / V, vb = a + nv * V;
    double sum[2] = {0.0, 0.0};
    float vmax = -__builtin_inff(), vmin = __builtin_inff();
    int at = -1;   // the batch of the maximum: its first vector, or -1: a single pixel
    int k1 = npix; // ... and that pixel
    auto single = [&](int k) {
      const float v = frame_px<DT>(f, fr * npix, k, scale);
      sum[0] += (double)v;
      vmin = fminf(vmin, v);
      if (v > vmax || (v == vmax && k < k1)) {
        vmax = v;
        k1 = k;
      }
    };
    if (tid < e - vb) single(vb + tid);
    constexpr int kStep = kFrameThreads * kScanDepth;
    float bmax = -__builtin_inff();
    for (int q = tid; q < nv; q += kStep) {
      float v[kScanDepth][V];
#pragma unroll
      for (int u = 0; u < kScanDepth; ++u) {
        // past the end: the batch's first vector again, left out of the sum
        const int qu = q + u * kFrameThreads;
        load_vec<DT>(fp + a + (int64_t)(qu < nv ? qu : q) * V, scale, v[u]);
      }
      float m = v[0][0];
#pragma unroll
      for (int u = 0; u < kScanDepth; ++u) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int c = 0; c < V; c += 2) {
          m = fmaxf(m, fmaxf(v[u][c], v[u][c + 1]));
          vmin = fminf(vmin, fminf(v[u][c], v[u][c + 1]));
          s0 += (double)v[u][c];
          s1 += (double)v[u][c + 1];
        }
        const bool in = q + u * kFrameThreads < nv;
        sum[0] += in ? s0 : 0.0;
        sum[1] += in ? s1 : 0.0;
      }
      if (m > bmax) {
        bmax = m;
        at = q;
      }
    }
    // the chunk's border pixels: rows 0 and H - 1 whole, the others' ends
    double border = 0.0;
    {
      const int ra = a / W, rb = (e - 1) / W;
      for (int r = ra + tid; r <= rb; r += kFrameThreads) {
        if (r == 0 || r == H - 1) continue;
        const int l = r * W, g = l + W - 1;
        if (l >= a) border += (double)frame_px<DT>(f, fr * npix, l, scale);
        if (g < e) border += (double)frame_px<DT>(f, fr * npix, g, scale);
      }
      const int top = min(e, W), bot = max(a, (H - 1) * W);
      for (int k = a + tid; k < top; k += kFrameThreads)
        border += (double)frame_px<DT>(f, fr * npix, k, scale);
      for (int k = bot + tid; k < e; k += kFrameThreads)
        border += (double)frame_px<DT>(f, fr * npix, k, scale);
    }
    // the workgroup's sums (waves in order) and extremes
    const double ws = wave_sum(sum[0] + sum[1]), wb = wave_sum(border);
    float wmax = fmaxf(vmax, bmax), wmin = vmin;
    for (int o = 32; o >= 1; o >>= 1) {
      wmax = fmaxf(wmax, __shfl_xor(wmax, o));
      wmin = fminf(wmin, __shfl_xor(wmin, o));
    }
    if ((tid & (kWave - 1)) == 0) {
      red[0][w] = ws;
      red[1][w] = wb;
      ext[0][w] = wmax;
      ext[1][w] = wmin;
    }
    if (tid == 0) first = (int)npix;
    __syncthreads();
    double tot = 0.0, tb = 0.0;
    float cmax = ext[0][0], cmin = ext[1][0];
#pragma unroll
    for (int q = 0; q < kFrameWaves; ++q) {
      tot += red[0][q];
      tb += red[1][q];
      cmax = fmaxf(cmax, ext[0][q]);
      cmin = fminf(cmin, ext[1][q]);
    }
    int k0 = vmax == cmax ? k1 : (int)npix;
    if (at >= 0 && bmax == cmax) {
#pragma unroll 1
      for (int u = kScanDepth - 1; u >= 0; --u) {
        const int qu = at + u * kFrameThreads;
        if (qu >= nv) continue;
        float v[V];
        load_vec<DT>(fp + a + (int64_t)qu * V, scale, v);
#pragma unroll
        for (int c = V - 1; c >= 0; --c)
          if (v[c] == cmax) k0 = min(k0, a + qu * V + c);
      }
    }
    if (k0 < npix) atomicMin(&first, k0);
    __syncthreads();
    if (tid == 0) parts[id] = {tot, tb, cmax, cmin, first, 0};
    __syncthreads();   // red, ext and first are rewritten by the next chunk
  }
}

// A frame's records combined (in chunk order within a thread, then over the
// threads in a fixed order), then pass 2.
template <int DT>
__global__ __launch_bounds__(kFrameThreads) void place_kernel(shape_frames f, int64_t chunks,
                                                              const FramePart* parts, int max_side,
                                                              int nbins, float* info,
                                                              int32_t* peak, int32_t* box,
                                                              uint32_t* status) {
  extern __shared__ long long bins[];   // nbins
  __shared__ double red[kFrameWaves];
  __shared__ float ext[2][kFrameWaves];
  __shared__ int first[kFrameWaves];
  __shared__ Crossing gc;
  const int tid = threadIdx.x, w = tid / kWave;
  const int H = f.height, W = f.width;
  const int64_t npix = (int64_t)H * W;
  for (int64_t fr = blockIdx.x; fr < f.n; fr += gridDim.x) {
    const FramePart* fp = parts + fr * chunks;
    double sum = 0.0, border = 0.0;
    float vmax = -__builtin_inff(), vmin = __builtin_inff();
    int im = (int)npix;
    for (int64_t c = tid; c < chunks; c += kFrameThreads) {
      const FramePart p = fp[c];
      sum += p.sum;
      border += p.border;
      vmin = fminf(vmin, p.vmin);
      if (p.vmax > vmax) {  // chunks in order: ties keep the first
        vmax = p.vmax;
        im = p.imax;
      }
    }
    for (int o = 32; o >= 1; o >>= 1) {
      const float v2 = __shfl_xor(vmax, o);
      const int i2 = __shfl_xor(im, o);
      if (v2 > vmax || (v2 == vmax && i2 < im)) {
        vmax = v2;
        im = i2;
      }
      vmin = fminf(vmin, __shfl_xor(vmin, o));
    }
    sum = block_sum(sum, red);
    border = block_sum(border, red);
    if ((tid & (kWave - 1)) == 0) {
      ext[0][w] = vmax;
      ext[1][w] = vmin;
      first[w] = im;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kFrameWaves; ++q) {
      if (ext[0][q] > vmax || (ext[0][q] == vmax && first[q] < im)) {
        vmax = ext[0][q];
        im = first[q];
      }
      vmin = fminf(vmin, ext[1][q]);
    }
    if (!__builtin_isfinite(sum)) {
      if (tid == 0) write_nonfinite(fr, info, peak, box, status);
      __syncthreads();
      continue;
    }
    const double sky = border / (double)(2 * W + 2 * H - 4);
    const double F = fma(-(double)npix, sky, sum);
    const double mabs = fmax(fabs((double)vmax - sky), fabs((double)vmin - sky));
    const int i0 = im / W, j0 = im - i0 * W;
    const float scale = (DT == SHAPE_F16_SCALED) ? f.scale[fr] : 1.0f;
    place_box<DT>(f, fr, scale, sky, F, mabs, i0, j0, max_side, nbins, bins, gc, info, peak, box,
                  status);
    __syncthreads();
  }
}

// Pixels a workgroup of scan_kernel reads: a frame is cut by its own size alone,
// so that its sums round alike however many frames it is measured with.  At
// most two batches of vectors per thread in FP32, four in FP16 (32 and 64 KiB),
// whole batches, about equal parts.  One batch costs large calls the workgroup's
// end, longer chunks cost a single frame its spread (us at 1 / 2 / 4 / 8 batches):
// 4,096 frames of 512 x 512 FP32 843 / 732 / 728 / 734, FP16 550 / 418 / 390 / 405; 4
// of 2048 x 2048 FP32 24 / 22 / 22 / 22, FP16 18 / 16 / 16 / 17; one of 512 x 512 FP32
// 11.3 / 10.9 / 12.5 / 13.6.
int64_t scan_chunk(const shape_frames& f) {
  const int64_t npix = (int64_t)f.height * f.width;
  const int64_t batch = (int64_t)kFrameThreads * kScanDepth * (f.dtype == SHAPE_F32 ? 4 : 8);
  const int64_t most = (f.dtype == SHAPE_F32 ? 2 : 4) * batch;
  const int64_t parts = (npix + most - 1) / most;
  const int64_t chunk = ((npix + parts - 1) / parts + batch - 1) / batch * batch;
  return chunk < npix ? chunk : npix;
}

// Exclusive prefix sum of side^2 over the boxes (one workgroup of 1024).
__global__ __launch_bounds__(1024) void offsets_kernel(const int32_t* box, int64_t n,
                                                       int64_t* offset, int64_t* total) {
  __shared__ long long part[1024 / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  long long carry = 0;
  for (int64_t c0 = 0; c0 < n; c0 += 1024) {
    const int64_t k = c0 + tid;
    const long long s = k < n ? (long long)box[k * 3 + 2] : 0;
    long long v = s * s;
    for (int o = 1; o < kWave; o <<= 1) {
      const long long u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    if (lane == kWave - 1) part[w] = v;
    __syncthreads();
    long long before = 0, all = 0;
    for (int q = 0; q < 1024 / kWave; ++q) {
      if (q < w) before += part[q];
      all += part[q];
    }
    if (k < n) offset[k] = carry + before + v - s * s;
    carry += all;
    __syncthreads();
  }
  if (tid == 0) *total = carry;
}

// Copy each box into the packed stamps (FP32), one workgroup per frame.
// A box outside its frame, or whose cut-out would not fit in the capacity,
// copies nothing and gets side 0 (its stamp is then rejected downstream).
template <int DT>
__global__ __launch_bounds__(kFrameThreads) void cut_kernel(shape_frames f, const int32_t* box,
                                                            const int64_t* offset, float* stamps,
                                                            int64_t capacity, int32_t* sides) {
  const int W = f.width;
  const int64_t npix = (int64_t)f.height * W;
  for (int64_t fr = blockIdx.x; fr < f.n; fr += gridDim.x) {
    const int ox = box[fr * 3 + 0], oy = box[fr * 3 + 1];
    int s = box[fr * 3 + 2];
    const int64_t o0 = offset[fr];
    const bool fits = s > 0 && ox >= 0 && oy >= 0 && ox <= W - s && oy <= f.height - s &&
                      o0 >= 0 && o0 <= capacity - (int64_t)s * s;
    if (!fits) s = 0;
    if (threadIdx.x == 0 && sides) sides[fr] = s;
    if (s == 0) continue;
    const float scale = (DT == SHAPE_F16_SCALED) ? f.scale[fr] : 1.0f;
    const int64_t base = fr * npix + (int64_t)oy * W + ox, o = o0;
    const int n = s * s;
    for (int q = threadIdx.x; q < n; q += kFrameThreads) {
      const int i = q / s, j = q - i * s;
      stamps[o + q] = frame_px<DT>(f, base, (int64_t)i * W + j, scale);
    }
  }
}

}  // namespace

int frame_bins(int height, int width) {
  // rings 0 .. ceil(sqrt((H-1)^2 + (W-1)^2))
  const double d = sqrt((double)(height - 1) * (height - 1) + (double)(width - 1) * (width - 1));
  return (int)ceil(d) + 2;
}

hipError_t launch_frame_detect(const shape_frames& f, int max_side, float* info, int32_t* peak,
                               int32_t* box, uint32_t* status, hipStream_t stream) {
  const int nbins = frame_bins(f.height, f.width);
  const size_t lds = (size_t)nbins * sizeof(long long);
  const int64_t grid = f.n < (1ll << 30) ? f.n : (1ll << 30);
  const int64_t npix = (int64_t)f.height * f.width;
  const size_t align = f.dtype == SHAPE_F32 ? 16 : 8;
  const bool vec4 = npix % 4 == 0 && reinterpret_cast<uintptr_t>(f.pixels) % align == 0;
  if (f.dtype == SHAPE_F32)
    hipLaunchKernelGGL(detect_kernel<SHAPE_F32>, dim3((unsigned)grid), dim3(kFrameThreads), lds,
                       stream, f, max_side, nbins, vec4, info, peak, box, status);
  else
    hipLaunchKernelGGL(detect_kernel<SHAPE_F16_SCALED>, dim3((unsigned)grid), dim3(kFrameThreads),
                       lds, stream, f, max_side, nbins, vec4, info, peak, box, status);
  return hipGetLastError();
}

size_t frame_workspace_bytes(const shape_frames& f) {
  const int64_t npix = (int64_t)f.height * f.width, chunk = scan_chunk(f);
  return (size_t)f.n * (size_t)((npix + chunk - 1) / chunk) * sizeof(FramePart);
}

hipError_t launch_frame_detect_ws(const shape_frames& f, int max_side, float* info, int32_t* peak,
                                  int32_t* box, uint32_t* status, void* ws, hipStream_t stream) {
  // Up to SHAPE_FRAME_WHOLE pixels one workgroup reads a frame as fast as two
  // launches do (us, one / split: 5,000 frames of 64 x 64 49 / 54, of 128 x 128 88 /
  // 93, of 192 x 192 155 / 158; 300 of 192 x 192 19 / 18, one 12.5 / 11; 300 of 256 x
  // 256 28 / 25).
  if ((int64_t)f.height * f.width <= SHAPE_FRAME_WHOLE)
    return launch_frame_detect(f, max_side, info, peak, box, status, stream);
  const int nbins = frame_bins(f.height, f.width);
  const size_t lds = (size_t)nbins * sizeof(long long);
  const int64_t cap = 1ll << 30;
  const int64_t chunk = scan_chunk(f), chunks = ((int64_t)f.height * f.width + chunk - 1) / chunk;
  const dim3 gs((unsigned)(f.n * chunks < cap ? f.n * chunks : cap));
  const dim3 gp((unsigned)(f.n < cap ? f.n : cap)), t(kFrameThreads);
  FramePart* parts = static_cast<FramePart*>(ws);
  if (f.dtype == SHAPE_F32) {
    hipLaunchKernelGGL(scan_kernel<SHAPE_F32>, gs, t, 0, stream, f, chunk, chunks, parts);
    hipLaunchKernelGGL(place_kernel<SHAPE_F32>, gp, t, lds, stream, f, chunks, parts, max_side,
                       nbins, info, peak, box, status);
  } else {
    hipLaunchKernelGGL(scan_kernel<SHAPE_F16_SCALED>, gs, t, 0, stream, f, chunk, chunks, parts);
    hipLaunchKernelGGL(place_kernel<SHAPE_F16_SCALED>, gp, t, lds, stream, f, chunks, parts,
                       max_side, nbins, info, peak, box, status);
  }
  return hipGetLastError();
}

hipError_t launch_frame_offsets(const int32_t* box, int64_t n, int64_t* offset, int64_t* total,
                                hipStream_t stream) {
  hipLaunchKernelGGL(offsets_kernel, dim3(1), dim3(1024), 0, stream, box, n, offset, total);
  return hipGetLastError();
}

hipError_t launch_frame_cut(const shape_frames& f, const int32_t* box, const int64_t* offset,
                            float* stamps, int64_t capacity, int32_t* sides, hipStream_t stream) {
  const int64_t grid = f.n < (1ll << 30) ? f.n : (1ll << 30);
  if (f.dtype == SHAPE_F32)
    hipLaunchKernelGGL(cut_kernel<SHAPE_F32>, dim3((unsigned)grid), dim3(kFrameThreads), 0,
                       stream, f, box, offset, stamps, capacity, sides);
  else
    hipLaunchKernelGGL(cut_kernel<SHAPE_F16_SCALED>, dim3((unsigned)grid), dim3(kFrameThreads), 0,
                       stream, f, box, offset, stamps, capacity, sides);
  return hipGetLastError();
}

}  // namespace shape
