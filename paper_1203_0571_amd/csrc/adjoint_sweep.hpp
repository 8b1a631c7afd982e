// The FP64 sweep of a Sersic stamp at given parameters: chi^2, J^T r and
// J^T J, by one wave.
//
// Bound by FP64 issue, so what a pixel costs is the series of its powers and
// logarithm.  Instead of t = (R / Re)^(1/n) as an exp2 of a log2 and t / R^2 by a
// reciprocal, both come from one product
//   t / R^2 = E_e C_j (1 + r)^beta,  R^2 = 2^e c_j (1 + r),  beta = 1 / 2n - 1,
// with c_j the centre of the j-th of 128 intervals of [1, 2), |r| < 1/256: the
// stamp's tables E_e = 2^(beta e) Re^(-1/n) (64 exponents, one per lane) and
// C_j = c_j^beta, and the binomial series to r^5 (the first dropped term is
// below 4e-15).  ln(1 + r) to r^5 gives the logarithm of the n column from the
// same r (dropped: below 6e-16), and m0 = e^(-b t) takes the 64-point exp2
// table with its series to degree 4 (4e-14).  No reciprocal, and the constant
// factors are applied after the sweep.
//
// Any side takes the moment form: the wave's work is cut into items, an item a
// run of rows of one pixel column (sersic_parts to a column), lane l taking
// items l, l + 64, ...: along an item u1 is fixed, so R^2 is a quadratic in u2,
// and the four shape columns are h times forms in (u1, u2) of degree 1 and 2.
// The pixels sum h u2^j and h^2 u2^j, an item adds these times powers of u1 to
// the stamp's sums, and the forms' coefficients are applied once per stamp.
//
// Measured against the lane-stride or row-layout sweep by 64-point log2 and
// exp2 tables, one wave per stamp (us; chi^2 / with gradient / with the normal
// matrix): 65,536 of 64 x 64 FP32 585 / 812 / 1,178 -> 469 / 666 / 978, FP16
// 573 / 788 / 1,099 -> 434 / 621 / 947; 20,000 of 48 x 48 FP16 129 / 185 / 255 ->
// 97 / 130 / 213; 8,000 of 128 x 128 FP32 354 / 491 / 723 -> 228 / 313 / 446.
// Smaller stamps and mixed sides keep that sweep (adjoint.hip).  On the 64 x 64
// FP32 batch the counters give 47, 70 and 107 VALU instructions per pixel, the
// work per stamp and per item among them, issued in 0.75, 0.76 and 0.79 of the
// SIMDs' slots of four cycles (a loop of FP64 FMAs on registers reaches 0.84).
#pragma once

#include "sweep.hpp"

namespace shape {

constexpr int kPowTab = 128;        // intervals of [1, 2)
constexpr int kPowExp = 64;         // binary exponents kPowExpLo .. + 63
constexpr int kPowExpLo = -25;
constexpr int kAhead = 4;           // rows loaded ahead of their use

// Stamps a workgroup takes at most: a stamp's constants (b(n) by its series, a
// logarithm, reciprocals: some 400 instructions and a chain of loads) are
// formed for all of them at once, one per lane.  Four for chi^2 alone, whose five
// waves per SIMD leave a workgroup 8 KB of LDS.
template <bool GRAD>
constexpr int kChi2Chunk = GRAD ? 8 : 4;
enum SersicDo { kSkip = 0, kCovered = 1, kGeneral = 2 };

// LDS of the sweep: the tables every stamp uses, and the stamp's.
template <int CHUNK>
struct SersicTables {
  double ex[kF64Tab];               // 2^(j / 64) / 24
  // 2 / c_j, log2 c_j - 1 and the stamp's c_j^beta (one address for all three)
  struct Interval {
    double rcp, log, pow, pad;
  } at[kPowTab];
  double E[kPowExp];                // the stamp's, at the exponent's low bits
  // the constants of a chunk of stamps, formed one stamp per lane, and what to
  // do with each (SersicDo)
  Trial<double> t[CHUNK];
  int todo[CHUNK];
};

template <int CHUNK>
__device__ __forceinline__ void sersic_tables_fill(SersicTables<CHUNK>& tab, int lane) {
  for (int j = lane; j < kF64Tab; j += kWave)
    tab.ex[j] = exp2_series(j / (double)kF64Tab) * (1.0 / 24.0);
  for (int j = lane; j < kPowTab; j += kWave) {
    const double c = 1.0 + (j + 0.5) / kPowTab;
    tab.at[j].rcp = 2.0 / c;
    tab.at[j].log = log2_series(c) - 1.0;
  }
}

// An entry of an LDS table at a byte offset.
template <typename T>
__device__ __forceinline__ const T& at_byte(const T* table, uint32_t byte) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(table) + byte);
}

// A wave-uniform value kept in vector registers (an instruction takes one
// operand from scalar registers).
__device__ __forceinline__ double in_vgpr(double v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Parts of a column for each side: the count, of at most 8, whose items fill the
// wave's lanes at the least cost, a row at 1 and an item's own work (column
// constants, recombination) at 2 rows.  Sides 64 and 128 fill them
// exactly; 48 takes 4 parts (3 rounds of 12 rows), 100 takes 5 (8 rounds of 20).
struct SersicParts {
  uint8_t of[kMaxSide + 1] = {};
  constexpr SersicParts() {
    for (int w = kMinSide; w <= kMaxSide; ++w) {
      int best = 0;
      for (int p = 1; p <= 8 && p <= w; ++p) {
        const int rows = (w + p - 1) / p;
        if (rows * (p - 1) >= w) continue;   // an empty last part
        const int cost = (w * p + kWave - 1) / kWave * (rows + 2);
        if (best == 0 || cost < best) {
          best = cost;
          of[w] = (uint8_t)p;
        }
      }
    }
  }
};
static __constant__ const SersicParts kSersicParts;

// Whether the tables and the moment form cover the stamp: positive sizes in the
// ranges the series are cut for, and R^2 of every pixel between 2^-24 (above the
// model's floor) and 2^38.  The ellipse's axes bound R^2 by |u|^2 (1 - e) / (1 + e)
// and |u|^2 (1 + e) / (1 - e).  Where the ellipse is long, the shape columns' sums
// cancel in the forms' coefficients: J^T J from the moments is good to its FP32
// rounding (6e-8) up to e = 0.95, but off by up to 3e-7 of an entry at 0.98, 2e-5 at
// 0.995 and 1e-2 at 0.9995.  Other stamps take the general sweep, whose columns are
// formed per pixel (6e-8 at every e).
__device__ __forceinline__ bool sersic_covered(const double* p, int side) {
  const double e = sqrt(p[2] * p[2] + p[3] * p[3]);
  if (!(e < 0.95 && p[4] >= 1e-3 && p[4] <= 1e5 && p[5] >= 0.1 && p[5] <= 20.0)) return false;
  const double ratio = (1.0 - e) / (1.0 + e), last = side - 1;
  const double dx = p[0] - fmin(fmax(rint(p[0]), 0.0), last);
  const double dy = p[1] - fmin(fmax(rint(p[1]), 0.0), last);
  const double mx = fmax(fabs(p[0]), fabs(p[0] - last)), my = fmax(fabs(p[1]), fabs(p[1] - last));
  return (dx * dx + dy * dy) * ratio >= 0x1p-24 && mx * mx + my * my <= 0x1p38 * ratio;
}

// The powers of a pixel at R^2: t, t / R^2, m0 and log2 R^2.
struct SersicPowers {
  double t, tr, m0, L;
};

// The wave's sums over a Sersic stamp that the tables cover: c2 = sum r^2, g = J^T r
// (GRAD), A = J^T J (JTJ), per lane.
template <int DT, bool GRAD, bool JTJ>
__device__ __forceinline__ void sersic_sweep(const shape_batch& b, const Stamp& st,
                                             SersicTables<kChi2Chunk<GRAD>>& tab,
                                             const Trial<double>& t, int lane,
                                             Acc<GRAD ? 0xFFu : 0u, double>& acc) {
  auto uni = [](double v) { return Arith<double>::uni(v); };
  // The constants are read from LDS where they are used, so that the pixel loop
  // holds only its own (all in registers they spilled).
  const double beta = uni(t.ha - 1.0), I0 = uni(t.I0), k5a = uni(t.k5a), qa = uni(t.qa);
  const double sky = in_vgpr(t.sky), k5b = in_vgpr(t.k5b);
  wave_sync();   // the previous stamp's reads of the tables are done
  const int e0 = kPowExpLo + lane;
  tab.E[(e0 + 1023) & (kPowExp - 1)] = exp2_series(fma(beta, (double)e0, t.hc));
#pragma unroll 1
  for (int j = lane; j < kPowTab; j += kWave)
    tab.at[j].pow = exp2_series(beta * (tab.at[j].log + 1.0));
  wave_sync();
  // binomial coefficients of (1 + r)^beta
  const double b2 = uni(beta * (beta - 1.0) * 0.5), b3 = uni(b2 * (beta - 2.0) * (1.0 / 3.0));
  const double b4 = in_vgpr(b3 * (beta - 3.0) * 0.25), b5 = uni(b4 * (beta - 4.0) * 0.2);
  const double zb = uni(t.nb2 * kLn2);                  // -b
  const double zk = uni(t.nb2 * (double)kF64Tab);       // -b log2 e 64
  const double tmax = -740.0 / (t.nb2 * kLn2);
  // The sums: gs, Xs and Ys of the shape columns as sums of h u1, h u2, h u1^2, h u1 u2, h u2^2
  // times r, the Re, n and I0 columns, and 1; Ms of h^2 over the forms of degree
  // 2, 3 and 4
  double c2 = 0.0, gs[5] = {}, g4 = 0.0, g5 = 0.0, g6 = 0.0, g7 = 0.0, A[9] = {};
  double Xs[3][5] = {}, Ys[5] = {}, Ms[12] = {};

  const int W = st.side, P = kSersicParts.of[W], rows = (W + P - 1) / P, items = W * P;
  const bool even = rows * P == W && items % kWave == 0;   // every lane has `rows` rows
  using E = typename std::conditional<DT == SHAPE_F32, float, _Float16>::type;
  const char* sp = static_cast<const char*>(stamp_base<DT>(b, st));
#pragma unroll 1
  for (int i0 = 0; i0 < items; i0 += kWave) {
    const int it = i0 + lane < items ? i0 + lane : items - 1, part = it / W, col = it - part * W;
    const int r0 = part * rows;
    // rows of this lane's item (none past the last item)
    const int nr = i0 + lane >= items ? 0 : W - r0 < rows ? W - r0 : rows;
    const double u1 = (double)col - t.x0;
    // the item's H_j = h u2^j (j = 0..2) against r; h^2 u2^s; against Re, n, I0; alone
    double mg[3] = {}, mM[5] = {}, mX[3][3] = {}, mY[3] = {};
    double u2 = (double)r0 - t.y0;
    const double qb = t.qb1 * u1, qc = t.qc2 * (u1 * u1);
    auto pixel = [&](float raw) {
      const double R2 = fma(fma(qa, u2, qb), u2, qc);
      SersicPowers w;
      const uint32_t hi = (uint32_t)(__builtin_bit_cast(uint64_t, R2) >> 32);
      // the interval (7 bits of the fraction) and the exponent's low 6 bits
      const auto& iv = at_byte(tab.at, (hi >> 8) & ((kPowTab - 1) * 32u));
      const double Ee = at_byte(tab.E, (hi >> 17) & ((kPowExp - 1) * 8u));
      const double r = fma(__builtin_amdgcn_frexp_mant(R2), iv.rcp, -1.0);
      const double pw = fma(fma(fma(fma(fma(b5, r, b4), r, b3), r, b2), r, beta), r, 1.0);
      w.tr = Ee * iv.pow * pw;
      w.t = w.tr * R2;
      // m0 = e^z, z = -b t = K ln 2 / 64 + y (cut at z = -740, where m0 c is 0);
      // 24 e^y = 24 + 24 y + 12 y^2 + 4 y^3 + y^4: two of the constants are
      // free as operands
      const double tc = fmin(w.t, tmax), K = __builtin_rint(zk * tc);
      const int ki = (int)K;
      const double y = fma(K, -kLn2 / kF64Tab, zb * tc);
      const double ey = fma(fma(fma(y + 4.0, y, 12.0), y, 24.0), y, 24.0);
      w.m0 = __builtin_ldexp(at_byte(tab.ex, ((uint32_t)ki << 3) & ((kF64Tab - 1) * 8u)) * ey,
                             ki >> 6);
      if constexpr (GRAD) {
        // log2 R^2 = e + log2 c_j + log2 e ln(1 + r), 4 ln(1 + r) / r in q
        const double q = fma(fma(fma(fma(0.8, r, -1.0), r, 4.0 / 3.0), r, -2.0), r, 4.0);
        w.L = fma(r * q, 0.25 * kLog2e, (double)__builtin_amdgcn_frexp_exp(R2) + iv.log);
      }
      const double m0 = w.m0;
      const double d = residual<DT>(raw, st.scale, fma(I0, m0, sky));
      c2 = fma(d, d, c2);
      if constexpr (GRAD) {
        const double c = m0 * w.t, h = m0 * w.tr, jn = c * fma(w.L, k5a, k5b);
        const double h1 = h * u2, h2 = h1 * u2;
        const double H[3] = {h, h1, h2};
#pragma unroll
        for (int k = 0; k < 3; ++k) mg[k] = fma(H[k], d, mg[k]);
        g4 = fma(c, d, g4);
        g5 = fma(jn, d, g5);
        g6 = fma(m0, d, g6);
        g7 += d;
        if constexpr (JTJ) {
#pragma unroll
          for (int q = 0; q < 5; ++q)
            mM[q] = fma(H[q < 3 ? q : 2], H[q < 3 ? 0 : q - 2], mM[q]);
          const double J[3] = {c, jn, m0};
#pragma unroll
          for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int v = 0; v < 3; ++v) mX[v][k] = fma(H[k], J[v], mX[v][k]);
            mY[k] += H[k];
          }
          // (Re, n, I0) among themselves, and their sums
          A[0] = fma(c, c, A[0]);
          A[1] = fma(c, jn, A[1]);
          A[2] = fma(c, m0, A[2]);
          A[3] += c;
          A[4] = fma(jn, jn, A[4]);
          A[5] = fma(jn, m0, A[5]);
          A[6] += jn;
          A[7] = fma(m0, m0, A[7]);
          A[8] += m0;
        }
      }
      u2 += 1.0;
    };
    // Rows are loaded kAhead ahead, in groups of kAhead whose rows the scheduler
    // may not mix (mixed, the series' temporaries spill).
    const uint32_t down = (uint32_t)(W * sizeof(E)), first = (uint32_t)((r0 * W + col) * sizeof(E));
    const uint32_t last = first + (nr > 1 ? nr - 1 : 0) * down;
    uint32_t byte = first;
    E ahead[kAhead];
    auto load = [&](int k) {
      ahead[k] = *reinterpret_cast<const E*>(sp + byte);
      byte = byte + down < last ? byte + down : last;
    };
#pragma unroll
    for (int k = 0; k < kAhead; ++k) load(k);
    int q = 0;
    if (even) {   // wave-uniform
#pragma unroll 1
      for (; q + kAhead <= rows; q += kAhead) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
          const float raw = (float)ahead[k];
          load(k);
          pixel(raw);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll 1
    for (; q < rows; q += kAhead) {
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const float raw = (float)ahead[k];
        load(k);
        if (q + k < nr) pixel(raw);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (GRAD) {
      const double uu = u1 * u1;
      auto add = [&](double (&sum)[5], const double (&m)[3]) {
        sum[0] = fma(u1, m[0], sum[0]);
        sum[1] += m[1];
        sum[2] = fma(uu, m[0], sum[2]);
        sum[3] = fma(u1, m[1], sum[3]);
        sum[4] += m[2];
      };
      add(gs, mg);
      if constexpr (JTJ) {
#pragma unroll
        for (int v = 0; v < 3; ++v) add(Xs[v], mX[v]);
        add(Ys, mY);
        const double up[5] = {1.0, u1, uu, uu * u1, uu * uu};
        int k = 0;
#pragma unroll
        for (int d = 2; d <= 4; ++d)
#pragma unroll
          for (int j = 0; j <= d; ++j, ++k)
            Ms[k] = j == d ? Ms[k] + mM[j] : fma(up[d - j], mM[j], Ms[k]);
      }
    }
  }
  acc.c2 = c2;
  if constexpr (GRAD) {
    // shape column a is k7 times the form sum_j C[a][j] u1^(d-j) u2^j, of degree
    // d = 1 for the centre and 2 for the ellipticity
    const double k7 = t.k7, k4 = t.k4;
    const double C[4][3] = {{t.n11 * k7, t.n12 * k7, 0.0},
                            {t.n12 * k7, t.n22 * k7, 0.0},
                            {fma(t.e1, t.qc2, -t.a11) * k7, t.e1 * t.qb1 * k7, t.p2a * k7},
                            {fma(t.e2, t.qc2, -t.a12) * k7, fma(t.e2, t.qb1, -2.0) * k7, t.p3a * k7}};
    auto form = [&](int a, const double (&sum)[5]) {
      return a < 2 ? fma(C[a][0], sum[0], C[a][1] * sum[1])
                   : fma(C[a][0], sum[2], fma(C[a][1], sum[3], C[a][2] * sum[4]));
    };
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      acc.g[a] = form(a, gs);
      if constexpr (JTJ) {
        acc.A[tri(a, 4)] = k4 * form(a, Xs[0]);
        acc.A[tri(a, 5)] = form(a, Xs[1]);
        acc.A[tri(a, 6)] = form(a, Xs[2]);
        acc.A[tri(a, 7)] = form(a, Ys);
#pragma unroll
        for (int c = a; c < 4; ++c) {
          const int da = a < 2 ? 1 : 2, dc = c < 2 ? 1 : 2;
          const int at = da + dc == 2 ? 0 : da + dc == 3 ? 3 : 7;
          double q = 0.0;
#pragma unroll
          for (int i = 0; i <= da; ++i)
#pragma unroll
            for (int j = 0; j <= dc; ++j) q = fma(C[a][i] * C[c][j], Ms[at + i + j], q);
          acc.A[tri(a, c)] = q;
        }
      }
    }
    acc.g[4] = k4 * g4;
    acc.g[5] = g5;
    acc.g[6] = g6;
    acc.g[7] = g7;
    if constexpr (JTJ) {
      acc.A[tri(4, 4)] = k4 * k4 * A[0];
      acc.A[tri(4, 5)] = k4 * A[1];
      acc.A[tri(4, 6)] = k4 * A[2];
      acc.A[tri(4, 7)] = k4 * A[3];
      acc.A[tri(5, 5)] = A[4];
      acc.A[tri(5, 6)] = A[5];
      acc.A[tri(5, 7)] = A[6];
      acc.A[tri(6, 6)] = A[7];
      acc.A[tri(6, 7)] = A[8];
    }
  }
}

}  // namespace shape
