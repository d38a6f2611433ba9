// Oscillator strengths and the Lorentzian eigen-sum of the macroscopic
// dielectric function (paper Sec. 4.4, eqs. chir and osci); the optical-limit
// transition coefficients and dielectric tensor (eqs. tlambdai, epsmij), the
// loss function and the dynamic structure factor (eq. Lofeps).
#include "bse_internal.h"
#include "common.h"
#include "timing.h"

namespace {

// osc[l] = |sum_a conj(XpY[a, l]) probe[a]|^2, one wavefront per column l.
__global__ __launch_bounds__(256) void k_oscillator(int64_t n, const double2* __restrict__ X,
                                                    int64_t ldx, const double2* __restrict__ p,
                                                    double* __restrict__ osc) {
  const int64_t l = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (l >= n) return;
  const double2* col = X + l * ldx;
  double2 acc = make_double2(0.0, 0.0);
  for (int64_t a = lane; a < n; a += 64) acc = cadd(acc, cmulc(col[a], p[a]));
  acc = wave_sum2(acc);
  if (lane == 0) osc[l] = cabs2(acc);
}

// The Lorentzian sums of F frequencies per lane,
//   S_ab(w) = sum_l conj(t_la) t_lb g_l(w),  g_l(w) = 1/(w - E_l + i eta) - 1/(w + E_l + i eta)
// (ND = 0: osc[l] in place of conj(t) t).  With d = (w - E + i eta) (w + E + i eta)
// = m + 2 i eta w, m = (w - E)(w + E) - eta^2, both fractions are one:
//   g = 2 E conj(d) / |d|^2,
// one reciprocal, and since conj(t_a) t_b is Hermitian its ND^2 real numbers are
// taken once per l and multiply the two real numbers of g.
// Where |d|^2 is not well inside the range of double precision (or not a number) the
// wavefront takes both fractions as they stand.
//
// Bound by the vector ALU: about 13 + 2 ND^2 instructions per (w, l).  A wavefront
// holds LZ_GROUPS F frequencies, 16 lanes sharing the l of each (one pass over E and t
// for all of them, sums over 16 lanes at the end); the LZ_WAVES wavefronts of a block
// split l.  N = 6144, 4000 w: 30 us for the spectrum, 53 us for the
// 3 x 3 tensor (45 and 104 us with two divisions per term, a wavefront per w and all
// nine complex products).
constexpr int LZ_WAVES = 8, LZ_GROUPS = 4;

BSE_DEV double2 lorentz_pair(double w, double e, double eta, double eta2) {
  const double x1 = w - e, x2 = w + e;
  const double i1 = 1.0 / (x1 * x1 + eta2), i2 = 1.0 / (x2 * x2 + eta2);
  // 1/(x + i eta) = (x - i eta) / (x^2 + eta^2)
  return make_double2(x1 * i1 - x2 * i2, -eta * i1 + eta * i2);
}

// The real numbers of level l: osc[l], or Re and Im of conj(t_a) t_b for a <= b.
template <int ND>
BSE_DEV void level_weights(const double* __restrict__ osc, const double2* __restrict__ t,
                           int64_t ldt, int64_t l, double (&W)[ND ? ND * ND : 1]) {
  if constexpr (ND == 0) {
    W[0] = osc[l];
  } else {
    double2 tv[ND];
#pragma unroll
    for (int a = 0; a < ND; ++a) tv[a] = t[l + a * ldt];
    int q = 0;
#pragma unroll
    for (int a = 0; a < ND; ++a) {
      W[q++] = cabs2(tv[a]);
#pragma unroll
      for (int b = a + 1; b < ND; ++b) {
        const double2 v = cmulc(tv[a], tv[b]);
        W[q++] = v.x;
        W[q++] = v.y;
      }
    }
  }
}

// emit(j, f, R, I) by one thread per frequency: R[q], I[q] = sum_l W_q Re g, Im g.
template <int ND, int F, class Emit>
BSE_DEV void lorentz_sums(int64_t n, const double* __restrict__ E, const double* __restrict__ osc,
                          const double2* __restrict__ t, int64_t ldt, double eta, int64_t nw,
                          const double* __restrict__ omega, Emit emit) {
  constexpr int NT = ND ? ND * ND : 1;
  constexpr int NV = 2 * NT;                 // sums of a frequency
  constexpr int NF = LZ_GROUPS * F;          // frequencies of a block
  __shared__ double part[LZ_WAVES][NF][NV];
  const int tid = threadIdx.x, wid = tid >> 6, lane = tid & 63;
  const int li = lane & 15, gi = lane >> 4;
  const int64_t j0 = (int64_t)blockIdx.x * NF;
  const double eta2 = eta * eta;
  double w[F], acc[F][NV];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    w[f] = omega[min(j0 + gi * F + f, nw - 1)];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[f][q] = 0.0;
  }
  for (int64_t l = wid * 16 + li; l < n; l += 16 * LZ_WAVES) {
    const double e = E[l];
    double W[NT];
    level_weights<ND>(osc, t, ldt, l, W);
    double2 g[F];
    bool ok = true;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const double c = 2.0 * eta * w[f];
      const double m = fma(w[f] - e, w[f] + e, -eta2), d = fma(m, m, c * c);
      // 2^-950 <= d < 2^950
      ok &= (unsigned)__double2hiint(d) - (73u << 20) < (1900u << 20);
      const double r = 2.0 * e * fast_rcp(d);
      g[f] = make_double2(m * r, -c * r);
    }
    if (!__all(ok)) {
#pragma unroll
      for (int f = 0; f < F; ++f) g[f] = lorentz_pair(w[f], e, eta, eta2);
    }
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        acc[f][2 * q] = fma(W[q], g[f].x, acc[f][2 * q]);
        acc[f][2 * q + 1] = fma(W[q], g[f].y, acc[f][2 * q + 1]);
      }
  }
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const double v = row_sum(acc[f][q]);
      if (li == 0) part[wid][gi * F + f][q] = v;
    }
  __syncthreads();
  double* sums = &part[0][0][0];  // the first wavefront's part becomes the whole
  for (int e = tid; e < NF * NV; e += 64 * LZ_WAVES) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < LZ_WAVES; ++k) v += sums[k * NF * NV + e];
    sums[e] = v;
  }
  __syncthreads();
  if (tid < NF && j0 + tid < nw) emit(j0 + tid, part[0][tid]);
}

// eps[j] = 1 - pref sum_l osc[l] g_l(w_j)
template <int F>
__global__ __launch_bounds__(64 * LZ_WAVES) void k_spectrum(int64_t n, const double* __restrict__ E,
                                                  const double* __restrict__ osc, double pref,
                                                  double eta, int64_t nw,
                                                  const double* __restrict__ omega,
                                                  double2* __restrict__ eps) {
  lorentz_sums<0, F>(n, E, osc, nullptr, 0, eta, nw, omega, [&](int64_t j, const double* S) {
    eps[j] = make_double2(1.0 - pref * S[0], -pref * S[1]);
  });
}


// t[l + i ldt] = -i sum_a conj(X[a, l]) p[a + i ldp] for TC consecutive
// columns l per block.  Thread tid takes rows tid, tid + 256, ...: per row it
// loads the NP probe values once and the row's element of each of the TC
// columns (256 consecutive elements of a column per block and step, so every
// column is read once, coalesced).  Sums: per wavefront, then the four
// wavefronts' partials in order (deterministic).
constexpr int TR_THREADS = 256, TR_COLS = 8;
template <int NP>
__global__ __launch_bounds__(TR_THREADS) void k_transitions(int64_t n,
                                                         const double2* __restrict__ X,
                                                         int64_t ldx,
                                                         const double2* __restrict__ p,
                                                         int64_t ldp, double2* __restrict__ t,
                                                         int64_t ldt) {
  __shared__ double2 part[TR_THREADS / 64][TR_COLS * NP];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t l0 = (int64_t)blockIdx.x * TR_COLS;
  const int ncol = (int)std::min<int64_t>(TR_COLS, n - l0);
  double2 acc[TR_COLS][NP];
#pragma unroll
  for (int c = 0; c < TR_COLS; ++c)
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[c][i] = make_double2(0.0, 0.0);
  for (int64_t a = tid; a < n; a += TR_THREADS) {
    double2 pv[NP], xv[TR_COLS];
#pragma unroll
    for (int i = 0; i < NP; ++i) pv[i] = p[a + i * ldp];
#pragma unroll
    for (int c = 0; c < TR_COLS; ++c)
      xv[c] = X[a + (l0 + std::min(c, ncol - 1)) * ldx];  // clamped column, masked below
#pragma unroll
    for (int c = 0; c < TR_COLS; ++c)
#pragma unroll
      for (int i = 0; i < NP; ++i) acc[c][i] = cadd(acc[c][i], cmulc(xv[c], pv[i]));
  }
#pragma unroll
  for (int c = 0; c < TR_COLS; ++c)
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const double2 v = wave_sum2(acc[c][i]);
      if (lane == 0) part[wid][c * NP + i] = v;
    }
  __syncthreads();
  if (tid < ncol * NP) {
    const int c = tid / NP, i = tid % NP;
    double2 v = part[0][tid];
#pragma unroll
    for (int w = 1; w < TR_THREADS / 64; ++w) v = cadd(v, part[w][tid]);
    t[(l0 + c) + i * ldt] = make_double2(v.y, -v.x);  // times -i
  }
}

// eps[(j ND + a) ND + b] = delta_ab - pref sum_l conj(t_la) t_lb g_l(w_j); CODE = 8 ND + F
template <int CODE>
__global__ __launch_bounds__(64 * LZ_WAVES) void k_dielectric_tensor(
    int64_t n, const double* __restrict__ E, const double2* __restrict__ t, int64_t ldt,
    double pref, double eta, int64_t nw, const double* __restrict__ omega,
    double2* __restrict__ eps) {
  constexpr int ND = CODE / 8, F = CODE % 8;
  lorentz_sums<ND, F>(n, E, nullptr, t, ldt, eta, nw, omega, [&](int64_t j, const double* S) {
    int q = 0;
#pragma unroll
    for (int a = 0; a < ND; ++a) {
      eps[(j * ND + a) * ND + a] = make_double2(1.0 - pref * S[2 * q], -pref * S[2 * q + 1]);
      ++q;
#pragma unroll
      for (int b = a + 1; b < ND; ++b) {
        // (x + i y) g and, below the diagonal, (x - i y) g
        const double xr = S[2 * q], xi = S[2 * q + 1], yr = S[2 * q + 2], yi = S[2 * q + 3];
        eps[(j * ND + a) * ND + b] = make_double2(-pref * (xr - yi), -pref * (xi + yr));
        eps[(j * ND + b) * ND + a] = make_double2(-pref * (xr + yi), -pref * (xi - yr));
        q += 2;
      }
    }
  });
}

// loss[j] = -Im 1/eps[j inc] = Im eps / |eps|^2; sqw[j] = loss[j] vinv / pi.
__global__ __launch_bounds__(256) void k_loss(int64_t nw, const double2* __restrict__ eps,
                                              int64_t inc, double vinv,
                                              double* __restrict__ loss,
                                              double* __restrict__ sqw) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= nw) return;
  const double2 e = eps[j * inc];
  const double L = e.y / cabs2(e);
  loss[j] = L;
  if (sqw) sqw[j] = L * vinv * (1.0 / M_PI);
}

}  // namespace

hipError_t launch_oscillator(int64_t n, const double2* XpY, int64_t ldx, const double2* probe,
                             double* osc, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  BSE_LAUNCH(k_oscillator, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, n, XpY, ldx,
                     probe, osc);
  return hipGetLastError();
}

// Frequencies per lane: as many as leave a block for three in four of 256 compute
// units.  The order of the sums is the same for all.
static int lorentz_f(int64_t nw) {
  for (int f : {4, 2})
    if (nw >= 192 * LZ_GROUPS * f) return f;
  return 1;
}

hipError_t launch_spectrum(int64_t n, const double* E, const double* osc, double pref, double eta,
                           int64_t nw, const double* omega, double2* eps, hipStream_t s) {
  if (nw <= 0) return hipSuccess;
  const int f = lorentz_f(nw);
  const dim3 grid((unsigned)cdiv(nw, LZ_GROUPS * f)), block(64 * LZ_WAVES);
  switch (f) {
    case 1: BSE_LAUNCH(k_spectrum<1>, grid, block, 0, s, n, E, osc, pref, eta, nw, omega, eps); break;
    case 2: BSE_LAUNCH(k_spectrum<2>, grid, block, 0, s, n, E, osc, pref, eta, nw, omega, eps); break;
    default: BSE_LAUNCH(k_spectrum<4>, grid, block, 0, s, n, E, osc, pref, eta, nw, omega, eps);
  }
  return hipGetLastError();
}

hipError_t launch_transitions(int64_t n, const double2* XpY, int64_t ldx, int nprobe,
                              const double2* probe, int64_t ldp, double2* t, int64_t ldt,
                              hipStream_t s) {
  const dim3 grid((unsigned)cdiv(n, TR_COLS)), block(TR_THREADS);
  switch (nprobe) {
    case 1: BSE_LAUNCH(k_transitions<1>, grid, block, 0, s, n, XpY, ldx, probe, ldp, t, ldt); break;
    case 2: BSE_LAUNCH(k_transitions<2>, grid, block, 0, s, n, XpY, ldx, probe, ldp, t, ldt); break;
    case 3: BSE_LAUNCH(k_transitions<3>, grid, block, 0, s, n, XpY, ldx, probe, ldp, t, ldt); break;
    case 4: BSE_LAUNCH(k_transitions<4>, grid, block, 0, s, n, XpY, ldx, probe, ldp, t, ldt); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_dielectric_tensor(int64_t n, const double* E, int nd, const double2* t,
                                    int64_t ldt, double pref, double eta, int64_t nw,
                                    const double* omega, double2* eps, hipStream_t s) {
  const int f = lorentz_f(nw);
  const dim3 grid((unsigned)cdiv(nw, LZ_GROUPS * f)), block(64 * LZ_WAVES);
#define TENSOR_CASE(ND, F)                                                                        \
  case ND * 8 + F:                                                                                \
    BSE_LAUNCH(k_dielectric_tensor<ND * 8 + F>, grid, block, 0, s, n, E, t, ldt, pref, eta, nw, omega, \
               eps);                                                                              \
    break;
  switch (nd * 8 + f) {
    TENSOR_CASE(1, 1) TENSOR_CASE(1, 2) TENSOR_CASE(1, 4)
    TENSOR_CASE(2, 1) TENSOR_CASE(2, 2) TENSOR_CASE(2, 4)
    TENSOR_CASE(3, 1) TENSOR_CASE(3, 2) TENSOR_CASE(3, 4)
    default: return hipErrorInvalidValue;
  }
#undef TENSOR_CASE
  return hipGetLastError();
}

hipError_t launch_loss(int64_t nw, const double2* eps, int64_t inc, double vinv, double* loss,
                       double* sqw, hipStream_t s) {
  BSE_LAUNCH(k_loss, dim3((unsigned)cdiv(nw, 256)), dim3(256), 0, s, nw, eps, inc, vinv, loss,
             sqw);
  return hipGetLastError();
}
