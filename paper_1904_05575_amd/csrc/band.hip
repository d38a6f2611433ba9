// Reduction of a Hermitian matrix to real symmetric tridiagonal form in two
// stages, for the solves that form no eigenvectors (Sec. 4.3 with the probe of
// Sec. 4.4 carried along): dense to a band of half width BW by block
// reflectors, whose work is matrix products, then the band to tridiagonal form
// by chasing bulges down the band.  The one-stage sweep (hetrd.hip) reads the
// trailing triangle once per column; here it is read and written once per BW
// columns, in a kernel that works on the matrix cores.
// n = 6144 (one-stage sweep: 190 ms, 618 GB of triangle reads): k_band_step 31.7 ms (29
// TFLOP/s issued, in three real products per complex one: neither the matrix cores nor
// memory bound it), k_band_x 8.1, k_band_panel 6.8, k_band_chol 4.6, k_band_w 4.4,
// k_band_chase 22.6.  The panel kernels are chains: 10 to 19 us per launch at any order.
//
// The parts are published methods: QR by two Cholesky passes (Yamamoto, Nakatsukasa,
// Yanagisawa and Fukaya, ETNA 44, 2015), the reflector form rebuilt from Q (Ballard,
// Demmel, Grigori, Jacquelin, Nguyen and Solomonik, IPDPS 2014), the chase (Schwarz,
// Numer. Math. 12, 1968; Lang, SIAM J. Sci. Comput. 14, 1993).
//
// Stage 1, panel k (columns j0 = BW k .., trailing rows and columns t = j0 + BW ..):
//   k_band_chol   R1 from the Gram matrix of the panel P = S[t:, j0:j0+BW]
//                 (Cholesky), Q1 = P R1^-1, Gram partials of Q1
//   k_band_panel  R2 from the Gram matrix of Q1 (the second Cholesky pass makes
//                 Q = Q1 R2^-1 orthonormal to rounding), then the reflector whose
//                 first columns are Q's: with D a diagonal of modulus one that
//                 opposes the pivots of Q_top - D, V = Q - [D; 0], H = I - V T V^H,
//                 T = -D^* (Q_top - D)^-H, and P = H [D R2 R1; 0]
//   k_band_step   the trailing triangle S -= V W^H + W V^H of the previous
//                 panel and, from the same registers, the partial products of
//                 X = S V with this panel's V
//   k_band_x      X from the partial products, partials of Z = V^H X, H^H on the probe
//   k_band_w      W = X T - 1/2 V T^H Z T, the next panel's columns updated,
//                 Gram partials of the next panel
// Panels whose Gram matrix is not safely positive definite (columns that are
// dependent, or fewer rows than the factorisation needs) take Householder's
// column-by-column factorisation in one block of k_band_panel, over the rows before
// the part that is zero in every column; panels that are zero take H = I.
//
// Stage 2: k_band_chase (below).
//
// All reductions have a fixed order and no kernel uses floating-point atomics:
// a repeated run gives the same bits, on its own or in a batch.
#include <algorithm>
#include <vector>

#include "bse_internal.h"
#include "common.h"
#include "mfma_tile.h"
#include "solve_internal.h"
#include "timing.h"

namespace {

constexpr int BW = BAND_W;
static_assert(BW == 16, "one 16 x 16 matrix-core tile per block of the band");
constexpr int DIRECT_ROWS = 64;   // panels with fewer rows are factored column by column
// Elements of E = Q1^H Q1 - I (real and imaginary parts) up to which the second pass of a
// panel takes its series: they bound ||E|| by 1.5 BW SERIES_MAX, and the series' errors, a
// few ||E||^4, have to stay below rounding for the panel to be orthonormal to rounding.
// (Well-conditioned panels have E near 1e-14; this limit is met from cond(P) ~ 1e5 on.)
constexpr double SERIES_MAX = 2e-6;
constexpr double fourth(double x) { return x * x * x * x; }
static_assert(8 * fourth(1.5 * BW * SERIES_MAX) < 1.1e-16, "the series is exact to rounding");
constexpr double COLUMN_ZERO = 1e-280;  // squared norm up to which a column takes H = I
constexpr double PIVOT_LEAST = 1e-11;   // of its diagonal: a panel's pivots on the Gram route
static_assert(COLUMN_ZERO * PIVOT_LEAST > 1e-300, "the pivots' reciprocals are finite");
constexpr int LDT = BW + 1;       // padded row of a 16 x 16 tile in LDS
constexpr int ABS = 2 * BW + 2;   // band storage per column: 2 BW diagonals, the probe, one spare
                                  // (in LDS a row of the band then steps by 2 BW + 1 values, over
                                  // all banks; by 2 BW, 16 lanes meet in one)

// Complex elements of the stored band, rounded to 256 bytes.
__host__ __device__ inline int64_t band_elems(int64_t n) { return (n * ABS + 15) & ~(int64_t)15; }

// Rows of a block of the panel kernels (one wavefront per 16 rows) for a trailing
// matrix of order m: 64 give each wavefront a SIMD of its own; beyond 4096 rows
// 128, since every block reads all blocks' 16 x 16 partial sums.
__host__ __device__ inline int panel_rows(int64_t m) { return m > 4096 ? 128 : 64; }
__host__ __device__ inline int panel_blocks(int64_t m) { return cdiv(m, panel_rows(m)); }

// Tile edge of k_band_step at trailing order m: below 512 a launch of 64 x 64 tiles
// leaves most compute units idle (n = 324: 17.8 us per launch, 11.6 with 32 x 32);
// above it the smaller tile gains in that kernel what its slots cost k_band_x (n =
// 2048, both kernels, small tiles up to 512, 768, 1024, 1408: 4.76, 4.76, 4.80, 4.94 ms).
constexpr int STEP_SMALL = 512;
__host__ __device__ inline int step_tile(int64_t m) { return m > STEP_SMALL ? 64 : 32; }
// Halves of a tile's rows: beyond STEP_TALL a block takes tiles of 128 rows x 64
// columns, whose halves add their column sums in LDS, so that half the slots are written
// and read (16 KB per tile of 64 KB, each way).  k_band_step itself does not gain (its two
// more barriers per tile), k_band_x does where the slots leave the caches.  Both kernels,
// tall tiles never, beyond 3072, 2048, 1024: n = 2048: 4.72, 4.82, 4.75, 4.98 ms; n = 4200:
// 17.5, 17.2, 17.1, 17.4 ms; n = 6144: 42.0, 40.0, 39.8, 40.2 ms (n = 10368: 176 -> 151).
constexpr int STEP_TALL = 2048;
__host__ __device__ inline int step_halves(int64_t m) { return m > STEP_TALL ? 2 : 1; }

__host__ __device__ inline int band_ctl_ints(int n) { return 2 + n / CHASE_SWEEPS + 1; }

struct BandProb {
  double2* M;
  int64_t ld;
  int n, ycs;
  double2* VW;   // n x 64 as four n x BW row-major arrays: V, W of even and of odd panels
  double2* Q1;   // n x BW row-major
  double2* X;    // n x BW row-major
  double2* Y;    // partial products of k_band_step: slots of n x BW
  double2* g1;   // Gram partials of the panel, BW x BW per block
  double2* g2;   // Gram partials of Q1
  double2* z;    // partials of V^H X
  double2* pd;   // partials of V^H y, BW per block
  double2* sm;   // T, L1 (BW x BW each)
  double2* yp;   // probe or null
  double2* AB;   // band, ABS values per column
  double *dd, *ee;
  int32_t* ctl;  // [0] panel state, [1] ticket of the chase, [2 ..] its groups' progress
  int32_t* info;
};
// They travel by value in the kernel arguments, so that the compiler knows every
// pointer to be device memory (and loads through it do not count as LDS loads).
struct BandArgs {
  BandProb p[BAND_BATCH_MAX];
};
// A launch's blocks, problem after problem: problem p owns blocks [b[p], b[p+1]);
// a problem with nothing to do at a step owns none.
struct BandFirst {
  int32_t b[BAND_BATCH_MAX + 1];
};

// The problem that owns this block (a uniform scan of the block ranges in the
// kernel arguments).
BSE_DEV int band_problem(const BandFirst& f) {
  int p = 0;
  while (p + 1 < BAND_BATCH_MAX && (int)blockIdx.x >= f.b[p + 1]) ++p;
  return p;
}

BSE_DEV double2* v_of(const BandProb& p, int k) {
  return p.VW + (int64_t)(k & 1) * 2 * BW * p.n;
}
BSE_DEV double2* w_of(const BandProb& p, int k) {
  return p.VW + ((int64_t)(k & 1) * 2 + 1) * BW * p.n;
}

BSE_DEV double2 czero() { return make_double2(0.0, 0.0); }
BSE_DEV double2 keep2(bool ok, double2 v) { return make_double2(ok ? v.x : 0.0, ok ? v.y : 0.0); }

// Sum over the four rows (lanes l, l ^ 16, l ^ 32, l ^ 48); every lane gets it.
BSE_DEV double quad_rows_sum(double v) {
  const long long b = __double_as_longlong(v);
  const auto l0 = __builtin_amdgcn_permlane16_swap((int)b, (int)b, false, false);
  const auto h0 = __builtin_amdgcn_permlane16_swap((int)(b >> 32), (int)(b >> 32), false, false);
  v = __longlong_as_double(((long long)h0[0] << 32) | (unsigned int)l0[0]) +
      __longlong_as_double(((long long)h0[1] << 32) | (unsigned int)l0[1]);
  const long long c = __double_as_longlong(v);
  const auto l1 = __builtin_amdgcn_permlane32_swap((int)c, (int)c, false, false);
  const auto h1 = __builtin_amdgcn_permlane32_swap((int)(c >> 32), (int)(c >> 32), false, false);
  return __longlong_as_double(((long long)h1[0] << 32) | (unsigned int)l1[0]) +
         __longlong_as_double(((long long)h1[1] << 32) | (unsigned int)l1[1]);
}
BSE_DEV double2 quad_rows_sum(double2 v) {
  return make_double2(quad_rows_sum(v.x), quad_rows_sum(v.y));
}
BSE_DEV double lane_value(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum of `nb` blocks' 16 x 16 partials into out (256 values, LDS); tmp: 256
// values.  NW = 8: two threads per value (even and odd blocks); the order is fixed.
template <int NW>
BSE_DEV void sum_partials(const double2* __restrict__ part, int nb, double2* out, double2* tmp) {
  constexpr int ST2 = NW / 4;
  const int e = threadIdx.x & 255, h = threadIdx.x >> 8;
  double2 s = czero();
  int b = h;
  for (; b + 15 * ST2 < nb; b += 16 * ST2) {
    double2 v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = part[(int64_t)(b + ST2 * u) * 256 + e];
#pragma unroll
    for (int u = 0; u < 16; ++u) s = cadd(s, v[u]);
  }
  if (b < nb) {  // the rest, together (clamped, masked)
    double2 v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = part[(int64_t)min(b + ST2 * u, nb - 1) * 256 + e];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (b + ST2 * u < nb) s = cadd(s, v[u]);
  }
  if (NW == 8) {
    if (h) tmp[e] = s;
    __syncthreads();
  }
  if (!h) out[e] = NW == 8 ? cadd(s, tmp[e]) : s;
  __syncthreads();
}

// Block-wide sum of the wavefronts' 16 x 16 results into part[0..255].
template <int NW>
BSE_DEV void reduce_tiles(const Acc& a, double2* red, double2* __restrict__ part) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    red[wid * 256 + ((lane >> 4) + 4 * r) * BW + (lane & 15)] = a.at(r);
  __syncthreads();
  if (threadIdx.x < 256) {
    double2 s = czero();
#pragma unroll
    for (int w = 0; w < NW; ++w) s = cadd(s, red[w * 256 + threadIdx.x]);
    part[threadIdx.x] = s;
  }
}

struct StepShare {  // values of the current elimination step, two steps' buffers
  double2 row[2][2][BW];  // pivot row of the matrix and of the augmented identity
  double2 col[2][BW];     // pivot column
};

// Cholesky factor and its inverse of the 16 x 16 Hermitian matrix in G (LDS,
// row-major), by the block's first 256 threads, each with one element of the
// matrix and one of the identity beside it; one barrier per column.  L and Li:
// LDS, rows of LDT.  Returns false (uniformly) when a pivot is not above tol
// times its diagonal (tol times each diagonal has to be a normal number).
BSE_DEV bool chol_inv(const double2* G, double2* L, double2* Li, double* dg, StepShare& sh,
                      double tol) {
  const int e = threadIdx.x & 255, i = e >> 4, j = e & 15;
  const bool on = threadIdx.x < 256;
  double2 v = G[e], y = make_double2(i == j ? 1.0 : 0.0, 0.0);
  bool ok = true;
  if (on) {
    if (i == 0) {
      sh.row[0][0][j] = v;
      sh.row[0][1][j] = y;
    }
    if (j == 0) sh.col[0][i] = v;
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < BW; ++s) {
    const int cur = s & 1, nxt = cur ^ 1;
    const double p = sh.col[cur][s].x;
    const double2 ci = sh.col[cur][i];
    ok = ok && p > tol * G[s * BW + s].x;
    if (on && i > s) {
      const double2 l = cneg(cscale(ci, fast_rcp(p)));
      if (j > s) v = cfma(l, sh.row[cur][0][j], v);
      y = cfma(l, sh.row[cur][1][j], y);
    }
    if (s + 1 < BW) {
      if (on) {
        if (i == s + 1) {
          sh.row[nxt][0][j] = v;
          sh.row[nxt][1][j] = y;
        }
        if (j == s + 1) sh.col[nxt][i] = v;
      }
      __syncthreads();
    }
  }
  if (on && i == j) dg[i] = fast_rsq(v.x);
  __syncthreads();
  if (on) {
    // the diagonal real, as the pivots were taken: what is left of its imaginary part is
    // rounding of G, but relative to a small pivot it would make Li L differ from 1
    double2 l = cscale(v, dg[j]);
    if (i == j) l.y = 0.0;
    L[i * LDT + j] = i >= j ? l : czero();
    Li[i * LDT + j] = i >= j ? cscale(y, dg[i]) : czero();
  }
  __syncthreads();
  return ok;
}

// ------------------------------------------------------- panel, first pass
// Q1 = P R1^-1 with R1 from the Gram matrix.  Panel state: 0 ok, 1 the Gram
// matrix is not safely positive definite, 2 the panel is zero.
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_band_chol(BandArgs a, BandFirst f, int k) {
  constexpr int RB = 16 * NW;
  const int pi = band_problem(f);
  const BandProb& p = a.p[pi];
  if (failed(p.info)) return;
  const int bx = (int)blockIdx.x - f.b[pi];
  const int j0 = BW * k, t = j0 + BW, n = p.n;
  __shared__ double2 red[NW * 256];
  __shared__ double2 G[256], tmp[256], L[BW * LDT], Li[BW * LDT];
  __shared__ double dg[BW];
  __shared__ StepShare sh;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, lo = lane & 15, hi = lane >> 4;

  const int row = t + bx * RB + wid * 16 + lo;  // this lane's row of P^T
  double2 pt[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    pt[c] = p.M[min(row, n - 1) + (int64_t)(j0 + hi + 4 * c) * p.ld];
  // the partials come from k_band_w over rows j0 .. (t = 0: the first panel)
  sum_partials<NW>(p.g1, panel_blocks(n - j0), G, tmp);
  // every column zero, as a reflector takes it: nothing to reflect; some: not by the Gram
  // route, where the reciprocals of their pivots could overflow
  double least = G[0].x, most = G[0].x;
#pragma unroll
  for (int s = 1; s < BW; ++s) {
    least = fmin(least, G[s * BW + s].x);
    most = fmax(most, G[s * BW + s].x);
  }
  const bool zero = most <= COLUMN_ZERO, small = least <= COLUMN_ZERO;
  if (zero) {
    if (bx == 0 && tid == 0) p.ctl[0] = 2;
    return;
  }
  // a pivot of PIVOT_LEAST of its diagonal leaves the first pass orthonormal to about
  // 1e-5, which the second pass squares away (orthonormality alone: the panel's own
  // residual is Q1's to keep, below)
  const bool ok = !small && chol_inv(G, L, Li, dg, sh, PIVOT_LEAST);
  if (bx == 0 && tid == 0) p.ctl[0] = ok ? 0 : 1;
  if (!ok) return;
  if (bx == 0 && tid < 256) p.sm[256 + tid] = L[(tid >> 4) * LDT + (tid & 15)];

  // Q1^T = conj(L)^-1 P^T by the explicit inverse, then once more for what it left: the
  // inverse alone leaves P - Q1 R1 of the order u cond(P) ||P||, which no second pass
  // sees and which is lost when the panel becomes [R; 0]; the correction leaves u ||P||
  // (eigenvalue errors of 2e-13 to 3e-10 ||A|| on panels of condition 10^5.5 to 10^8 without
  // it and with a complex diagonal in L, below 6e-15 with both; solve at n = 2000: 17.46 ->
  // 17.55 ms)
  Acc q;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    pt[c] = keep2(row < n, pt[c]);
    q.mac(cconj(Li[lo * LDT + hi + 4 * c]), pt[c]);
  }
  double2 qv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) qv[r] = q.at(r);
  Acc back, fix;
#pragma unroll
  for (int c = 0; c < 4; ++c) back.mac(cconj(L[lo * LDT + hi + 4 * c]), qv[c]);
#pragma unroll
  for (int c = 0; c < 4; ++c)
    fix.mac(cconj(Li[lo * LDT + hi + 4 * c]), csub(pt[c], back.at(c)));
  double2* tr = red + wid * 256;  // the wavefront's tile, transposed through LDS
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    qv[r] = cadd(qv[r], fix.at(r));
    if (row < n) p.Q1[(int64_t)row * BW + hi + 4 * r] = qv[r];
    tr[lo * BW + ((hi + 4 * r) ^ lo)] = qv[r];  // [row][vec], swizzled
  }
  wave_lds_sync();
  Acc g;
  double2 x[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int rr = hi + 4 * c;
    x[c] = tr[rr * BW + (lo ^ rr)];
  }
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < 4; ++c) g.mac(cconj(x[c]), x[c]);
  reduce_tiles<NW>(g, red, p.g2 + (int64_t)bx * 256);
}

// ------------------------------------------------ column-by-column panel
// Panels whose rows past the first m <= 64 are zero, in registers of the block's first 256 threads:
// thread (c, l) holds rows l + 16 q of column c, so a sum over rows is one over
// the 16 lanes of a DPP row; one barrier per column.  xcol: 2 x 64 values, gv: 2 x
// BW, Tl: BW x LDT (LDS).  Columns already reduced hold their reflector, whose
// product with the new one gives T's next column.
BSE_DEV void panel_small(const BandProb& p, int k, int m, double2* xcol, double2* gv,
                         double2* Tl) {
  const int j0 = BW * k, t = j0 + BW, n = p.n;
  const int tid = threadIdx.x, l = tid & 15, c = tid >> 4;
  const bool on = tid < 256;
  double2* V = v_of(p, k);
  double2 a[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = l + 16 * q;
    a[q] = keep2(on && r < m, p.M[min(t + r, n - 1) + (int64_t)(j0 + (c & 15)) * p.ld]);
  }
  if (on) Tl[c * LDT + l] = czero();
  const int jn = min(BW, m);
  double2 tprev = czero();
  for (int j = 0; j <= jn; ++j) {
    double2* xc = xcol + (j & 1) * 64;
    if (on && c == j && j < jn) {
#pragma unroll
      for (int q = 0; q < 4; ++q) xc[l + 16 * q] = a[q];
    }
    __syncthreads();
    if (on && j > 0) {  // T[:i, i] = -tau_i T[:i, :i] (V^H v_i), i = j - 1
      const int i = j - 1;
      if (tid < i) {
        double2 v = czero();
        for (int q = tid; q < i; ++q) v = cfma(Tl[tid * LDT + q], gv[(i & 1) * BW + q], v);
        Tl[tid * LDT + i] = cneg(cmul(tprev, v));
      } else if (tid == i) {
        Tl[i * LDT + i] = tprev;
      }
    }
    if (j == jn) break;
    double2 u[4];
    double xn = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u[q] = xc[l + 16 * q];
      if (l + 16 * q > j) xn += cabs2(u[q]);
    }
    const double2 al = xc[j];
    xn = row_sum(xn);
    const double nn = cabs2(al) + xn;
    double2 tau = czero(), scal = czero(), beta = al;
    if (xn != 0.0 && nn > COLUMN_ZERO) {
      const double b = -copysign(sqrt(nn), al.x);
      beta = make_double2(b, 0.0);
      tau = make_double2((b - al.x) / b, -al.y / b);
      const double2 dn = make_double2(al.x - b, al.y);
      const double q = 1.0 / cabs2(dn);
      scal = make_double2(dn.x * q, -dn.y * q);
    }
    double2 g = czero();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = l + 16 * q;
      u[q] = r > j ? cmul(scal, u[q]) : make_double2(r == j ? 1.0 : 0.0, 0.0);
      g = cfmac(u[q], a[q], g);
    }
    g = row_sum(g);
    if (on && c > j) {
      g = cneg(cmulc(tau, g));
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = cfma(u[q], g, a[q]);
    } else if (on && c < j) {
      if (l == 0) gv[(j & 1) * BW + c] = cconj(g);
    } else if (on) {  // column j: R above and on the diagonal, then its reflector
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = l + 16 * q;
        if (r <= j) p.M[t + r + (int64_t)(j0 + j) * p.ld] = r == j ? beta : a[q];
        a[q] = u[q];
      }
    }
    tprev = tau;
  }
  // columns past the last reflector (fewer rows than columns) hold R
  if (on && c >= jn) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = l + 16 * q;
      if (r < m) p.M[t + r + (int64_t)(j0 + c) * p.ld] = a[q];
      a[q] = czero();
    }
  }
  double2 d = czero();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = l + 16 * q;
    if (on && r < m) {
      V[(int64_t)(t + r) * BW + c] = a[q];
      if (p.yp) d = cfmac(a[q], p.yp[t + r], d);
    }
  }
  d = row_sum(d);
  if (on && l == 0) p.pd[c] = d;
  __syncthreads();
  if (on) p.sm[tid] = Tl[c * LDT + l];
}

// Householder factorisation of P = S[t:t+m, j0:j0+BW], the rows past m zero, by one
// block, in place (row i <= column j of the result is R); the first m rows of V, and T,
// as the fast path leaves them.
// sums: NW * BW values, sv: BW values (LDS); Tl: BW * LDT (LDS).
template <int NW>
BSE_DEV void panel_direct(const BandProb& p, int k, int m, double2* sums, double2* sv,
                          double2* Tl) {
  constexpr int NT = 64 * NW;
  const int j0 = BW * k, t = j0 + BW;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  double2* V = v_of(p, k);
  double2* P = p.M + t + (int64_t)j0 * p.ld;
  auto col = [&](int r, int c) -> double2& { return P[r + (int64_t)c * p.ld]; };
  // sums over the block of up to BW values per thread, into sv
  auto block_sums = [&](const double2(&s)[BW]) {
#pragma unroll
    for (int c = 0; c < BW; ++c) {
      const double2 v = wave_sum2(s[c]);
      if (lane == 0) sums[wid * BW + c] = v;
    }
    __syncthreads();
    if (tid < BW) {
      double2 v = czero();
      for (int w = 0; w < NW; ++w) v = cadd(v, sums[w * BW + tid]);
      sv[tid] = v;
    }
    __syncthreads();
  };
  for (int e = tid; e < BW * LDT; e += NT) Tl[e] = czero();
  for (int64_t e = tid; e < (int64_t)m * BW; e += NT) V[(int64_t)t * BW + e] = czero();
  __syncthreads();
  const int jn = min(BW, m);
  for (int j = 0; j < jn; ++j) {
    double2 s[BW];
#pragma unroll
    for (int c = 0; c < BW; ++c) s[c] = czero();
    for (int r = j + 1 + tid; r < m; r += NT) {
      const double2 x = col(r, j);
#pragma unroll
      for (int c = 0; c < BW; ++c)
        if (c >= j) s[c] = cadd(s[c], cmulc(x, col(r, c)));
    }
    block_sums(s);
    const double2 al = col(j, j);
    const double xn2 = sv[j].x, nn = cabs2(al) + xn2;
    double2 tau = czero(), scal = czero(), beta = al;
    if (xn2 != 0.0 && nn > COLUMN_ZERO) {
      const double b = -copysign(sqrt(nn), al.x);
      beta = make_double2(b, 0.0);
      tau = make_double2((b - al.x) / b, -al.y / b);
      const double2 dn = make_double2(al.x - b, al.y);
      const double q = 1.0 / cabs2(dn);
      scal = make_double2(dn.x * q, -dn.y * q);
    }
    // v^H A_c = A[j][c] + conj(scal) s_c
    double2 gc[BW];
#pragma unroll
    for (int c = 0; c < BW; ++c)
      gc[c] = c > j ? cmulc(tau, cadd(col(j, c), cmulc(scal, sv[c]))) : czero();
    __syncthreads();  // every thread has read row j
    for (int r = j + tid; r < m; r += NT) {
      const double2 v = r == j ? make_double2(1.0, 0.0) : cmul(scal, col(r, j));
      V[(int64_t)(t + r) * BW + j] = v;
#pragma unroll
      for (int c = 0; c < BW; ++c)
        if (c > j) col(r, c) = csub(col(r, c), cmul(v, gc[c]));
      if (r == j) col(j, j) = beta;
    }
    if (tid == 0) Tl[j * LDT + j] = tau;
    __syncthreads();
  }
  // T[:i, i] = -tau_i T[:i, :i] (V^H v_i)
  for (int i = 1; i < jn; ++i) {
    double2 s[BW];
#pragma unroll
    for (int c = 0; c < BW; ++c) s[c] = czero();
    for (int r = i + tid; r < m; r += NT) {
      const double2 x = V[(int64_t)(t + r) * BW + i];
#pragma unroll
      for (int c = 0; c < BW; ++c)
        if (c < i) s[c] = cadd(s[c], cmulc(V[(int64_t)(t + r) * BW + c], x));
    }
    block_sums(s);
    double2 v = czero();
    if (tid < i) {
      for (int c = tid; c < i; ++c) v = cadd(v, cmul(Tl[tid * LDT + c], sv[c]));
      v = cmul(Tl[i * LDT + i], v);
    }
    __syncthreads();
    if (tid < i) Tl[tid * LDT + i] = make_double2(-v.x, -v.y);
    __syncthreads();
  }
  if (tid < 256) p.sm[tid] = Tl[(tid >> 4) * LDT + (tid & 15)];
  if (p.yp) {  // V^H y, into the first block's partial
    double2 s[BW];
#pragma unroll
    for (int c = 0; c < BW; ++c) s[c] = czero();
    for (int r = tid; r < m; r += NT) {
      const double2 y = p.yp[t + r];
#pragma unroll
      for (int c = 0; c < BW; ++c) s[c] = cadd(s[c], cmulc(V[(int64_t)(t + r) * BW + c], y));
    }
    block_sums(s);
    if (tid < BW) p.pd[tid] = sv[tid];
  }
}

// Rows of the panel before the part that is zero in all its columns, from the Gram
// partials of its row blocks (k_band_w's, over rows j0 ..): matrices that fall into blocks
// or bands have few, wherever their columns are dependent.
BSE_DEV int panel_extent(const BandProb& p, int j0, int* last) {
  const int mw = p.n - j0;
  if (threadIdx.x == 0) *last = 0;
  __syncthreads();
  for (int b = threadIdx.x; b < panel_blocks(mw); b += blockDim.x) {
    bool some = false;
    for (int s = 0; s < BW; ++s) some = some || p.g1[(int64_t)b * 256 + 17 * s].x != 0.0;
    if (some) atomicMax(last, b);
  }
  __syncthreads();
  return min((*last + 1) * panel_rows(mw), mw) - BW;
}

// ------------------------------------------------------ panel, second pass
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_band_panel(BandArgs a, BandFirst f, int k) {
  constexpr int RB = 16 * NW;
  const int pi = band_problem(f);
  const BandProb& p = a.p[pi];
  if (failed(p.info)) return;
  const int bx = (int)blockIdx.x - f.b[pi];
  const int j0 = BW * k, t = j0 + BW, n = p.n, m = n - t;
  __shared__ double2 red[NW * 256];
  __shared__ double2 G[256], tmp[256], L[BW * LDT], Li[BW * LDT];
  __shared__ double2 Dv[BW];
  __shared__ double dg[BW];
  __shared__ StepShare sh;
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, lo = lane & 15, hi = lane >> 4;
  double2* V = v_of(p, k);
  if (m < DIRECT_ROWS) {  // uniform; one block
    panel_small(p, k, m, red, G, L);
    return;
  }
  const int row = t + bx * RB + wid * 16 + lo;
  const int e = tid & 255, i = e >> 4, j = e & 15;
  const bool on = tid < 256;
  int state = p.ctl[0];  // uniform
  double2 qf[4];
  if (state == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) qf[c] = p.Q1[(int64_t)min(row, n - 1) * BW + hi + 4 * c];
    const double2 qt = p.Q1[(int64_t)(t + i) * BW + j];
    sum_partials<NW>(p.g2, panel_blocks(m), G, tmp);
    // R2 (in L) and its inverse (in Li), upper triangular, R2^H R2 = G = I + E.  For
    // a small E from the fixed point X = upper(E - X^H X) (diagonal halved) of R2
    // = I + X, whose error goes from ||E||^2 to ||E||^3 and ||E||^4, and 1 - X + X^2 -
    // X^3: four products in place of sixteen dependent steps
    const double2 E = csub(G[e], make_double2(i == j ? 1.0 : 0.0, 0.0));
    const bool tiny = __syncthreads_and(fabs(E.x) < SERIES_MAX && fabs(E.y) < SERIES_MAX);
    if (tiny) {
      const double half = i < j ? 1.0 : i == j ? 0.5 : 0.0;
      double2 x = cscale(E, half);
      for (int it = 0; it < 2; ++it) {
        if (on) Li[i * LDT + j] = x;
        __syncthreads();
        double2 r = E;
#pragma unroll
        for (int q = 0; q < BW; ++q) r = cfmac(cneg(Li[q * LDT + i]), Li[q * LDT + j], r);
        x = cscale(r, half);
        __syncthreads();
      }
      const double2 one = make_double2(i == j ? 1.0 : 0.0, 0.0);
      double2 y = csub(one, x);
      if (on) L[i * LDT + j] = cneg(x);
      for (int it = 0; it < 2; ++it) {
        if (on) Li[i * LDT + j] = y;
        __syncthreads();
        y = one;
#pragma unroll
        for (int q = 0; q < BW; ++q) y = cfma(L[i * LDT + q], Li[q * LDT + j], y);
        __syncthreads();
      }
      if (on) {
        L[i * LDT + j] = cadd(one, x);
        Li[i * LDT + j] = y;
      }
    } else if (chol_inv(G, L, Li, dg, sh, 0.5)) {  // lower factors, transposed
      const double2 l = cconj(L[j * LDT + i]), li = cconj(Li[j * LDT + i]);
      __syncthreads();
      if (on) {
        L[i * LDT + j] = l;
        Li[i * LDT + j] = li;
      }
    } else {
      state = 1;
    }
    if (on) tmp[e] = qt;
    __syncthreads();
  }
  double2 y = make_double2(i == j ? 1.0 : 0.0, 0.0);
  if (state == 0) {
    // ---- (Q_top - D)^-1, Q_top = Q1[:16] R2^-1, by Gauss-Jordan elimination beside
    // the identity (one element of each per thread, one barrier per column); D_s
    // opposes the pivot's phase, so that no pivot is below 1
    double2 v = czero();
#pragma unroll
    for (int q = 0; q < BW; ++q) v = cfma(tmp[i * BW + q], Li[q * LDT + j], v);
    if (on) {
      if (i == 0) {
        sh.row[0][0][j] = v;
        sh.row[0][1][j] = y;
      }
      if (j == 0) sh.col[0][i] = v;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < BW; ++s) {
      const int cur = s & 1, nxt = cur ^ 1;
      const double2 pv = sh.col[cur][s], ci = sh.col[cur][i];
      const double2 rv = sh.row[cur][0][j], ry = sh.row[cur][1][j];
      const double a2 = cabs2(pv);
      double2 D = make_double2(-1.0, 0.0), inv = make_double2(1.0, 0.0);
      if (a2 > 1e-290) {
        const double ra = fast_rsq(a2), ab = a2 * ra;
        D = make_double2(-pv.x * ra, -pv.y * ra);
        inv = cscale(cconj(pv), ra * fast_rcp(ab + 1.0));  // 1 / (pv - D)
      }
      if (i == s) {
        v = cmul(rv, inv);
        y = cmul(ry, inv);
        if (on && j == s) Dv[s] = D;
      } else {
        const double2 l = cneg(cmul(ci, inv));
        v = cfma(l, rv, v);
        y = cfma(l, ry, y);
      }
      if (s + 1 < BW) {
        if (on) {
          if (i == s + 1) {
            sh.row[nxt][0][j] = v;
            sh.row[nxt][1][j] = y;
          }
          if (j == s + 1) sh.col[nxt][i] = v;
        }
        __syncthreads();
      }
    }
    // an inverse far above the order of 1 would cost H its unitarity
    if (!__syncthreads_and(fabs(y.x) < 1e3 && fabs(y.y) < 1e3)) state = 1;
  }
  if (state != 0) {
    // 1: column by column, by the first block; 2: H = I.  V and its probe partials are
    // cleared where that leaves them
    const int me = state == 1 ? panel_extent(p, j0, &last) : 0;
    if (row < n && row - t >= me) {
#pragma unroll
      for (int r = 0; r < 4; ++r) V[(int64_t)row * BW + hi + 4 * r] = czero();
    }
    if ((bx > 0 || state == 2) && tid < BW) p.pd[(int64_t)bx * BW + tid] = czero();
    if (bx > 0) return;
    if (state == 2) {
      if (on) p.sm[tid] = czero();
    } else if (me <= 64) {
      panel_small(p, k, me, red, G, L);
    } else {
      panel_direct<NW>(p, k, me, red, G, L);
    }
    return;
  }
  if (bx == 0 && on) {  // T = -D^* (Q_top - D)^-H and R = D R2 R1
    p.sm[j * BW + i] = cneg(cconj(cmul(Dv[j], y)));
    if (i <= j) {
      double2 r = czero();
      for (int q = i; q <= j; ++q) r = cfmac(p.sm[256 + j * BW + q], L[i * LDT + q], r);
      p.M[t + i + (int64_t)(j0 + j) * p.ld] = cmul(Dv[i], r);
    }
  }
  Acc acc;  // V = Q1 R2^-1 - [D; 0]
#pragma unroll
  for (int c = 0; c < 4; ++c)
    acc.mac(Li[(hi + 4 * c) * LDT + lo], keep2(row < n, qf[c]));
  const bool top = bx == 0 && wid == 0;
  const double2 yr = p.yp ? p.yp[min(row, n - 1)] : czero();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int vec = hi + 4 * r;
    double2 o = acc.at(r);
    if (top && lo == vec) o = csub(o, Dv[vec]);
    if (row < n) V[(int64_t)row * BW + vec] = o;
    const double2 d = row_sum(keep2(row < n, cmulc(o, yr)));
    if (lo == 0) red[wid * BW + vec] = d;
  }
  __syncthreads();
  if (tid < BW) {
    double2 s = czero();
#pragma unroll
    for (int w = 0; w < NW; ++w) s = cadd(s, red[w * BW + tid]);
    p.pd[(int64_t)bx * BW + tid] = s;
  }
}

// ------------------------------------------------ trailing update and S V
// Tiles of the lower triangle of the trailing matrix (order m from row t), RH ST x
// ST in tile-row order, RH (I + 1) of them in tile-row I; block b of G takes the run
// [T b / G, T (b+1) / G).  A tile-row's part inside one run is a piece.  Row r of
// tile-row Ir collects
//   Y[p][r]        p = 0 .. nrs - 1   the pieces of tile-row Ir: S V over them
//   Y[ycs + I][r]  I = Ir .. nI - 1   tile (I, r / ST): S^H V_I
__host__ __device__ inline int64_t run_start(int64_t T, int G, int b) { return T * b / G; }
__host__ __device__ inline int block_of(int64_t T, int G, int64_t t) {
  return (int)(((t + 1) * G - 1) / T);
}

// CODE = ST RH: tiles of ST columns and RH ST rows.
template <int CODE>
struct StepShape {
  static constexpr int ST = CODE > 64 ? 64 : CODE, RH = CODE / ST, RT = RH * ST;
};

template <int ST, int RH>
struct StepSmem {
  double2 v[RH * ST][LDT], w[RH * ST][LDT];  // previous panel's V and W, the tile-row's rows
  double2 x[RH * ST][LDT];                   // this panel's V
  double2 tr[RH * ST / 16][16 * LDT];        // per wavefront: a 16 x 16 block, transposed
  double2 col[RH > 1 ? ST / 16 : 1][256];    // the lower half's column sums
};

// Wavefront w of a block: tile columns 16 wc .. 16 wc + 15 of the row half rh, w = rh SR + wc.
template <int CODE>
__global__ __launch_bounds__(4 * CODE, 2) void k_band_step(BandArgs a, BandFirst f, int k) {
  constexpr int ST = StepShape<CODE>::ST, RH = StepShape<CODE>::RH, RT = StepShape<CODE>::RT;
  constexpr int SR = ST / 16;              // 16-row blocks of a half, its wavefronts
  constexpr int STEP_THREADS = 64 * SR * RH;
  const int pi = band_problem(f);
  const BandProb& p = a.p[pi];
  if (failed(p.info)) return;
  const int bx = (int)blockIdx.x - f.b[pi], G = f.b[pi + 1] - f.b[pi];
  const int t = BW * (k + 1), n = p.n, nI = cdiv(n - t, RT);
  const int64_t T = (int64_t)RH * nI * (nI + 1) / 2, N16 = (int64_t)n * BW, ld = p.ld;
  const int64_t t_end = run_start(T, G, bx + 1);
  __shared__ StepSmem<ST, RH> sm;
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 15, hi = lane >> 4;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wid % SR, rh = wid / SR;
  const bool upd = k > 0;  // a previous panel to apply
  const double2* __restrict__ Vn = v_of(p, k);
  const double2* __restrict__ Vp = v_of(p, k - 1);
  const double2* __restrict__ Wp = w_of(p, k - 1);
  double2* __restrict__ M = p.M;
  double2* __restrict__ Y = p.Y;

  int64_t tt = run_start(T, G, bx);
  int I = (int)((sqrt(8.0 * (double)(tt / RH) + 1.0) - 1.0) * 0.5);
  if ((int64_t)(I + 1) * (I + 2) / 2 <= tt / RH) ++I;
  if ((int64_t)I * (I + 1) / 2 > tt / RH) --I;
  int J = (int)(tt - (int64_t)RH * I * (I + 1) / 2);

  auto stage_rows = [&]() {  // the tile-row's rows of V, W and this panel's V
    for (int e = tid; e < RT * BW; e += STEP_THREADS) {
      const int r = e >> 4, c = e & 15, row = t + I * RT + r;
      const int64_t at = (int64_t)min(row, n - 1) * BW + c;
      const bool ok = row < n;
      sm.x[r][c] = keep2(ok, Vn[at]);
      if (upd) {
        sm.v[r][c] = keep2(ok, Vp[at]);
        sm.w[r][c] = keep2(ok, Wp[at]);
      }
    }
  };
  // block (rs, wc) of the half of tile (I, J), as the transposed 16 x 16 block: register r
  // of lane l holds row l % 16, column l / 16 + 4 r
  auto load = [&](double2(&s)[4], int I_, int J_, int rs) {
    const int64_t row = min(t + I_ * RT + rh * ST + rs * 16 + lo, n - 1);
    const int c0 = t + J_ * ST + wc * 16 + hi;
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = M[row + (int64_t)min(c0 + 4 * r, n - 1) * ld];
  };

  Acc row_acc[SR];
  stage_rows();
  double2 s[4], sn[4];
  load(s, I, J, 0);
  __syncthreads();
  while (tt < t_end) {  // uniform
    const int cj = t + J * ST + wc * 16;  // first column of this wavefront
    // this wavefront's columns of the operands
    double2 aw[4], av[4], ax[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const bool okm = cj + lo < n, okk = cj + hi + 4 * c < n;
      const int64_t at = (int64_t)min(cj + lo, n - 1) * BW + hi + 4 * c;
      if (upd) {
        aw[c] = keep2(okm, cconj(Wp[at]));
        av[c] = keep2(okm, cconj(Vp[at]));
      }
      ax[c] = keep2(okk, Vn[(int64_t)min(cj + hi + 4 * c, n - 1) * BW + lo]);
    }
    const bool row_end = J + 1 == RH * (I + 1);
    const int In = row_end ? I + 1 : I, Jn = row_end ? 0 : J + 1;
    const bool more = tt + 1 < t_end;
    Acc col;
#pragma unroll
    for (int rs = 0; rs < SR; ++rs) {
      // the next block's loads (past the run: this tile again, unused)
      if (rs + 1 < SR)
        load(sn, I, J, rs + 1);
      else
        load(sn, more ? In : I, more ? Jn : J, 0);
      const int off = ((I * RH + rh) - J) * SR + rs - wc;  // 16-row blocks below the diagonal
      const bool below = off > 0, diag = off == 0;         // uniform
      if (below || diag) {
        const int r0 = rh * ST + rs * 16;
        if (upd) {
          Acc u;
#pragma unroll
          for (int c = 0; c < 4; ++c) u.mac(aw[c], sm.v[r0 + lo][hi + 4 * c]);
#pragma unroll
          for (int c = 0; c < 4; ++c) u.mac(av[c], sm.w[r0 + lo][hi + 4 * c]);
          const int row = t + I * RT + r0 + lo;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            s[r] = csub(s[r], u.at(r));
            const int colr = cj + hi + 4 * r;
            if (row < n && colr < n && (below || lo >= hi + 4 * r))
              M[row + (int64_t)colr * ld] = s[r];
          }
        }
        if (diag) {  // lower triangle of the block, the diagonal real
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int cc = hi + 4 * r;
            s[r] = make_double2(lo >= cc ? s[r].x : 0.0, lo > cc ? s[r].y : 0.0);
          }
        }
        // transposed through LDS for the product with S^H
        double2* tr = sm.tr[wid];
#pragma unroll
        for (int r = 0; r < 4; ++r) tr[(hi + 4 * r) * LDT + lo] = s[r];
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 4; ++c) row_acc[rs].mac(ax[c], s[c]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          double2 v = cconj(tr[lo * LDT + hi + 4 * c]);  // conj S[row hi + 4c][column lo]
          if (diag && lo == hi + 4 * c) v = czero();
          col.mac(sm.x[r0 + hi + 4 * c][lo], v);
        }
        wave_lds_sync();
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = sn[r];
    }
    // S_IJ^H V_I: [vec][column] of this wavefront's 16 columns, the lower half's through LDS
    if constexpr (RH > 1) {
      __syncthreads();  // the previous tile's are read
      if (rh > 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sm.col[wc][(hi + 4 * r) * 16 + lo] = col.at(r);
      }
      __syncthreads();
    }
    if (rh == 0 && cj + lo < n) {
      double2* y = Y + (int64_t)(p.ycs + I) * N16 + (int64_t)(cj + lo) * BW;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double2 v = col.at(r);
        if constexpr (RH > 1) v = cadd(v, sm.col[wc][(hi + 4 * r) * 16 + lo]);
        y[hi + 4 * r] = v;
      }
    }
    if (row_end || !more) {
      // end of a piece: the wavefronts' row sums, two 16-row blocks at a time
      // through the operand rows' space
      double2* red = &sm.v[0][0];  // RH x SR x 2 x 256 values of the 3 RT LDT there are
      static_assert(RH * SR * 2 * 256 <= 3 * RT * LDT, "row sums fit in the operand rows");
      const int slot = bx - block_of(T, G, (int64_t)RH * I * (I + 1) / 2);
      double2* y = Y + (int64_t)slot * N16;
#pragma unroll
      for (int half = 0; half < SR / 2; ++half) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            red[(wid * 2 + q) * 256 + lo * BW + hi + 4 * r] = row_acc[2 * half + q].at(r);
        __syncthreads();
        for (int e = tid; e < RH * 512; e += STEP_THREADS) {
          const int q = e >> 9;  // row half
          const int row = t + I * RT + q * ST + half * 32 + ((e & 511) >> 4);
          double2 o = czero();
#pragma unroll
          for (int w = 0; w < SR; ++w) o = cadd(o, red[(q * SR + w) * 512 + (e & 511)]);
          if (row < n) y[(int64_t)row * BW + (e & 15)] = o;
        }
      }
#pragma unroll
      for (int rs = 0; rs < SR; ++rs) row_acc[rs] = Acc();
      __syncthreads();
      if (more) {
        I = In;
        J = Jn;
        stage_rows();
        __syncthreads();
      }
    } else {
      J = Jn;
    }
    ++tt;
  }
}

// --------------------------------------------------- X, V^H X and the probe
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_band_x(BandArgs a, BandFirst f, int k, BandFirst gs) {
  constexpr int RB = 16 * NW, NT = 64 * NW;
  const int pi = band_problem(f);
  const BandProb& p = a.p[pi];
  if (failed(p.info)) return;
  const int bx = (int)blockIdx.x - f.b[pi];
  const int t = BW * (k + 1), n = p.n, m = n - t;
  const int RH = step_halves(m), rows = RH * step_tile(m), nI = cdiv(m, rows);
  const int G = gs.b[pi];  // blocks of this problem's k_band_step launch
  const int64_t T = (int64_t)RH * nI * (nI + 1) / 2, N16 = (int64_t)n * BW;
  __shared__ double2 xs[RB * LDT];
  __shared__ double2 red[NW * 256];
  __shared__ double2 sc[BW], cv[BW], Ts[256];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, lo = lane & 15, hi = lane >> 4;
  const double2* V = v_of(p, k);
  if (p.yp) {
    if (tid < 256) Ts[tid] = p.sm[tid];
    const int c = tid & 15, g = tid >> 4;  // partial sums of the blocks' V^H y
    double2 s = czero();
    for (int b = g; b < panel_blocks(m); b += NT / BW) s = cadd(s, p.pd[(int64_t)b * BW + c]);
    red[g * BW + c] = s;
  }
  double2 vf[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    vf[c] = V[(int64_t)min(t + bx * RB + wid * 16 + hi + 4 * c, n - 1) * BW + lo];
  // the sums over the slots: column c of rows rr0 + 16 w, the rows of a tile-row at
  // a time (four rows per thread, eight slots of each in flight)
  {
    const int c = tid & 15, rr0 = tid >> 4;
    constexpr int RT = NT / BW;      // rows per pass
    constexpr int QR = RB / RT;      // passes
    static_assert(QR == 4 && RT * 4 == RB, "four rows per thread");
    double2 x[QR];
    int nrs[QR], tot[QR], Ir[QR], lr[QR], most = 0;
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      x[q] = czero();
      lr[q] = min(bx * RB + rr0 + RT * q, m - 1);
      Ir[q] = lr[q] / rows;
      const int64_t s0 = (int64_t)RH * Ir[q] * (Ir[q] + 1) / 2;
      nrs[q] = block_of(T, G, s0 + RH * (Ir[q] + 1) - 1) - block_of(T, G, s0) + 1;
      tot[q] = nrs[q] + nI - Ir[q];
      most = max(most, tot[q]);
    }
    const double2* __restrict__ Y = p.Y + (int64_t)t * BW + c;
    for (int u0 = 0; u0 < most; u0 += 8) {
      double2 v[QR][8];
#pragma unroll
      for (int q = 0; q < QR; ++q)
#pragma unroll
        for (int w = 0; w < 8; ++w) {
          const int u = min(u0 + w, tot[q] - 1);
          v[q][w] = Y[(int64_t)(u < nrs[q] ? u : p.ycs + Ir[q] + u - nrs[q]) * N16 +
                      (int64_t)lr[q] * BW];
        }
#pragma unroll
      for (int q = 0; q < QR; ++q)
#pragma unroll
        for (int w = 0; w < 8; ++w)
          if (u0 + w < tot[q]) x[q] = cadd(x[q], v[q][w]);
    }
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      const int rr = rr0 + RT * q;
      const bool in = bx * RB + rr < m;
      if (in) p.X[(int64_t)(t + bx * RB + rr) * BW + c] = x[q];
      xs[rr * LDT + c] = keep2(in, x[q]);
    }
  }
  __syncthreads();
  if (p.yp && tid < BW) {
    double2 s = czero();
    for (int g = 0; g < NT / BW; ++g) s = cadd(s, red[g * BW + tid]);
    sc[tid] = s;
  }
  Acc z;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int rr = wid * 16 + hi + 4 * c;
    z.mac(keep2(t + bx * RB + rr < n, cconj(vf[c])), xs[rr * LDT + lo]);
  }
  __syncthreads();
  if (p.yp && tid < BW) {  // T^H (V^H y)
    double2 s = czero();
    for (int i = 0; i < BW; ++i) s = cfmac(Ts[i * BW + tid], sc[i], s);
    cv[tid] = s;
  }
  reduce_tiles<NW>(z, red, p.z + (int64_t)bx * 256);
  if (p.yp) {  // y -= V (T^H (V^H y)), four threads per row
    const int row = t + bx * RB + (tid >> 2), c0 = 4 * (tid & 3);
    double2 d = czero();
    if (row < n) {
#pragma unroll
      for (int q = 0; q < 4; ++q) d = cfma(V[(int64_t)row * BW + c0 + q], cv[c0 + q], d);
    }
    d.x += dpp_mov<0xB1>(d.x);
    d.y += dpp_mov<0xB1>(d.y);
    d.x += dpp_mov<0x4E>(d.x);
    d.y += dpp_mov<0x4E>(d.y);
    if (row < n && c0 == 0) p.yp[row] = csub(p.yp[row], d);
  }
}

// ------------------------------------- W, the next panel's columns, its Gram
// k < 0: nothing to apply, the Gram partials of the first panel.
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_band_w(BandArgs a, BandFirst f, int k) {
  constexpr int RB = 16 * NW;
  const int pi = band_problem(f);
  const BandProb& p = a.p[pi];
  if (failed(p.info)) return;
  const int bx = (int)blockIdx.x - f.b[pi];
  const int t = BW * (k + 1), n = p.n, m = n - t;
  __shared__ double2 red[NW * 256];
  __shared__ double2 Z[256], tmp[256], Ts[256], Xt[256], Vt[256], Wc[BW * LDT];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, lo = lane & 15, hi = lane >> 4;
  const int row = t + bx * RB + wid * 16 + lo;
  double2 s[4];  // the next panel's columns t .. t + 15 on this row (transposed block)
#pragma unroll
  for (int r = 0; r < 4; ++r)
    s[r] = p.M[min(row, n - 1) + (int64_t)min(t + hi + 4 * r, n - 1) * p.ld];
  if (k >= 0) {
    const double2* V = v_of(p, k);
    double2* W = w_of(p, k);
    double2 xf[4], vf[4];  // this tile's rows of X and V
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int64_t at = (int64_t)min(row, n - 1) * BW + hi + 4 * c;
      xf[c] = keep2(row < n, p.X[at]);
      vf[c] = keep2(row < n, V[at]);
    }
    const int e = tid & 255, i = e >> 4, j = e & 15;
    if (tid < 256) {
      const int64_t at = (int64_t)min(t + i, n - 1) * BW + j;
      Ts[e] = p.sm[e];
      Xt[e] = keep2(t + i < n, p.X[at]);
      Vt[e] = keep2(t + i < n, V[at]);
    }
    sum_partials<NW>(p.z, panel_blocks(m), Z, tmp);
    // Z T and X_top T, then N = -1/2 T^H (Z T), then W_top = X_top T + V_top N: one
    // element per thread on the vector ALU (chains of 16; the matrix cores would
    // take twelve dependent products for each)
    double2 zt = czero(), xt = czero(), nn = czero();
    if (tid < 256) {
#pragma unroll
      for (int q = 0; q < BW; ++q) {
        zt = cfma(Z[i * BW + q], Ts[q * BW + j], zt);
        xt = cfma(Xt[i * BW + q], Ts[q * BW + j], xt);
      }
      tmp[e] = zt;
    }
    __syncthreads();
    if (tid < 256) {
#pragma unroll
      for (int q = 0; q < BW; ++q) nn = cfmac(Ts[q * BW + i], tmp[q * BW + j], nn);
      Z[e] = cscale(nn, -0.5);
    }
    __syncthreads();
    if (tid < 256) {
#pragma unroll
      for (int q = 0; q < BW; ++q) xt = cfma(Vt[i * BW + q], Z[q * BW + j], xt);
      Wc[i * LDT + j] = xt;
    }
    Acc wt;  // W^T of this tile
#pragma unroll
    for (int c = 0; c < 4; ++c) wt.mac(Ts[(hi + 4 * c) * BW + lo], xf[c]);
#pragma unroll
    for (int c = 0; c < 4; ++c) wt.mac(Z[(hi + 4 * c) * BW + lo], vf[c]);
    __syncthreads();
    Acc u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 wr = wt.at(r);
      if (row < n) W[(int64_t)row * BW + hi + 4 * r] = wr;
      u.mac(cconj(Wc[lo * LDT + hi + 4 * r]), vf[r]);
      u.mac(cconj(Vt[lo * BW + hi + 4 * r]), wr);
    }
    // lower triangle only in the top tile, its diagonal real
    const bool top = bx == 0 && wid == 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = hi + 4 * r;
      s[r] = csub(s[r], u.at(r));
      if (top && lo == c) s[r].y = 0.0;
      if (row < n && t + c < n && (!top || lo >= c)) p.M[row + (int64_t)(t + c) * p.ld] = s[r];
    }
  }
  // Gram partials of the next panel: rows t + 16 ..
  Acc g;
  {
    double2* tr = red + wid * 256;
    const bool ok = row < n && row >= t + BW;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = hi + 4 * r;
      tr[lo * BW + (c ^ lo)] = keep2(ok && t + c < n, s[r]);
    }
    wave_lds_sync();
    double2 x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int rr = hi + 4 * c;
      x[c] = tr[rr * BW + (lo ^ rr)];
    }
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < 4; ++c) g.mac(cconj(x[c]), x[c]);
  }
  reduce_tiles<NW>(g, red, p.g1 + (int64_t)bx * 256);
}

// ------------------------------------------------------------ band storage
// AB[c][d] = S[c + d][c] for d <= BW, zero for the diagonals that bulges will
// use, and the probe; the chase's ticket and progress words are cleared, also for a
// problem that has failed: the ticket of a batch is its first problem's.
__global__ void k_band_pack(BandArgs a, BandFirst f) {
  const int pi = band_problem(f);
  const BandProb& p = a.p[pi];
  const int bx = (int)blockIdx.x - f.b[pi], nb = f.b[pi + 1] - f.b[pi];
  const int n = p.n;
  for (int e = bx * blockDim.x + threadIdx.x; e < band_ctl_ints(n); e += nb * blockDim.x)
    p.ctl[e] = 0;
  if (failed(p.info)) return;
  for (int64_t e = (int64_t)bx * blockDim.x + threadIdx.x; e < (int64_t)n * ABS;
       e += (int64_t)nb * blockDim.x) {
    const int c = (int)(e / ABS), d = (int)(e % ABS);
    double2 v = czero();
    if (d <= BW && c + d < n) v = p.M[c + d + (int64_t)c * p.ld];
    if (d == 0) v.y = 0.0;
    if (d == 2 * BW && p.yp) v = p.yp[c];
    p.AB[e] = v;
  }
}

// -------------------------------------------------------------- the chase
// Band to tridiagonal.  Sweep s (s = 0 .. n - 2) reduces column s: its task k =
// 0 forms the reflector of A[s+1 .. s+BW, s] and applies it on both sides of
// the diagonal block; task k >= 1, on rows R_k = s + 1 + BW k .. (BW of them) and
// columns R_{k-1}, applies the previous reflector from the right to that block,
// forms the reflector that annihilates the block's first column below its first
// row, and applies it from the left to the block and on both sides to the
// diagonal block of R_k.  Only the first column of a bulge is annihilated; the
// rest stays for the next sweep, whose blocks sit one row further down, so 2 BW
// diagonals are stored.  Task (s, k) needs task (s - 1, k + 1) to be done: sweep s
// runs two tasks behind sweep s - 1.
//
// A block takes CS consecutive sweeps (a group) and moves with them down the
// band: at step i sweep w of the group does task i - 2 w, with one barrier per
// step; the columns in use lie in a ring of LDS.  A column leaves the ring for
// memory when the group's last sweep has passed it, and the next group's first
// sweep takes it from there.  The chain of dependent tasks, 2 n of them, is what
// bounds the kernel: grouping keeps the hand-over between blocks out of all but
// one step in 2 CS, and wavefronts of their own carry the columns into the ring
// (FW of them, requests two steps ahead) and out of it (LW of them), so that the
// sweeps do not wait for memory.
//
// Groups are taken in order from a ticket counter, and a group waits only for
// progress of the group before it, which a running block holds, so every wait
// ends whatever blocks are resident.  Columns that pass between blocks are
// stored through the L2 caches and loaded past them (device scope, the XCDs' L2
// caches are not coherent by themselves); the progress word follows a wait for
// the stores.
constexpr int CS = CHASE_SWEEPS;
constexpr int FW = 2;  // wavefronts that fetch columns, in turn
constexpr int LW = 2;  // wavefronts that store finished columns, in turn
constexpr int CH_THREADS = 64 * (2 * CS + FW + LW);
constexpr int RING = 256;  // columns in LDS: 31 CS + 17 in use, 16 more on their way out
static_assert(31 * CS + 17 + 16 <= RING, "the ring holds a group's columns");
constexpr int CHASE_SPIN = 1 << 22;  // polls before a group gives up (never reached in order)

// 16-byte loads and stores at device scope (sc1).  The buffer descriptor's size
// makes loads past the band zero and drops stores there.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int DEVICE_SCOPE = 0x10;
constexpr int BUFFER_FLAGS = 0x00027000;  // raw buffer, 32-bit data

// One task of a sweep takes two wavefronts: one works on the block below the
// diagonal and forms the reflector, the other applies the reflector to the
// diagonal block and the probe one step later (what the next sweep needs of them
// is then still one step ahead of its use).  The kernel is bound by what its four
// SIMDs issue per step.  Lane l: lo = l % 16, hi = l / 16.  Blocks that are updated
// are held with column lo and rows hi + 4 c, so that sums over rows run over the
// lane's four values and the four lane groups.  (The rank-two updates on the matrix
// cores, a 16 x 16 x 4 product each for the real and the imaginary part, take more
// instructions to arrange than the vector ALU's 32.)
// A group of CS sweeps follows the one before it by about ten steps of 1.2 us: n = 324,
// 1875, 6144: 0.97, 6.3, 22.6 ms (1.09, 7.1, 26.6 ms when a group waited for 33 columns
// in place of chunks of 16, polled within the step and gave both tasks the same
// priority).  CS = 2, 3, 5: 0.96, 0.99, 1.02 ms at n = 324, 7.2, 6.8, 7.5 at 1875, 7.7,
// 7.5, 8.2 at 2048 (CS = 4: 6.9), 31.0, 25.5, 26.8 at 6144.

// The block at rows r0 .. r0 + 15 and columns r0 - 16 .. r0 - 1 (first: the column
// s alone), by one wavefront: the previous reflector from the right, B - z v^H; the
// reflector u of the first column x; and u from the left,
//   B - z v^H - u G,  G = conj(tau) (u^H B - (u^H z) v^H),
// u^H z from the first column of u^H B and u^H x = x_0 + conj(scal) sum_{i>0} |x_i|^2.
// x: the first column (element lo); v, vq, tau: the sweep's reflector at lo and at
// hi + 4 c (in: of the previous task; out: u).  ub: BW + 1 values of LDS that take u
// and tau for the other wavefront.  Returns the column's new first element.
BSE_DEV double chase_bulge(double2* ring, double2* ub, int lo, int hi, int r0, bool first,
                           double2 x, double2& v, double2 (&vq)[4], double2& tau) {
  // element (i, j) of the block is diagonal BW + i - j of column r0 - BW + j
  auto at = [&](int i, int j) { return ((r0 - BW + j) & (RING - 1)) * ABS + BW + i - j; };
  double2 Bt[4], xq[4], zq[4], b0 = czero();
  if (!first) {  // uniform
    double2 B[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) B[c] = ring[at(lo, hi + 4 * c)];
#pragma unroll
    for (int c = 0; c < 4; ++c) Bt[c] = ring[at(hi + 4 * c, lo)];
    b0 = ring[at(0, lo)];
#pragma unroll
    for (int c = 0; c < 4; ++c) zq[c] = ring[at(hi + 4 * c, 0)];
    const double2 z0 = cfma(B[2], vq[2], cmul(B[0], vq[0]));
    const double2 z1 = cfma(B[3], vq[3], cmul(B[1], vq[1]));
    const double2 z = quad_rows_sum(cadd(z0, z1));
    x = cfma(cneg(tau), z, x);  // the reflector's first element is 1
  }
  ub[lo] = x;  // (the four lane groups hold the same values)
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < 4; ++c) xq[c] = ub[hi + 4 * c];
  // beta, tau, scal: I - tau u u^H with u = (1, scal x_1, ...) takes x to (beta, 0, ...)
  const double xn2 = row_sum(lo > 0 ? cabs2(x) : 0.0);
  const double2 al = make_double2(lane_value(x.x, 0), lane_value(x.y, 0));
  const double nn = fma(al.x, al.x, fma(al.y, al.y, xn2));
  const bool ok = nn > COLUMN_ZERO && (xn2 != 0.0 || al.y != 0.0);
  const double r = fast_rsq(nn), rb = -copysign(r, al.x), b = nn * rb;
  const double2 dn = make_double2(al.x - b, al.y);
  const double q = fast_rcp(cabs2(dn));
  const double2 scal = keep2(ok, make_double2(dn.x * q, -dn.y * q));
  const double2 tn = keep2(ok, make_double2(-dn.x * rb, -al.y * rb));
  const double beta = ok ? b : al.x;
  double2 u = cmul(scal, x);
  u.x = lo == 0 ? 1.0 : u.x;
  u.y = lo == 0 ? 0.0 : u.y;
#pragma unroll
  for (int c = 0; c < 4; ++c) vq[c] = cmul(scal, xq[c]);
  vq[0].x = hi == 0 ? 1.0 : vq[0].x;
  vq[0].y = hi == 0 ? 0.0 : vq[0].y;
  if (!first) {
    // u^H B with the unscaled x (it does not wait for the scalars)
#pragma unroll
    for (int c = 0; c < 4; ++c) zq[c] = csub(xq[c], zq[c]);  // -z, from the first column
    xq[0] = keep2(hi > 0, xq[0]);
    const double2 g0 = cfmac(xq[2], Bt[2], cmulc(xq[0], Bt[0]));
    const double2 g1 = cfmac(xq[3], Bt[3], cmulc(xq[1], Bt[1]));
    const double2 ug = cfmac(scal, quad_rows_sum(cadd(g0, g1)), b0);
    const double2 ux = make_double2(fma(scal.x, xn2, al.x), fma(-scal.y, xn2, al.y));
    const double2 uz = csub(ux, make_double2(lane_value(ug.x, 0), lane_value(ug.y, 0)));  // -u^H z
    const double2 G = cmulc(cneg(tn), cfmac(v, uz, ug));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      // the first column is known: (beta, 0, ...)
      double2 o = cfma(vq[c], G, cfmac(v, zq[c], Bt[c]));
      o.x = lo ? o.x : (c == 0 && hi == 0 ? beta : 0.0);
      o.y = lo ? o.y : 0.0;
      ring[at(hi + 4 * c, lo)] = o;
    }
  }
  ub[lo] = u;
  ub[BW] = tn;
  tau = tn;
  v = u;
  return beta;
}

// The diagonal block at rows r0 .. r0 + 15 and the probe's rows, with the reflector
// in ub: D := H^H D H = D - u w^H - w u^H, w = tau D u - 1/2 |tau|^2 (u^H D u) u, and
// y := H^H y.  ws: BW values of LDS.
BSE_DEV void chase_diag(double2* ring, const double2* ub, double2* ws, int lo, int hi, int r0) {
  auto slot = [&](int c) { return ((r0 + c) & (RING - 1)) * ABS; };
  int oD[4];
  double2 D[4], uq[4], wq[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int i = hi + 4 * c;
    oD[c] = slot(min(i, lo)) + abs(i - lo);
    D[c] = ring[oD[c]];
    uq[c] = ub[i];
  }
  const int oy = slot(lo) + 2 * BW;
  const double2 u = ub[lo], tau = ub[BW], y = ring[oy];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int i = hi + 4 * c;
    D[c].y = i == lo ? 0.0 : i > lo ? D[c].y : -D[c].y;
  }
  // (D u)_lo = sum_i conj(D_i,lo) u_i
  const double2 q0 = cfmac(D[2], uq[2], cmulc(D[0], uq[0]));
  const double2 q1 = cfmac(D[3], uq[3], cmulc(D[1], uq[1]));
  const double2 q = quad_rows_sum(cadd(q0, q1));
  const double uq2 = row_sum(fma(u.x, q.x, u.y * q.y));
  const double hl = -0.5 * cabs2(tau) * uq2;
  const double2 tq = cmul(tau, q);
  const double2 w = make_double2(fma(u.x, hl, tq.x), fma(u.y, hl, tq.y));
  ws[lo] = w;
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < 4; ++c) wq[c] = ws[hi + 4 * c];
  const double2 sy = row_sum(cmulc(u, y));
  if (hi == 0) ring[oy] = cfma(cmulc(tau, u), cneg(sy), y);
  const double2 nu = cneg(u), nw = cneg(w);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int i = hi + 4 * c;
    double2 d = cfmac(nu, wq[c], cfmac(nw, uq[c], D[c]));
    if (i == lo) d.y = 0.0;
    if (i >= lo) ring[oD[c]] = d;
  }
}

// The lane number, opaque to the compiler: what a kind of wavefront derives from
// it stays inside that kind's loop (hoisted out of it, the index values of all
// kinds would be live, and spilled, in each).
BSE_DEV int opaque_lane() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

__global__ __launch_bounds__(CH_THREADS) void k_band_chase(BandArgs a, int np, int gmax) {
  __shared__ double2 ring[RING * ABS];
  __shared__ double2 ub[CS][2][BW + 1], ws[CS][BW];
  __shared__ int tick;
  constexpr int CHUNK = BW * ABS;  // values of 16 columns
  constexpr int PER = (CHUNK + 63) / 64;
  const int tid = threadIdx.x;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto slot = [](int c) { return (c & (RING - 1)) * ABS; };
  auto wrap = [](int e) { return e >= RING * ABS ? e - RING * ABS : e; };
  for (;;) {
    __syncthreads();
    if (tid == 0) {
      // the next group of a problem that has not failed: one thread looks, since
      // another block may set info between two wavefronts' looks
      int t;
      do {
        t = __hip_atomic_fetch_add(a.p[0].ctl + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } while (t >= 0 && t < gmax * np &&
               (t / np * CS >= max(a.p[t % np].n - 1, 1) || failed(a.p[t % np].info)));
      tick = t;
    }
    __syncthreads();
    const int tk = __builtin_amdgcn_readfirstlane(tick);
    if (tk < 0 || tk >= gmax * np) return;  // every ticket is taken
    const int pi = tk % np, g = tk / np;
    const BandProb& p = a.p[pi];
    const int n = p.n, s0 = g * CS;
    const __amdgpu_buffer_rsrc_t AB = __builtin_amdgcn_make_buffer_rsrc(
        (void*)p.AB, (short)0, n * ABS * (int)sizeof(double2), BUFFER_FLAGS);
    int32_t* prog = p.ctl + 2;
    int seen = g ? 0 : n;  // columns below this are final in memory
    // wait until the previous group has left every column below `need`
    auto wait_for = [&](int need) {
      for (int spin = 0; seen < need; ++spin) {
        seen = __hip_atomic_load(prog + g - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (spin > CHASE_SPIN) {
          set_info(p.info, BSE_INFO_NO_CONVERGE);
          seen = n;
        }
      }
      asm volatile("" ::: "memory");
    };
    // columns c0 .. c0 + 15 by one wavefront; columns past the band come as zeros,
    // which the last tasks' blocks reach
    u32x4 pre[PER];
    auto fetch = [&](int lane, int c0) {
#pragma unroll
      for (int u = 0; u < PER; ++u)
        pre[u] = __builtin_amdgcn_raw_buffer_load_b128(AB, (c0 * ABS + lane + 64 * u) * 16, 0,
                                                       DEVICE_SCOPE);
    };
    auto put = [&](int lane, int c0) {
      const int to = (c0 & (RING - 1)) * ABS + lane;
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (lane + 64 * u < CHUNK) *(u32x4*)&ring[wrap(to + 64 * u)] = pre[u];
    };
    const int slast = min(s0 + CS, n - 1) - 1;  // last sweep of the group
    // its last task, the diagonal block one step later
    const int steps = n > 1 ? 2 * (slast - s0) + (n - 2 - slast) / BW + 2 : 0;
    const int dw = wid - CS, fw = wid - 2 * CS;  // diagonal; fetching (FW: storing)
    const int lw = fw - FW;
    // step j takes columns s0 + 16 j .. + 15 (its bulge reaches the first of them);
    // those of step 0 first, those of step 1 put at step 0
    if (fw == 0 || fw == 1) {
      const int lane = opaque_lane();
      wait_for(min(n, s0 + BW * (fw + 1)));
      fetch(lane, s0 + BW * fw);
      if (fw == 0) put(lane, s0);
    }
    __syncthreads();
    // the three kinds of wavefronts, each with one barrier per step
    if (dw < 0) {
      const int lane = opaque_lane(), lo = lane & 15, hi = lane >> 4;
      double2 vq[4] = {}, v = czero(), tau = czero();
      const int s = s0 + wid;
      for (int i = 0; i < steps; ++i) {
        const int k = i - 2 * wid, r0 = s + 1 + BW * k;  // first row of the task
        if (s <= slast && k >= 0 && r0 < n) {            // uniform
          const double2 x = ring[k ? slot(r0 - BW) + BW + lo : slot(s) + 1 + lo];
          const double beta = chase_bulge(ring, ub[wid][i & 1], lo, hi, r0, k == 0, x, v, vq, tau);
          if (k == 0 && lane == 0) {
            p.ee[s] = beta;
            p.dd[s] = ring[slot(s)].x;
            if (p.yp) p.yp[s] = ring[slot(s) + 2 * BW];
          }
        }
        __syncthreads();
      }
    } else if (fw < 0) {
      const int lane = opaque_lane(), lo = lane & 15, hi = lane >> 4;
      __builtin_amdgcn_s_setprio(2);  // the longer of the two tasks of a step on its SIMD
      const int s = s0 + dw;
      for (int i = 0; i < steps; ++i) {
        const int k = i - 1 - 2 * dw, r0 = s + 1 + BW * k;
        if (s <= slast && k >= 0 && r0 < n)  // uniform
          chase_diag(ring, ub[dw][(i & 1) ^ 1], ws[dw], lo, hi, r0);
        __syncthreads();
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (lw < 0) {
      // the previous group's progress is asked for one step before it is needed: in a
      // steady flow no step waits for a poll
      const int lane = opaque_lane();
      int asked = seen;
      for (int i = 0; i < steps; ++i) {
        if ((i & 1) == fw) {  // request the columns of step i + 2
          seen = max(seen, asked);
          wait_for(min(n, s0 + BW * (i + 3)));
          fetch(lane, s0 + BW * (i + 2));
        } else {
          put(lane, s0 + BW * (i + 1));
          if (seen < n)
            asked = __hip_atomic_load(prog + g - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
      }
    } else {
      // columns that the group's last sweep passed at step i - 1 go to memory at
      // step i and are published at step i + 1
      const int lane = opaque_lane();
      int left = 0;
      for (int i = 0; i < steps; ++i) {
        const int kl = i - 1 - 2 * (CS - 1);
        if ((i & (LW - 1)) == lw) {
          if (kl >= 1) {
            const int c0 = s0 + CS + BW * (kl - 1);
            const int from = (c0 & (RING - 1)) * ABS + lane;
            u32x4 v[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) v[u] = *(const u32x4*)&ring[wrap(from + 64 * u)];
#pragma unroll
            for (int u = 0; u < PER; ++u)
              if (lane + 64 * u < CHUNK)
                __builtin_amdgcn_raw_buffer_store_b128(v[u], AB, (c0 * ABS + lane + 64 * u) * 16, 0,
                                                       DEVICE_SCOPE);
            left = min(c0 + BW, n);
          }
        } else if (left) {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          if (lane == 0)
            __hip_atomic_store(prog + g, left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
      }
    }
    // what is left of the band, and the last diagonal element
    {
      const int kl = steps - 2 - 2 * (CS - 1);
      const int c0 = s0 + CS + (kl >= 1 ? BW * kl : 0);
      const int from = (c0 & (RING - 1)) * ABS;
      for (int e = tid; e < (n - c0) * ABS; e += CH_THREADS)
        __builtin_amdgcn_raw_buffer_store_b128(*(const u32x4*)&ring[wrap(from + e)], AB,
                                               (c0 * ABS + e) * 16, 0, DEVICE_SCOPE);
    }
    if (slast == n - 2 && tid == 0) {
      const int last = n - 1;
      p.dd[last] = ring[slot(last)].x;
      if (p.yp) p.yp[last] = ring[slot(last) + 2 * BW];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) __hip_atomic_store(prog + g, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

int device_cus() {
  static const int cus = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    return v;
  }();
  return cus;
}

// The control words in complex elements, rounded to 256 bytes.
int64_t ctl_elems(int64_t n) { return (((int64_t)band_ctl_ints((int)n) + 63) / 64) * 16; }

// Blocks of a k_band_step launch over a trailing matrix of order m: up to eight
// wavefronts per compute unit, two per SIMD.
int step_grid(int64_t m) {
  const int64_t rh = step_halves(m), rt = rh * step_tile(m);
  const int64_t nI = (m + rt - 1) / rt, T = rh * nI * (nI + 1) / 2;
  return (int)std::max<int64_t>(1, std::min<int64_t>((128 / rt) * device_cus(), T));
}

// Slots of k_band_step's partial products: two per tile-row, for the largest order
// of each tile edge.
int64_t step_slots(int64_t n) {
  return 2 * std::max((n + 63) / 64, (std::min<int64_t>(n, STEP_SMALL) + 31) / 32);
}

}  // namespace

bool tridiagonalise_band(const BandItem* it_all, int np_all, hipStream_t s) {
  for (int g0 = 0; g0 < np_all; g0 += BAND_BATCH_MAX) {
    const BandItem* it = it_all + g0;
    const int np = std::min(BAND_BATCH_MAX, np_all - g0);
    BandArgs A{};
    int64_t nmax = 0;
    for (int q = 0; q < np; ++q) {
      const int64_t n = it[q].n, nb = (n + 63) / 64;
      BandProb& p = A.p[q];
      p.M = it[q].M;
      p.ld = it[q].ld;
      p.n = (int)n;
      p.ycs = (int)(step_slots(n) / 2);
      p.VW = it[q].b.VW;
      p.Q1 = it[q].b.q1x;
      p.X = p.Q1 + n * BW;
      p.g1 = it[q].b.part;
      p.g2 = p.g1 + nb * 256;
      p.z = p.g2 + nb * 256;
      p.pd = p.z + nb * 256;
      p.sm = p.pd + nb * BW;
      p.yp = it[q].b.yproj;
      p.AB = it[q].b.big;
      p.ctl = (int32_t*)(p.AB + band_elems(n));
      p.Y = p.AB + band_elems(n) + ctl_elems(n);
      p.dd = it[q].b.dd;
      p.ee = it[q].b.ee;
      p.info = it[q].info;
      nmax = std::max(nmax, n);
    }
    // block ranges of a launch: `blocks(n)` blocks for the problems with panel k
    auto ranges = [&](auto blocks) {
      BandFirst f{};
      int tot = 0;
      for (int q = 0; q < BAND_BATCH_MAX; ++q) {
        f.b[q] = tot;
        if (q < np) tot += blocks((int64_t)A.p[q].n);
      }
      f.b[BAND_BATCH_MAX] = tot;
      return f;
    };
    // the panel kernels, in one launch per block size for the problems whose
    // trailing order asks for it
    auto panel = [&](int t, int least, auto launch) {
      for (int rows : {64, 128}) {
        const BandFirst f = ranges([&](int64_t n) {
          return n - t >= least && panel_rows(n - t) == rows ? panel_blocks(n - t) : 0;
        });
        if (f.b[BAND_BATCH_MAX] > 0) launch(rows, f, dim3(f.b[BAND_BATCH_MAX]));
      }
    };
#define BAND_LAUNCH(name, least, ...)                                                        \
  panel(t, least, [&](int rows, const BandFirst& f, dim3 grid) {                              \
    if (rows == 64)                                                                          \
      BSE_LAUNCH(name<4>, grid, dim3(256), 0, s, A, f, __VA_ARGS__);                          \
    else                                                                                     \
      BSE_LAUNCH(name<8>, grid, dim3(512), 0, s, A, f, __VA_ARGS__);                          \
  })
    int t = 0;  // first row and column of the trailing matrix
    BAND_LAUNCH(k_band_w, BW + 1, -1);
    for (int k = 0; BW * (k + 1) < nmax; ++k) {
      t = BW * (k + 1);
      BandFirst gs{};  // blocks of each problem's k_band_step launch
      for (int q = 0; q < np; ++q) gs.b[q] = A.p[q].n > t ? step_grid(A.p[q].n - t) : 0;
      BAND_LAUNCH(k_band_chol, DIRECT_ROWS, k);
      BAND_LAUNCH(k_band_panel, 1, k);
      for (int rt : {32, 64, 128}) {
        const BandFirst fs = ranges([&](int64_t n) {
          return n > t && step_halves(n - t) * step_tile(n - t) == rt ? step_grid(n - t) : 0;
        });
        const dim3 grid(fs.b[BAND_BATCH_MAX]);
        if (grid.x == 0) continue;
        if (rt == 32)
          BSE_LAUNCH(k_band_step<32>, grid, dim3(128), 0, s, A, fs, k);
        else if (rt == 64)
          BSE_LAUNCH(k_band_step<64>, grid, dim3(256), 0, s, A, fs, k);
        else
          BSE_LAUNCH(k_band_step<128>, grid, dim3(512), 0, s, A, fs, k);
      }
      BAND_LAUNCH(k_band_x, 1, k, gs);
      BAND_LAUNCH(k_band_w, 1, k);
    }
#undef BAND_LAUNCH
    const BandFirst fp = ranges([&](int64_t n) { return (int)std::min<int64_t>(cdiv(n * ABS, 256), 1024); });
    BSE_LAUNCH(k_band_pack, dim3(fp.b[BAND_BATCH_MAX]), dim3(256), 0, s, A, fp);
    // sweeps in flight: one group per 2 CS BW columns of the band, with room
    const int gmax = (int)std::max<int64_t>(cdiv(nmax - 1, CS), 1);
    int64_t blocks = 0;
    for (int q = 0; q < np; ++q) blocks += std::min<int64_t>(cdiv(A.p[q].n, 2 * CS * BW) + 2, gmax);
    BSE_LAUNCH(k_band_chase, dim3((unsigned)std::min<int64_t>(blocks, device_cus())),
               dim3(CH_THREADS), 0, s, A, np, gmax);
  }
  return hipGetLastError() == hipSuccess;
}

int64_t band_big_bytes(int64_t n) {
  const int64_t slots = n > BW ? step_slots(n) * n * BW : 0;
  return 16 * (band_elems(n) + ctl_elems(n) + slots);
}
int64_t band_part_bytes(int64_t n) {
  if (n <= BW) return 0;  // no panel
  return 16 * (((n + 63) / 64) * (3 * 256 + BW) + 512);
}
