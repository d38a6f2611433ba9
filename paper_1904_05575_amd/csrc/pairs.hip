// Plane-wave pair elements from orbitals (paper Sec. 4.1, for orbitals
// expanded in plane waves: the cell integral of the orbital product keeps the
// plane waves whose wave vectors cancel):
//   M_mn(k, k', G) = sum_K conj(C_m,k(K)) C_n,k'(K + G)
//   N_mn(k, k', G) = sum_K conj(C_m,k(K)) conj(C_n,k'(-K - G))
// over the orbitals' plane-wave sphere K (terms whose partner K + G or -K - G
// lies outside it are absent), for every pair ik <= ik': Mvv, Mcc (and Ncv, Nvc
// for the full BSE), and M_cv at k = k'.
#include "bse_internal.h"
#include "common.h"
#include "timing.h"

namespace {

// The sum is bound by the vector ALU, at 8 flop per (K, G) inside the sphere and pair
// of bands, if nothing else gets in its way: lanes that hold different G skip
// different K and gather from LDS with conflicts.  So G and K are uniform here: the 64
// lanes of a wavefront hold 64 columns (k', n) of one k, staged in LDS as [K'][column],
// a K outside the sphere is skipped, the partner's row is one conflict-free 16-byte
// read per lane, and conj(C_m,k(K)) comes through the scalar cache for na <= 5 bands
// m: 4 na FMA instructions per read.  Four G (two on small meshes) are summed one after
// the other and stored together, 64 consecutive bytes per element.
// 23436 pairs of 4 + 5 bands, 89 G and 89 K (45 % of them inside the sphere): 2.15 ms,
// the vector ALU busy for 68 % of it, 2.7 GB written; a lane per G with blocks padded
// to 4 x 4 bands, both operands gathered from LDS, took 4.4 ms, and 8 k' x 8 G per
// wavefront (no conflicts, but 97 % of the K in some lane's sphere) 2.9 ms.
constexpr int PG_WAVES = 16;  // four wavefronts per SIMD, one block per compute unit
constexpr int PG_THREADS = 64 * PG_WAVES;
constexpr int PG_MAXB = 5;    // bands of a block at k, of a side at k'
constexpr int PG_ROWS = 128;  // rows K' in LDS at a time
constexpr int PG_BATCH = 4;   // G of a task: 4 or 2
constexpr int PG_TR = 128;    // values of a wavefront's transposition buffer
constexpr int PG_MAXKINDS = 24;
constexpr int PG_LDS = 160 * 1024;

struct PgKind {
  double2* out;       // element (a, b, G) of pair p at out + p ps + a as + b bs + G
  int64_t ps, as, bs;
  int a0, na, nb;     // bands at k (into the nv + nc bands); bands at k'
  int ia, ib;         // first local index of this block within the array's a / b
  int modified;       // N-type element
  int diag_only;      // only diagonal pairs, p taken as ik (M_cv)
};
struct PgSide {       // a block of bands at k' and the kinds formed from it
  int b0, nb, first, count, diag;  // kinds [first, first + count), the diagonal ones last
};
struct PgKinds {
  PgKind k[PG_MAXKINDS];
  PgSide side[PG_MAXKINDS];
  int n, nsides;
};

// Groups of 64 columns of the rows k and nk - 1 - k together: at most this many.
__host__ __device__ inline int row_groups(int nk, int nb) { return ((nk + 1) * nb + 63) / 64 + 1; }

// Columns of a block: k', n of column c of row ik.
struct PgCols {
  int ik, c0, total, nb;
  BSE_DEV int jk(int c) const { return ik + c / nb; }
};

// Rows K' = r0 .. r0 + rows - 1 of the block's columns into LDS: a wavefront reads 8
// columns x 8 rows, 128 bytes of each column.
BSE_DEV void stage_rows(double2* ys, const double2* __restrict__ C, const PgCols& cols, int nbt,
                        int b0, int nkb, int r0, int rows) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int t = wid; t < (rows + 7) / 8 * 8; t += PG_WAVES) {
    const int cl = (t & 7) * 8 + (lane & 7), r = (t >> 3) * 8 + (lane >> 3);
    const int c = min(cols.c0 + cl, cols.total - 1);
    const int jk = cols.jk(c), n = c - (jk - cols.ik) * cols.nb;
    if (r < rows) ys[r * 64 + cl] = C[((int64_t)jk * nbt + b0 + n) * nkb + r0 + r];
  }
}

// One task: NA bands at k (uniform, xs: C_m,k) with the 64 columns, for NQ G from g0.
// nch > 1: the rows K' come in parts, staged by the whole block; all its wavefronts call
// with the same kind, those past the last G with none to sum.
template <int NQ, int NA, bool MOD, class Stage>
BSE_DEV void pair_task(const double2* __restrict__ xs, int nkb, const double2* ys,
                       const int32_t* __restrict__ tab, int ng, int g0, int nch, Stage stage,
                       double2* tr, const int (&pcol)[NQ], const PgKind& kd, int64_t pair0, int ik) {
  const int lane = threadIdx.x & 63;
  uint32_t xa[NA];  // bands of one k-point: at most 80 KB
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    xa[a] = (uint32_t)(a * nkb) * (uint32_t)sizeof(double2);
    asm("" : "+s"(xa[a]));  // one sum per load, not a chain of 64-bit ones
  }
  double2 acc[NQ][NA];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[q][a] = make_double2(0.0, 0.0);
  for (int ch = 0; ch < nch; ++ch) {
    const int r0 = ch * PG_ROWS, rows = min(PG_ROWS, nkb - r0);
    if (nch > 1) stage(r0, rows);
    for (int K0 = 0; K0 < nkb; K0 += 64) {
      int row[NQ];  // lane: the partner row of K0 + lane
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        row[q] = tab[(int64_t)min(K0 + lane, nkb - 1) * ng + min(g0 + q, ng - 1)] - r0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        uint64_t mask = __ballot(g0 + q < ng && K0 + lane < nkb && (unsigned)row[q] < (unsigned)rows);
        auto take = [&](double2 (&x)[NA], double2& y) __attribute__((always_inline)) {
          const int K = (int)__builtin_ctzll(mask);
          mask &= mask - 1;
          y = ys[__builtin_amdgcn_readlane(row[q], K) * 64 + lane];
          const uint32_t at = (uint32_t)(K0 + K) * (uint32_t)sizeof(double2);
#pragma unroll
          for (int a = 0; a < NA; ++a) x[a] = *(const double2*)((const char*)xs + (xa[a] + at));
        };
        auto add = [&](const double2 (&x)[NA], double2 y) __attribute__((always_inline)) {
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            // N: conj(x) conj(y) = conj(x y), negated when stored
            const double xr = x[a].x, xi = MOD ? -x[a].y : x[a].y;
            double2& t = acc[q][a];
            t.x = fma(xr, y.x, fma(xi, y.y, t.x));
            t.y = fma(xr, y.y, fma(-xi, y.x, t.y));
          }
        };
        const int terms = __popcll(mask);
        for (int i = terms >> 1; i > 0; --i) {  // two K, their loads in flight together
          double2 x0[NA], x1[NA], y0, y1;
          take(x0, y0);
          take(x1, y1);
#pragma unroll
          for (int a = 0; a < NA; ++a)
            asm volatile("" ::"s"(x0[a].x), "s"(x0[a].y), "s"(x1[a].x), "s"(x1[a].y));
          add(x0, y0);
          add(x1, y1);
        }
        if (terms & 1) {
          double2 x0[NA], y0;
          take(x0, y0);
          add(x0, y0);
        }
      }
    }
  }
  // through LDS, 32 columns at a time, into lanes with G fastest
  const int cl = lane & 31, sw = (cl >> 1) & (NQ - 1);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (lane >> 5 == h) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          tr[cl * NQ + (q ^ sw)] = make_double2(acc[q][a].x, MOD ? -acc[q][a].y : acc[q][a].y);
      }
      wave_lds_sync();
#pragma unroll
      for (int v = 0; v < NQ / 2; ++v) {
        const int e = lane + 64 * v, c = e / NQ, g = g0 + e % NQ, pc = pcol[h * (NQ / 2) + v];
        const double2 z = tr[c * NQ + (e % NQ ^ ((c >> 1) & (NQ - 1)))];
        const int jk = pc >> 3;
        if (pc >= 0 && g < ng && (!kd.diag_only || jk == ik))
          kd.out[(kd.diag_only ? ik : pair0 + jk) * kd.ps + (kd.ia + a) * kd.as +
                 (kd.ib + (pc & 7)) * kd.bs + g] = z;
      }
      wave_lds_sync();
    }
}

template <int NQ>
__global__ __launch_bounds__(PG_THREADS) void k_pair_elements(
    const double2* __restrict__ C, int nk, int nbt, int nkb, int ng,
    const int32_t* __restrict__ kpg, const int32_t* __restrict__ mkg, PgKinds kinds) {
  extern __shared__ double2 ys[];  // [min(nkb, PG_ROWS)][64], then the wavefronts' buffers
  const PgSide sd = kinds.side[blockIdx.y];
  // group -> row of the pair (k, nk - 1 - k) of rows and its group
  const int gp = row_groups(nk, sd.nb), hk = blockIdx.x / gp;
  if (hk >= (nk + 1) / 2) return;
  PgCols cols;
  cols.nb = sd.nb;
  cols.ik = hk;
  cols.total = (nk - hk) * sd.nb;
  int cg = blockIdx.x % gp;
  const int first = (cols.total + 63) / 64;
  if (cg >= first) {
    cg -= first;
    cols.ik = nk - 1 - hk;
    cols.total = (hk + 1) * sd.nb;
    if (cols.ik == hk || cg * 64 >= cols.total) return;
  }
  cols.c0 = cg * 64;
  const int ik = cols.ik;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rows0 = min(nkb, PG_ROWS), nch = (nkb + PG_ROWS - 1) / PG_ROWS;
  double2* tr = ys + rows0 * 64 + PG_TR * wid;
  int pcol[NQ];  // the columns this lane stores: k' << 3 | n
#pragma unroll
  for (int v = 0; v < NQ; ++v) {
    const int c = cols.c0 + 64 / NQ * v + lane / NQ, jk = cols.jk(c);
    pcol[v] = c < cols.total ? jk << 3 | (c - (jk - ik) * cols.nb) : -1;
  }
  const int64_t pair0 = (int64_t)ik * nk - (int64_t)ik * (ik - 1) / 2 - ik;  // + jk: the pair
  auto stage = [&](int r0, int rows) {
    __syncthreads();
    stage_rows(ys, C, cols, nbt, sd.b0, nkb, r0, rows);
    __syncthreads();
  };
  if (nch == 1) stage(0, nkb);
  const int nkinds = sd.count - (cg == 0 ? 0 : sd.diag);
  const int ngb = (ng + NQ - 1) / NQ;
  // rows in one part: the tasks of all kinds over the wavefronts; in several: kind by
  // kind, the block's wavefronts together
  const int step = PG_WAVES * (int)gridDim.z, t0 = wid + PG_WAVES * (int)blockIdx.z;
  const int per = nch == 1 ? ngb : (ngb + step - 1) / step * step;
  for (int t = t0; t < nkinds * per; t += step) {
    const PgKind& kd = kinds.k[sd.first + t / per];
    const int g0 = (t % per) * NQ;
    const int32_t* tab = kd.modified ? mkg : kpg;
    const double2* xs = C + ((int64_t)ik * nbt + kd.a0) * nkb;
#define PAIR_CASE(A, M)                                                                         \
  case M * 8 + A:                                                                               \
    pair_task<NQ, A, M>(xs, nkb, ys, tab, ng, g0, nch, stage, tr, pcol, kd, pair0, ik);             \
    break;
    switch (kd.modified * 8 + kd.na) {
      PAIR_CASE(1, 0) PAIR_CASE(2, 0) PAIR_CASE(3, 0) PAIR_CASE(4, 0) PAIR_CASE(5, 0)
      PAIR_CASE(1, 1) PAIR_CASE(2, 1) PAIR_CASE(3, 1) PAIR_CASE(4, 1) PAIR_CASE(5, 1)
    }
#undef PAIR_CASE
  }
}

// Parts of at most PG_MAXB of n bands, even: part i of `parts` begins at i n / parts.
int band_parts(int n) { return (n + PG_MAXB - 1) / PG_MAXB; }

// The kinds of an (na_tot x nb part) array of elements, appended to the list.
void add_kinds(PgKinds& ks, double2* out, int64_t ps, int64_t as, int64_t bs, int a0, int na_tot,
               int ib, int nb, int modified, int diag_only) {
  const int parts = band_parts(na_tot);
  for (int i = 0; i < parts; ++i) {
    PgKind& k = ks.k[ks.n++];
    k.out = out;
    k.ps = ps;
    k.as = as;
    k.bs = bs;
    k.ia = i * na_tot / parts;
    k.na = (i + 1) * na_tot / parts - k.ia;
    k.a0 = a0 + k.ia;
    k.ib = ib;
    k.nb = nb;
    k.modified = modified;
    k.diag_only = diag_only;
  }
}

// G per task (4 or 2) and blocks per 64 columns (grid.z).  A block's time, in units of one
// G's pass over K: its rounds of one task per wavefront, each as long as its G and 0.7,
// and 0.6 + 100 / N_K for its start and the rows it stages.  One block per compute unit;
// beyond 256 of them they queue.  So few blocks (small meshes) are split until every
// wavefront has one short task, a number a little above 256 so that no unit is left with a
// whole block more than the others, and large meshes take long tasks, whose stores are
// wider.  us of 4 G and one block per 64 columns against the choice (k-points, bands, N_G,
// N_K): 1, 4 + 4, 59, 59: 74 / 21 (2 G, 6 blocks); 27, 2 + 2, 51, 89: 77 / 24 (2 G, 5);
// 27, 3 + 4, 27, 27: 24.8 / 15.3 (2 G, 3); 64, 3 + 4, 113, 113: 403 / 314 (4 G, 2); 64,
// 3 + 4, 113, 169: 707 / 531 (4 G, 2); 125, 4 + 5, 59, 113: 739 with 4 G and one block, 837
// with two.  (Two G as a kernel of their own: half the code and no spilled registers,
// 20.0 -> 15.3 us at the third against a bound on G in the other.)
void pair_split(const PgKinds& ks, int nk, int ng, int nkb, int& nq, int& split) {
  const int nch = (nkb + PG_ROWS - 1) / PG_ROWS;
  double blocks = 0.0;  // of 64 columns, over the rows of k-points
  int most = 0, off_diag = 0;  // kinds of a block with diagonal pairs, of the others
  for (int i = 0; i < ks.nsides; ++i) {
    const PgSide& sd = ks.side[i];
    blocks += sd.nb * (double)nk * (nk + 1) / 128.0 + 0.5 * nk;
    most = std::max(most, sd.count);
    off_diag = std::max(off_diag, sd.count - sd.diag);
  }
  double best = 0.0;
  nq = PG_BATCH;
  split = 1;
  for (int q = PG_BATCH; q >= 2; q /= 2) {
    const int ngb = (ng + q - 1) / q;
    const int zmax = std::min(cdiv(nch > 1 ? ngb : most * ngb, PG_WAVES), 16);
    for (int z = 1; z <= zmax; ++z) {
      const int kinds = blocks * z <= 256.0 ? most : off_diag;
      const double t = nch > 1 ? kinds * cdiv(ngb, PG_WAVES * z) * (q + 0.7 + 0.6 * nch)
                               : cdiv(kinds * ngb, PG_WAVES * z) * (q + 0.7) + 0.6 + 100.0 / nkb;
      const double cost = t * std::max(1.0, blocks * z / 256.0 + 0.25);
      if (best == 0.0 || cost < 0.98 * best) {
        best = cost;
        nq = q;
        split = z;
      }
    }
  }
}

}  // namespace

extern "C" {

bse_status bse_pair_elements(const bse_orb_desc* d, const void* C, const int32_t* kpg,
                             const int32_t* mkg, void* Mcv, void* Mvv, void* Mcc, void* Ncv,
                             void* Nvc, hipStream_t stream) {
  launch_failure_reset();
  if (!d || d->nk <= 0 || d->nv <= 0 || d->nc <= 0 || d->ng <= 0 || d->nkb <= 0) return BSE_ERR_ARG;
  if (d->nk > 46340) return BSE_ERR_ARG;
  const bool full = d->coupling == BSE_FULL;
  if (d->coupling != BSE_FULL && d->coupling != BSE_TDA) return BSE_ERR_ARG;
  if (!C || !kpg || !Mcv || !Mvv || !Mcc) return BSE_ERR_ARG;
  if (full && (!mkg || !Ncv || !Nvc)) return BSE_ERR_ARG;
  const int nv = d->nv, nc = d->nc, ng = d->ng, nkb = d->nkb, nbt = nv + nc;
  // The limits of the interface, which are narrower than the kernel's own (any number of K,
  // in parts of PG_ROWS, while a k-point's offsets fit in 32 bits; PG_MAXKINDS pieces of
  // five bands): 160 KB for the coefficients of two k-points, 24 blocks of 4 x 4 bands.
  // They bound the kinds and offsets here too.
  if ((size_t)2 * nbt * nkb * sizeof(double2) > PG_LDS) return BSE_ERR_ARG;
  const int64_t v4 = (nv + 3) / 4, c4 = (nc + 3) / 4;
  if (v4 * v4 + c4 * c4 + (full ? 3 : 1) * v4 * c4 > PG_MAXKINDS) return BSE_ERR_ARG;
  PgKinds ks{};
  const int64_t G = ng;
  int nbmax = 0;
  for (int c = 0; c < 2; ++c) {  // bands at k' among the occupied, the unoccupied
    const int n = c ? nc : nv, parts = band_parts(n);
    for (int i = 0; i < parts; ++i) {
      PgSide& sd = ks.side[ks.nsides++];
      const int ib = i * n / parts;
      sd.b0 = (c ? nv : 0) + ib;
      sd.nb = (i + 1) * n / parts - ib;
      sd.first = ks.n;
      nbmax = std::max(nbmax, sd.nb);
      if (c) {
        add_kinds(ks, (double2*)Mcc, nc * nc * G, nc * G, G, nv, nc, ib, sd.nb, 0, 0);
        if (full) add_kinds(ks, (double2*)Nvc, nv * nc * G, nc * G, G, 0, nv, ib, sd.nb, 1, 0);
        const int before = ks.n;
        add_kinds(ks, (double2*)Mcv, nv * nc * G, nc * G, G, 0, nv, ib, sd.nb, 0, 1);
        sd.diag = ks.n - before;
      } else {
        add_kinds(ks, (double2*)Mvv, nv * nv * G, nv * G, G, 0, nv, ib, sd.nb, 0, 0);
        if (full) add_kinds(ks, (double2*)Ncv, nc * nv * G, nv * G, G, nv, nc, ib, sd.nb, 1, 0);
      }
      sd.count = ks.n - sd.first;
    }
  }
  const size_t lds = ((size_t)std::min(nkb, PG_ROWS) * 64 + PG_TR * PG_WAVES) * sizeof(double2);
  const int64_t groups = (int64_t)((d->nk + 1) / 2) * row_groups(d->nk, nbmax);
  int nq, split;
  pair_split(ks, d->nk, ng, nkb, nq, split);
  // (the parameter has the kernel's name, under which the launch is timed)
  auto launch = [&](auto* k_pair_elements) {
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute((const void*)k_pair_elements, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds) != hipSuccess)
      return false;
    BSE_LAUNCH(k_pair_elements, dim3((unsigned)groups, (unsigned)ks.nsides, (unsigned)split),
               dim3(PG_THREADS), lds, stream, (const double2*)C, d->nk, nbt, nkb, ng, kpg,
               full ? mkg : kpg, ks);
    return true;
  };
  if (!(nq == 4 ? launch(k_pair_elements<4>) : launch(k_pair_elements<2>))) return BSE_ERR_HIP;
  return hipGetLastError() == hipSuccess ? BSE_OK : BSE_ERR_HIP;
}

}  // extern "C"
