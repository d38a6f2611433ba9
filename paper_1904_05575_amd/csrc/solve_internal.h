// Internal interface between the eigensolver's translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int TRD_NB = 32;  // Householder panel width

// Small shared state of the tridiagonalisation kernels (complex slots):
//   [0] scal = 1/(alpha_x - beta) of the current reflector, [1] tau,
//   [2] S[b0][b0], the first diagonal element of the trailing matrix the
//       current reflector multiplies (b0 = c + 1),
//   [4, 4 + TRD_NB) V^H v and [4 + TRD_NB, 4 + 2 TRD_NB) W^H v over the panel
constexpr int HS_SCAL = 0, HS_TAU = 1, HS_S00 = 2, HS_SVV = 4, HS_SWV = 4 + TRD_NB,
              HS_SIZE = 4 + 2 * TRD_NB;

struct TrdBufs {
  double2* VW;      // n x 2*TRD_NB, [V | W] of the current panel (column-major, ld n)
  double2* WV;      // n x 2*TRD_NB, [W | V]
  double2* ybuf;    // n (unused by the lower-triangle sweep)
  double2* hs;      // HS_SIZE
  double2* part;    // trd_part_elems(n)
  double* dd;       // n   diagonal of T
  double* ee;       // n-1 off-diagonal of T
  double2* tau;     // n-1 reflector scalars
};

int64_t trd_part_elems(int64_t n);
bool tridiagonalise(double2* M, int64_t n, int64_t ld, const TrdBufs& w, int32_t* info,
                    hipStream_t s);

// Two-stage reduction (band.hip): dense to a band of half width BAND_W, then to
// tridiagonal form.  For solves that form no eigenvectors.
constexpr int BAND_W = 16;
constexpr int BAND_BATCH_MAX = 16;  // problems per launch
constexpr int CHASE_SWEEPS = 4;  // sweeps per block of the second stage

struct BandBufs {
  double2* VW;      // n x 4 BAND_W
  double2* q1x;     // n x 2 BAND_W
  double2* part;    // band_part_bytes(n)
  double2* big;     // band_big_bytes(n)
  double* dd;       // n   diagonal of T
  double* ee;       // n-1 off-diagonal of T
  double2* yproj;   // optional: vector y, replaced by Q^H y
};
struct BandItem {
  double2* M;
  int64_t n, ld;
  BandBufs b;
  int32_t* info;
};
int64_t band_big_bytes(int64_t n);
int64_t band_part_bytes(int64_t n);
// Every problem's matrix (lower triangle) to tridiagonal form, in groups of up
// to BAND_BATCH_MAX problems per launch; each problem's values do not depend on
// what else is in the batch.
bool tridiagonalise_band(const BandItem* it, int np, hipStream_t s);
