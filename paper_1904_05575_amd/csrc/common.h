// Shared device helpers of the BSE library (gfx950 / CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef double d4 __attribute__((ext_vector_type(4)));

#define BSE_DEV __device__ __forceinline__

struct cplx {
  double re, im;
};

BSE_DEV double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
BSE_DEV double2 cmulc(double2 a, double2 b) {  // conj(a) * b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
BSE_DEV double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
BSE_DEV double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
BSE_DEV double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
BSE_DEV double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
BSE_DEV double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }

// acc + a b and acc + conj(a) b in four fused operations each
BSE_DEV double2 cfma(double2 a, double2 b, double2 acc) {
  return make_double2(fma(-a.y, b.y, fma(a.x, b.x, acc.x)), fma(a.y, b.x, fma(a.x, b.y, acc.y)));
}
BSE_DEV double2 cfmac(double2 a, double2 b, double2 acc) {
  return make_double2(fma(a.y, b.y, fma(a.x, b.x, acc.x)), fma(-a.y, b.x, fma(a.x, b.y, acc.y)));
}
BSE_DEV double2 cneg(double2 a) { return make_double2(-a.x, -a.y); }

// 1/x and 1/sqrt(x) for positive normal x: the hardware estimate with Newton
// steps (short dependent chains).  Largest relative errors over 2^20 values in 2^-300 ..
// 2^300: 1.1e-16 and 1.4e-16.
BSE_DEV double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}
BSE_DEV double fast_rsq(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  r = fma(r, fma(-h * r, r, 0.5), r);
  return fma(r, fma(-h * r, r, 0.5), r);
}

// What a wavefront wrote to LDS before is there for its own reads after.
BSE_DEV void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int CTRL>
BSE_DEV double dpp_mov(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// Sum over the 16 lanes of each row; every lane of the row gets it.
BSE_DEV double row_sum(double v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  v += dpp_mov<0x140>(v);  // row_mirror
  return v;
}
BSE_DEV double2 row_sum(double2 v) { return make_double2(row_sum(v.x), row_sum(v.y)); }

// 64-lane wavefront sum (deterministic butterfly order).
BSE_DEV double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
BSE_DEV double2 wave_sum2(double2 v) {
  return make_double2(wave_sum(v.x), wave_sum(v.y));
}

// Block-wide sum of one double; every thread gets the result.  `sh` needs
// blockDim.x / 64 doubles of shared memory.  Deterministic.
BSE_DEV double block_sum(double v, double* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < nw; ++i) s += sh[i];
  return s;
}

// Device status word shared by every kernel of one call sequence: kernels
// return at entry when an earlier kernel recorded a failure.
BSE_DEV bool failed(const int32_t* info) { return info != nullptr && *(volatile const int32_t*)info != 0; }

// Record the first failure (0 -> code); later failures keep the first code.
BSE_DEV void set_info(int32_t* info, int32_t code) {
  if (info) atomicCAS(info, 0, code);
}

__host__ __device__ static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
