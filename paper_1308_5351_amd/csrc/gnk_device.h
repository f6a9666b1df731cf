// Device helpers shared by the pair kernels (Cauchy sums of the operators and
// of the geometric derivatives).
#pragma once

#include <hip/hip_runtime.h>

namespace gnk {

// Pointers into global memory. In the device pass they carry address space 1,
// so wave-uniform loads through them compile to scalar loads (a generic
// pointer read from a table in memory would give per-lane flat loads). The
// host pass only parses kernel bodies and keeps plain pointers.
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
using gptr = __attribute__((address_space(1))) T*;
#else
template <class T>
using gptr = T*;
#endif

// v_rcp_f64 is accurate to about 2^-24 on gfx950; one Newton step brings the
// reciprocal to about 2^-48 (a few ulp), below the rounding of the sums.
__device__ __forceinline__ double refine_rcp(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = __builtin_fma(-d, r, 1.0);
  return __builtin_fma(r, e, r);
}

// bounding circle {cx, cy, r, 0} of pts[i0, i1) by one wavefront: the centre of the
// bounding box, the radius widened by a relative margin so that rounding of the centre
// cannot hide a point
__device__ __forceinline__ double4 wave_circle(const double2* pts, int i0, int i1) {
  const int lane = threadIdx.x & 63;
  double xmin = 1e300, xmax = -1e300, ymin = 1e300, ymax = -1e300;
  for (int i = i0 + lane; i < i1; i += 64) {
    const double2 e = pts[i];
    xmin = fmin(xmin, e.x); xmax = fmax(xmax, e.x);
    ymin = fmin(ymin, e.y); ymax = fmax(ymax, e.y);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    xmin = fmin(xmin, __shfl_xor(xmin, off, 64));
    xmax = fmax(xmax, __shfl_xor(xmax, off, 64));
    ymin = fmin(ymin, __shfl_xor(ymin, off, 64));
    ymax = fmax(ymax, __shfl_xor(ymax, off, 64));
  }
  const double cx = 0.5 * (xmin + xmax), cy = 0.5 * (ymin + ymax);
  double r = 0.0;
  for (int i = i0 + lane; i < i1; i += 64) {
    const double2 e = pts[i];
    r = fmax(r, sqrt((e.x - cx) * (e.x - cx) + (e.y - cy) * (e.y - cy)));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) r = fmax(r, __shfl_xor(r, off, 64));
  return make_double4(cx, cy, r * (1.0 + 1e-12) + 1e-300, 0.0);
}

}  // namespace gnk
