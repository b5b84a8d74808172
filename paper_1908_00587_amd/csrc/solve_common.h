// Small device helpers shared by the radial-solve kernels.
#pragma once
#include "nsc_internal.h"

namespace nsc {

// Entries of the one-sided wall rows past the band, packed by distance from
// the wall: row t holds 4 - t of them (U right of the band in rows 0..3, L
// left of it in rows N-1-t).
__device__ __forceinline__ int edge_off(int t) { return t * 4 - (t * (t - 1)) / 2; }

// 16-byte load and store unit; arrays of it stay in registers (arrays of
// HIP's double2 do not)
typedef double Dbl2 __attribute__((ext_vector_type(2)));

struct Cd {
  double x, y;
};
__device__ __forceinline__ Cd operator+(Cd a, Cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ Cd operator-(Cd a, Cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ Cd operator*(double s, Cd a) { return {s * a.x, s * a.y}; }
__device__ __forceinline__ Cd ci(Cd a) { return {-a.y, a.x}; }  // i * a
__device__ __forceinline__ Cd ld(const double2 *p) {
  double2 v = *p;
  return {v.x, v.y};
}
__device__ __forceinline__ void st(double2 *p, Cd v) { *p = make_double2(v.x, v.y); }
__device__ __forceinline__ Cd fmac(double w, Cd v, Cd acc) { return {fma(w, v.x, acc.x), fma(w, v.y, acc.y)}; }

}  // namespace nsc
