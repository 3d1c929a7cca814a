// The few device names that csrc/dd.h uses, for a host compiler.
#pragma once
#include <cmath>
using std::fabs;
using std::fma;
using std::fmax;
using std::ilogb;
using std::ldexp;
#define __device__
#define __forceinline__ inline
struct double2 {
  double x, y;
};
inline double2 make_double2(double x, double y) { return double2{x, y}; }
// about as accurate as the hardware's approximation
inline double host_rcp(double x) { return (double)(1.0f / (float)x); }
#define __builtin_amdgcn_rcp host_rcp
