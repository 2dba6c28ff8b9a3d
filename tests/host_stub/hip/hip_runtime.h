// Stand-in for the HIP runtime header: lets a host compiler take the device
// headers of the force terms (csrc/bhq_terms.h, bhq_split.h).
#pragma once

#include <cmath>

#define __device__
#define __forceinline__ inline

using std::fma;

inline float __builtin_amdgcn_rsqf(float v) { return 1.0f / std::sqrt(v); }
inline double __builtin_amdgcn_rsq(double v) { return 1.0 / std::sqrt(v); }
inline float __builtin_amdgcn_fractf(float v) { return v - std::floor(v); }
