// Included ahead of the host checks by tests/test_forms_nan.py: the maxima they fold their deviations
// with keep a NaN operand, which std::fmax drops and std::max drops on its right.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <limits>
#include <random>
#include <vector>

namespace std {
inline double sticky_max(double a, double b) { return a != a ? a : (b != b ? b : (a < b ? b : a)); }
}  // namespace std

#define fmax sticky_max
#define max sticky_max
