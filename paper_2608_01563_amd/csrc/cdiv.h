// cdiv.h -- rounding-up division (host).
#pragma once

namespace mg {

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

}  // namespace mg
