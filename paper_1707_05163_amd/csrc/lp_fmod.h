// lp_fmod.h -- the floating-point remainder that brackets stage times (host code).
#pragma once

#include <cmath>

// fmod(a, P) for P > 0 (infinity too), bit for bit: where |a / P| < 2^51 the remainder
// a - n P with n = trunc(a / P), corrected by at most one, is exact in one fused
// multiply-add.  (The library's fmod divides bit by bit: 50 to 100 ns for each of a run's
// stage times.)
inline double exact_fmod(double a, double P)
{
    if (std::fabs(a) < P)
        return a;
    const double n = std::trunc(a / P);
    if (!(std::fabs(n) < 0x1p51))
        return std::fmod(a, P);
    double r = std::fma(-n, P, a);
    if (a >= 0.0) {
        if (r < 0.0)
            r = std::fma(-(n - 1.0), P, a);
        else if (r >= P)
            r = std::fma(-(n + 1.0), P, a);
    } else {
        if (r > 0.0)
            r = std::fma(-(n + 1.0), P, a);
        else if (r <= -P)
            r = std::fma(-(n - 1.0), P, a);
    }
    return r == 0.0 ? std::copysign(r, a) : r;  // zero has the sign of the dividend
}
