// The temperature of a LOGITS call as exp_of_logit (spec_accept.hip) takes it; host code only.
#pragma once
#include <cfloat>
#include <cmath>

namespace fsr {

struct TempScale {
    double c, c_hi, c_lo;  // 256 / (T ln2); the same in two parts
    float reach;           // largest magnitude of a logit that is taken as it is; -1: none is
};
// |z / T| up to 600, where the value and 2^32 times it are normal numbers.  A masked logit counts as one of -600, so the
// reach has to be that of the temperature: outside the normal range of a float (T below 2e-41 or above 5.6e35) there is none,
// and the statistics take a reference off first.
constexpr double kReach = 600.0;
inline TempScale temp_scale(double T) {
    const double reach = kReach * T;
    if (!(reach >= (double)FLT_MIN && reach <= (double)FLT_MAX)) return TempScale{0.0, 0.0, 0.0, -1.0f};
    TempScale t{};
    const long double c = 256.0L / (0.693147180559945309417232121458L * (long double)T);
    t.c = (double)c;
    int e = 0;
    const double m = std::frexp(t.c, &e);
    t.c_hi = std::ldexp(std::floor(std::ldexp(m, 29)), e - 29);
    t.c_lo = (double)(c - (long double)t.c_hi);
    t.reach = (float)reach;
    return t;
}

}  // namespace fsr
