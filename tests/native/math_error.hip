// Errors of sph_math.hpp's functions in units in the last place, from
// approximations off by a stated relative error: compiled for the host only.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <random>

#include "sph_math.hpp"

namespace {
// |got - want| in units of the last place of the exact value
double ulps(double got, long double want) {
    int e;
    frexpl(want, &e);
    return (double)(fabsl((long double)got - want) / ldexpl(1.0L, e - 53));
}
}  // namespace

// worst[0..2]: reciprocal, reciprocal square root, square root over n random
// arguments in 2^lo .. 2^hi, their approximations off by up to 2^-bits.
extern "C" void math_error(int64_t n, uint64_t seed, int lo, int hi, int bits, double* worst) {
    std::mt19937_64 rng(seed);
    std::uniform_real_distribution<double> ex(lo, hi), off(-1.0, 1.0);
    worst[0] = worst[1] = worst[2] = 0.0;
    for (int64_t i = 0; i < n; ++i) {
        const double x = exp2(ex(rng));
        const double d = 1.0 + ldexp(off(rng), -bits);
        const long double r = 1.0L / (long double)x, s = sqrtl((long double)x), q = 1.0L / s;
        const double y = (double)(r * d), z = (double)(q * d);
        const double e[3] = {ulps(sph::rcp_from(x, y), r), ulps(sph::rsqrt_from(x, z), q),
                             ulps(sph::sqrt_from(x, z), s)};
        for (int k = 0; k < 3; ++k) worst[k] = e[k] > worst[k] ? e[k] : worst[k];
    }
}
