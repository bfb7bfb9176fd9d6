// Host run of relax_component (lbm_math.h), built without contraction: one mode
// and its normal at a time, the post-collision populations are the mode's share
// with the noise product fused and the relaxed mode rounded before it.  Returns 1
// at the first population that differs.
#include <cmath>
#include <cstdio>

#include "lbm_math.h"

template <typename T>
int check(const char *name) {
    using namespace lbm;
    Coef<T> c = make_coef<T>(0.95, 0.05, 0.8, 1.1, 0.9, 1.3, 1e-4, 1);
    // population that shows mode k alone, and its factor
    const int where[Q] = {0, 0, 0, 0, 0, 1, 3, 7, 15, 11, 1, 3, 5, 7, 7, 11, 0, 1, 3};
    const int times[Q] = {0, 0, 0, 0, -1, 2, 1, 1, 1, 1, -2, -2, -2, 1, -1, 1, 1, -2, -1};
    uint32_t seed = 12345u;
    auto rnd = [&] {
        seed = seed * 1664525u + 1013904223u;
        return T((double)(int32_t)seed / 2147483648.0);
    };
    for (int n = 0; n < 200; n++)
        for (int k = 4; k < Q; k++) {
            T m[Q], zl[16], out[Q];
            for (T &v : m) v = T(0);
            for (T &v : zl) v = T(0);
            m[k] = T(0.01) * rnd();
            zl[k - 4] = T(3) * rnd();
            const T zero[3] = {T(0), T(0), T(0)}, rd = T(0.05) * rnd();
            T base[Q], m0[Q], z0[16];
            for (T &v : m0) v = T(0);
            for (T &v : z0) v = T(0);
            // rho0l = -rd + r: the density deviation is zero, so only mode k is there
            const T r = c.rho0[0] + rd;
            relax_component<T>(r, T(1), T(0), zero, m, zero, zero, zero, zl, c, out);
            relax_component<T>(r, T(1), T(0), zero, m0, zero, zero, zero, z0, c, base);
            const T sq = std::sqrt(r), amp = (k == 4 ? c.nb : k < 10 ? c.ns : c.ng) * sq;
            const T g = k == 4 ? c.gb : c.gs;
            const T relaxed = k < 10 ? T(inv_norm(k)) * (g * m[k]) : T(inv_norm(k)) * c.gg * m[k];
            const T a = std::fma(T(inv_norm(k) * sqrt_norm(k)) * amp, zl[k - 4], relaxed);
            const T w = T(wgt(where[k])), want = w * (T(times[k]) * a);
            if (base[where[k]] != T(0) || out[where[k]] != want) {
                std::printf("%s mode %d: %.17g for %.17g\n", name, k, (double)out[where[k]], (double)want);
                return 1;
            }
        }
    return 0;
}

int main() { return check<float>("float") || check<double>("double"); }
