// Host run of the sphere-box coordinates (lbm_kernels_impl.h): for origins over
// the whole int32 range, every wall mask and boxes as long as the lattice down to
// the smallest, every node that box_node accepts lies inside the lattice, on
// the coordinate that a 64-bit remainder gives, and every such node of a box that
// starts within one period of the lattice is accepted.  Prints the number of nodes
// checked; returns 1 at the first one that does not.
#include <climits>
#include <cstdio>

#include "lbm_kernels_impl.h"

int main() {
    using namespace lbm;
    const int sizes[][4] = {{16, 16, 24, 12}, {12, 13, 14, 12}, {64, 64, 256, 22}, {256, 10, 2000000, 10}};
    const int far[] = {0, -3, 5, 43, -100, 626, -540, 1000, 123457, -123458, (1 << 28) - 2, -(1 << 28) - 2,
                       INT_MAX - 2, INT_MAX, INT_MIN, INT_MIN + 1};
    long checked = 0;
    for (const auto &s : sizes)
        for (unsigned walls = 0; walls < 8; walls++)
            for (int ax = 0; ax < 3; ax++)
                for (const int f : far) {
                    Geo g;
                    g.nx = s[0]; g.ny = s[1]; g.nz = s[2];
                    g.wx = walls & 1u; g.wy = walls & 2u; g.wz = walls & 4u;
                    g.N = (int64_t)g.nx * g.ny * g.nz;
                    const int S = s[3], n3[3] = {g.nx, g.ny, g.nz};
                    int32_t org[3] = {1, -2, 3};
                    org[ax] = f;
                    for (int b = 0; b < S * S * S; b++) {
                        int bb[3], p[3];
                        const bool in = box_node(b, org, S, g, bb, p);
                        for (int a = 0; a < 3; a++) {
                            const bool wall = walls & (1u << a);
                            const int64_t raw = (int64_t)org[a] + bb[a];
                            const int64_t want = wall ? raw : (raw % n3[a] + n3[a]) % n3[a];
                            const bool lies = want >= 0 && want < n3[a];
                            if (in && (p[a] != want || !lies)) {
                                std::printf("origin %d axis %d walls %u node %d: %d for %lld of %d\n", f, ax, walls, b,
                                            p[a], (long long)want, n3[a]);
                                return 1;
                            }
                            checked++;
                        }
                        bool all = true;
                        for (int a = 0; a < 3; a++) {
                            const int64_t raw = (int64_t)org[a] + bb[a];
                            const bool wall = walls & (1u << a);
                            if (raw < (wall ? 0 : -n3[a]) || raw >= (wall ? n3[a] : 2 * n3[a])) all = false;
                        }
                        if (in != all) {
                            std::printf("origin %d axis %d walls %u node %d: in %d\n", f, ax, walls, b, (int)in);
                            return 1;
                        }
                    }
                }
    // where a box starts: two nodes before the sphere, at any position a diverging
    // sphere reaches
    const double at[] = {0.0, 7.9, -3.5, 1e6, -1e9, 1e300, -1e300};
    for (const double x : at) {
        const int32_t o = box_start(x);
        const double want = __builtin_floor(x) - 2.0;
        if (want >= -0x1p28 && want <= 0x1p28 ? o != (int32_t)want : (o < -(1 << 28) - 2 || o > (1 << 28))) {
            std::printf("start of %g: %d\n", x, o);
            return 1;
        }
    }
    std::printf("%ld coordinates\n", checked);
    return 0;
}
