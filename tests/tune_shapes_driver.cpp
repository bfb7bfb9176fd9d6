// The tuner's candidates (lbm_shape.h) on lattices of every size class: each one
// holds a row and fits LDS, none is there twice, and the shape a context starts
// with, any shape of its own and the rule's z-chunk for each block are among them
// (z-chunks of two planes and more).  Returns 1 at the first lattice that fails.
#include <cstdio>
#include <initializer_list>

#include "lbm_shape.h"

int main() {
    using namespace lbm;
    const int sizes[][3] = {{2, 3, 2},     {16, 16, 32},    {24, 24, 48},     {91, 21, 266},  {64, 64, 256}, {60, 60, 900},
                            {48, 48, 192}, {192, 192, 1024}, {256, 30, 12},   {150, 64, 64},  {50, 46, 130}, {33, 20, 40},
                            {128, 128, 128}, {12, 150, 700}, {250, 64, 40},   {18, 18, 362}};
    int other = 0;  // lattices whose default is no power of two
    for (const auto &s : sizes)
        for (const int prec : {LBM_FP64, LBM_FP32, LBM_FP16})
            for (const bool tau1 : {false, true})
                for (const int copies : {1, 7}) {
                    std::vector<lbm_params> p(copies);
                    std::vector<int> prim(copies);
                    for (int r = 0; r < copies; r++) {
                        p[r] = lbm_params{};
                        p[r].nx = s[0]; p[r].ny = s[1]; p[r].nz = s[2];
                        prim[r] = r;
                    }
                    const ShapeInput in = {p.data(), prim.data(), copies, prec, s[0], tau1};
                    const LaunchShape start = default_shape(in), own = {256, 7};
                    const auto list = tune_shapes(in, start), more = tune_shapes(in, own);
                    auto has = [](const std::vector<LaunchShape> &l, LaunchShape a) {
                        int n = 0;
                        for (const LaunchShape &b : l) n += a.block == b.block && a.cz == b.cz;
                        return n == 1;
                    };
                    bool ok = (start.cz < 2 || has(list, start)) && has(more, own);
                    for (const LaunchShape &a : list)
                        ok = ok && has(list, a) && a.block >= s[0] && a.cz >= 2 && main_lds_bytes(in, a.block) <= MAIN_LDS_MAX;
                    for (int block = 256; block <= 1024; block *= 2) {
                        if (main_lds_bytes(in, block) > MAIN_LDS_MAX) continue;
                        const int cz = auto_zchunk(in, block);
                        ok = ok && (cz < 2 || has(list, {block, cz}));
                        for (const int z : {2, 4, 8, 16, 32}) ok = ok && has(list, {block, z});
                    }
                    if (!ok) {
                        std::printf("%d x %d x %d, precision %d, tau1 %d, %d replicas\n", s[0], s[1], s[2], prec, tau1, copies);
                        return 1;
                    }
                    other += start.cz & (start.cz - 1) ? 1 : 0;
                }
    std::printf("%d defaults are no power of two\n", other);
    return other ? 0 : 1;
}
