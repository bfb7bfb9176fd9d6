// Launch shape of the main kernel (block threads and z-chunk length): LDS need,
// the default by an estimate of the kernel's cost, and the tuner's candidates.
// Host arithmetic only.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <vector>

#include "lbm.h"

namespace lbm {

constexpr int MAIN_BLOCK_MIN = 256, MAIN_BLOCK_MAX = 1024;
constexpr size_t MAIN_LDS_MAX = 64 * 1024;

struct LaunchShape {
    int block, cz;
};

// the entries of a context (prim: the first entry of each one's fluid)
struct ShapeInput {
    const lbm_params *p;
    const int *prim;
    int n, prec, maxnx;
    bool tau1;  // every relaxation time is 1
};

// rows of one main-kernel tile of replica q
inline int tile_rows(const lbm_params &q, int block) { return std::max(1, std::min(q.ny, block / q.nx)); }

// LDS of the main kernel: a 4-plane ring of both components' densities over the
// tile rows plus a one-row halo on each side
inline size_t main_lds_bytes(const ShapeInput &in, int block) {
    size_t elems = 0;
    for (int r = 0; r < in.n; r++)
        elems = std::max(elems, (size_t)8 * (tile_rows(in.p[r], block) + 2) * in.p[r].nx);
    return elems * (in.prec == LBM_FP64 ? 8 : 4);
}

// Cost of one main-kernel launch at a block and z-chunk cz: the root
// of the squares of two times, in planes that one wave collides.
//  - Work of a compute unit: each of its workgroups collides cz planes and fills
//    cz + 2, a fill costing half a collision, its two halo rows included; partly
//    filled tiles cost what full ones do.  While all workgroups are resident
//    the busiest unit holds a whole number of them; after that, 0.55 of what the
//    last round leaves idle is lost.  Resident are taken to be four waves per SIMD,
//    two in FP64, as the fit was made; by their registers FP64 with every relaxation
//    time 1 (140 and 165) and FP16 general relaxation with noise (136) run at three.
//  - Latency: a wave alone takes 2.4 times as long per plane as a SIMD's share.
// Blocks of 512 and 1024 wait for more waves at every plane: 1.08 and 1.23.
// Fitted to the main kernel's times at every shape on 29 lattices of 8 k to 38 M
// nodes (all storages, both relaxations, single and batched): the shape it picks
// takes 1.9% more than the best one in the mean and 11% at most.  A cost of total
// work and waves alone, with z-chunks of powers of two, took 9.8% and 48% (91 x 21
// x 266: 1024 x 2, 266 workgroups for 256 units, 82.7 us; 512 x 3 54.4), and the
// longest z-chunk up to 16 that keeps four waves per SIMD at 256 threads 54% at
// most (16 x 16 x 32: 24.6 us at z-chunk 2, 18.2 at 1; 192 x 192 x 1024 FP16: 2346
// us at 256 threads, 1912 at 1024 x 32).
inline double shape_cost(const ShapeInput &in, int block, int cz) {
    double work = 0.0, n = 0.0;
    int longest = 0;
    for (int r = 0; r < in.n; r++) {
        if (in.prim[r] != r) continue;
        const lbm_params &q = in.p[r];
        const int ty = tile_rows(q, block), z = std::min(cz, q.nz);
        const double tiles = (double)((q.ny + ty - 1) / ty) * ((q.nz + z - 1) / z);
        work += tiles * (z + 0.5 * (z + 2) * (1.0 + 2.0 * q.nx / block));
        n += tiles;
        longest = std::max(longest, z);
    }
    const int waves = block / 64;
    const double resident = std::max(1, 4 * (in.prec == LBM_FP64 ? 2 : 4) / waves);
    const double m = n / 256.0, rounds = std::ceil(m / resident);
    const double share = std::ceil(m) <= resident ? std::ceil(m) : m + 0.55 * (rounds * resident - m);
    const double busy = work / n * share * waves / 4.0 * (block == 256 ? 1.0 : block == 512 ? 1.08 : 1.23);
    const double wait = 2.4 * (longest + 0.5 * (longest + 2)) * std::max(1.0, m / resident);
    return std::sqrt(busy * busy + wait * wait);
}

// z-chunk of least cost at a block
inline int auto_zchunk(const ShapeInput &in, int block, double *cost = nullptr) {
    int best = 1;
    double least = 0.0;
    for (const int cz : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32}) {
        const double v = shape_cost(in, block, cz);
        if (cz == 1 || v < least) {
            best = cz;
            least = v;
        }
    }
    if (cost) *cost = least;
    return best;
}

// block and z-chunk of least cost.  1024 threads, which leave 128 VGPRs, are taken
// with FP32 arithmetic and every relaxation time 1 only.  FP64 spills 12 to 141
// registers there.  General relaxation fits in FP32 (no spill) and gains nothing:
// best at 512 and at 1024 threads 107.3 and 106.7 us on 64 x 64 x 256, 152.6 and
// 157.8 on 150 x 64 x 128, 814 and 832 on 192 x 192 x 256.  In FP16 it spills two or
// three with noise, none without, and is faster on most lattices (102 and 92, 146
// and 127, 1017 and 732), which tuning finds; the cost above was not fitted to it.
inline LaunchShape default_shape(const ShapeInput &in) {
    LaunchShape best = {MAIN_BLOCK_MIN, 1};
    double least = -1.0;
    for (int block = MAIN_BLOCK_MIN; block <= MAIN_BLOCK_MAX; block *= 2) {
        if (block == 1024 && (in.prec == LBM_FP64 || !in.tau1)) continue;
        if (main_lds_bytes(in, block) > MAIN_LDS_MAX) continue;
        double v;
        const int cz = auto_zchunk(in, block, &v);
        if (least < 0.0 || v < least) {
            least = v;
            best = {block, cz};
        }
    }
    return best;
}

// Shapes the tuner times, each one admissible: every block with z-chunks 2, 4, ...,
// 32 and the rule's own z-chunk for it, and the shape the context has, so that
// tuning does not leave a slower one.  Z-chunks of one plane are outside the tuner's
// range (2 and more): a lattice small enough to start with one is better left
// untuned.
inline std::vector<LaunchShape> tune_shapes(const ShapeInput &in, LaunchShape present) {
    std::vector<LaunchShape> out;
    auto add = [&](int block, int cz) {
        if (cz < 2) return;
        for (const LaunchShape &s : out)
            if (s.block == block && s.cz == cz) return;
        out.push_back({block, cz});
    };
    for (int block = MAIN_BLOCK_MIN; block <= MAIN_BLOCK_MAX; block *= 2) {
        if (block < in.maxnx || main_lds_bytes(in, block) > MAIN_LDS_MAX) continue;
        for (const int cz : {2, 4, 8, 16, 32}) add(block, cz);
        add(block, auto_zchunk(in, block));
        if (block == present.block) add(block, present.cz);
    }
    return out;
}

}  // namespace lbm
