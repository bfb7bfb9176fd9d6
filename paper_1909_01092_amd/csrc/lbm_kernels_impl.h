// HIP kernels (gfx950) of the fluctuating two-component D3Q19 step with one
// finite-size sphere per replica.  Instantiated once per storage precision
// by lbm_k_f64.hip / lbm_k_f32.hip / lbm_k_f16.hip.
//
// Paper: Xue, Biferale, Sbragaglia, Toschi, "A lattice Boltzmann study of
// particle settling in a fluctuating multicomponent fluid under
// confinement".  Sec. 2: eq. (density), eq. (lbe), MRT paragraph,
// eq. (sc-force), noise paragraph, particle paragraph (particle nodes,
// leap-frog Newton, moving bounce-back with momentum exchange,
// cover/uncover, mass correction, virtual wetting layer).  Sec. 3: eq. (fp).
//
// Storage.  Each replica keeps its populations on a lattice with one ghost row
// per y side and one ghost plane per z side, laid out
// [z+1][y+1][slot][x]: the 38 slots (component and direction) of an x-row lie
// next to each other, rows follow without padding.  Node x pulls population i of step
// n from position x - c_i, slot i, x wrapped around the row; a node whose
// x - c_i lies beyond an x-wall pulls slot opp(i) of itself (half-way
// bounce-back).  Whoever produces a value that does not arrive that way writes
// it into exactly the slot it is pulled from: a node next to a y- or z-wall
// writes its bounced value into the ghost, a node next to a periodic y- or
// z-face writes the wrapped copy into the ghost, the link kernel writes the
// sphere's moving-wall bounce-back into the particle node's slot, and uncovered
// nodes get f_eq written into the slots they pull from.
// Why this order: a wave reads and writes 76 streams.  With one array per
// direction these are 76 distant pages and, with ghost columns, rows that
// start inside a cache line which two rows share.  Slots side by side make
// every line of a tile's rows whole and put the streams of a row into a few
// pages: 38 loads and 38 stores per node without the collision move 5.2
// against 2.9 TB/s on rows of 32 FP32 nodes, 5.2 against 3.6 on 64, 4.6
// against 3.4 on 60, 5.1 against 4.0 on 192 FP16 nodes.  Padding the rows to
// whole lines loses where nx is no multiple of a line (3.3 TB/s at 60 nodes)
// and changes nothing where it is.
//
// One step = k_main (all nodes of all replicas) + k_links + k_particle
// (bounding box of each sphere).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lbm_kernels.h"
#include "lbm_math.h"
#include "lbm_types.h"

namespace lbm {

template <typename T>
__device__ __forceinline__ Coef<T> make_coef_dev(const RepDesc &D) {
    return coef_of<T>(D);
}

// ------------------------------------------------------------ storage forms
template <typename S> struct Rel { static constexpr bool value = false; };
template <> struct Rel<_Float16> { static constexpr bool value = true; };

template <typename S, typename T>
__device__ __forceinline__ T ld_dev(const S *p, T scale) {
    if constexpr (Rel<S>::value) return T((float)(*p)) * scale;
    else return T(*p);
}
template <typename S, typename T>
__device__ __forceinline__ void st_dev(S *p, T v, T inv_scale) {
    if constexpr (Rel<S>::value) *p = (S)(float)(v * inv_scale);
    else *p = (S)v;
}

// ------------------------------------------------------------------ geometry
struct Geo {
    int nx, ny, nz;
    bool wx, wy, wz;
    int64_t N;          // nodes
};

__device__ __forceinline__ Geo geo_of(const RepDesc &D) {
    Geo g;
    g.nx = D.nx; g.ny = D.ny; g.nz = D.nz;
    g.wx = D.walls & 1u; g.wy = D.walls & 2u; g.wz = D.walls & 4u;
    g.N = D.N;
    return g;
}

// element strides of a replica block: a row's 38 slots, a plane with its two
// ghost rows (fits 31 bits in bytes for every accepted lattice)
__device__ __forceinline__ int row_stride(const Geo &g) { return 2 * Q * g.nx; }
__device__ __forceinline__ int plane_stride(const Geo &g) { return 2 * Q * g.nx * (g.ny + 2); }

// Slot of population i of component l within a row.  Slots that are pulled from
// the same row and plane, i.e. of equal (c_y, c_z), are neighbours: where a
// slot's nx elements are no whole cache lines, two slots share a line, and one
// that is pulled a row or a plane later than the other is fetched twice.
// Read requests of L2 to memory, in order of (component, direction) and so:
// ensemble (32, 24 and 48 node rows) 7.5e7 and 6.6e7 per step, 60 x 60 x 900 7.6e6
// and 6.4e6.
struct SlotOf {
    int s, n;  // slot of component A; component B's is n further
};
constexpr SlotOf slot_of(int i) {
    constexpr int order[9][2] = {{0, 0}, {1, 0}, {-1, 0}, {0, 1}, {1, 1}, {-1, 1}, {0, -1}, {1, -1}, {-1, -1}};
    int at = 0;
    for (int k = 0; k < 9; k++) {
        int n = 0, idx = -1;
        for (int j = 0; j < Q; j++) {
            if (cy(j) != order[k][0] || cz(j) != order[k][1]) continue;
            if (j == i) idx = n;
            n++;
        }
        if (idx >= 0) return {at + idx, n};
        at += 2 * n;
    }
    return {0, 0};
}
struct SlotTable {
    int s[Q], n[Q];
    int dir[Q];  // directions in the order of their slots
};
constexpr SlotTable make_slots() {
    SlotTable t{};
    for (int i = 0; i < Q; i++) {
        t.s[i] = slot_of(i).s;
        t.n[i] = slot_of(i).n;
        int before = 0;
        for (int j = 0; j < Q; j++) before += slot_of(j).s < slot_of(i).s;
        t.dir[before] = i;
    }
    return t;
}
constexpr SlotTable SLOTS = make_slots();
__device__ __forceinline__ constexpr int slot(int l, int i) { return SLOTS.s[i] + l * SLOTS.n[i]; }

// element of slot s at position (x, y, z), 0 <= x < nx, -1 <= y <= ny, -1 <= z <= nz
__device__ __forceinline__ int64_t slot_at(int x, int y, int z, int s, const Geo &g) {
    return (int64_t)(z + 1) * plane_stride(g) + (int64_t)(y + 1) * row_stride(g) + s * g.nx + x;
}

// element that node (x, y, z) pulls population i of component l from
__device__ __forceinline__ int64_t pull_slot(int x, int y, int z, int l, int i, const Geo &g) {
    const int sx = x - cx(i);
    if (sx >= 0 && sx < g.nx) return slot_at(sx, y - cy(i), z - cz(i), slot(l, i), g);
    if (g.wx) return slot_at(x, y, z, slot(l, opp(i)), g);
    return slot_at(sx < 0 ? sx + g.nx : sx - g.nx, y - cy(i), z - cz(i), slot(l, i), g);
}
// unpadded node index (noise counter, fields)
__device__ __forceinline__ uint32_t nidx(int x, int y, int z, const Geo &g) {
    return (uint32_t)x + (uint32_t)g.nx * ((uint32_t)y + (uint32_t)g.ny * (uint32_t)z);
}
// bring a coordinate one layer outside the box back in; false = wall layer
__device__ __forceinline__ bool wrap1(int &v, int n, bool wall) {
    if (v < 0 || v >= n) {
        if (wall) return false;
        v = v < 0 ? v + n : v - n;
    }
    return true;
}
// wall layers mirror onto the adjacent node, periodic axes wrap
__device__ __forceinline__ int mirror1(int v, int n, bool wall) {
    if (v < 0) return wall ? 0 : v + n;
    if (v >= n) return wall ? n - 1 : v - n;
    return v;
}

// minimum-image separation along one axis (periodic axes only)
__device__ __forceinline__ double sepd(double d, int n, bool wall) {
#pragma clang fp contract(off)
    if (!wall) {
        const double h = 0.5 * (double)n;
        if (d > h) d = d - (double)n;
        else if (d < -h) d = d + (double)n;
    }
    return d;
}

// particle-node predicate |x - X|^2 < R^2 in FP64 with every product rounded
// on its own (no contraction), so every implementation decides identically.
__device__ __forceinline__ bool pnode(int x, int y, int z, const double *X, double R2,
                                      const Geo &g) {
#pragma clang fp contract(off)
    const double dx = sepd((double)x - X[0], g.nx, g.wx);
    const double dy = sepd((double)y - X[1], g.ny, g.wy);
    const double dz = sepd((double)z - X[2], g.nz, g.wz);
    double d2 = dx * dx + dy * dy;
    d2 = d2 + dz * dz;
    return d2 < R2;
}

__device__ __forceinline__ int find_rep(const int32_t *begin, int nrep, int wg) {
    int lo = 0, hi = nrep - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (begin[mid] <= wg) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// bbox array index of a box node, -1 when outside the array
__device__ __forceinline__ int bbox_index(int x, int y, int z, const int32_t *org, int S,
                                          const Geo &g) {
    int bx = x - org[0], by = y - org[1], bz = z - org[2];
    if (!g.wx) { if (bx < 0) bx += g.nx; else if (bx >= g.nx) bx -= g.nx; }
    if (!g.wy) { if (by < 0) by += g.ny; else if (by >= g.ny) by -= g.ny; }
    if (!g.wz) { if (bz < 0) bz += g.nz; else if (bz >= g.nz) bz -= g.nz; }
    if (bx < 0 || by < 0 || bz < 0 || bx >= S || by >= S || bz >= S) return -1;
    return (bz * S + by) * S + bx;
}

// position of bbox entry b (origin org, edge S); false when it lies in a wall layer
__device__ __forceinline__ bool bbox_pos(int b, const int32_t *org, int S, const Geo &g, int (&bb)[3],
                                         int (&p)[3]) {
    bb[0] = b % S; bb[1] = (b / S) % S; bb[2] = b / (S * S);
    const int n3[3] = {g.nx, g.ny, g.nz};
    const bool w3[3] = {g.wx, g.wy, g.wz};
    bool in = true;
    for (int q = 0; q < 3; q++) {
        int v = org[q] + bb[q];
        if (v < 0 || v >= n3[q]) {
            if (w3[q]) in = false;
            else v = ((v % n3[q]) + n3[q]) % n3[q];
        }
        p[q] = v;
    }
    return in;
}

// ------------------------------------------------------------------ pulling
// Populations f_{l i}(x, n) of a fluid node in deviation form (see the storage
// note at the top for where each comes from).
template <typename S, typename T>
struct PullCtx {
    const S *src;          // replica block
    int32_t nx, RS, PS;    // row length, row and plane strides
    bool wx;
    T scale[2];            // FP16 relative storage: rho0_l (times w_i per slot)
};

template <typename S, typename T>
__device__ __forceinline__ PullCtx<S, T> pull_ctx(const void *buf, const RepDesc &D, const Geo &g) {
    PullCtx<S, T> pc;
    pc.src = reinterpret_cast<const S *>(buf) + D.pop_off;
    pc.nx = g.nx;
    pc.RS = row_stride(g);
    pc.PS = plane_stride(g);
    pc.wx = g.wx;
    for (int l = 0; l < 2; l++) pc.scale[l] = Rel<S>::value ? T(D.rho0[l]) : T(1);
    return pc;
}

// Buffer access: scalar base (64-bit, in a descriptor) + per-lane 32-bit byte
// offset + scalar byte offset, so the 38 slots of a node cost one scalar
// addition each and no vector address arithmetic.  Offsets stay below 4 GiB
// (two planes of any accepted lattice do), so the descriptor's size check is
// left open.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc rsrc_of(const void *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00027000);
}

template <typename S>
__device__ __forceinline__ S buf_ld(Rsrc r, uint32_t vo, uint32_t so) {
    if constexpr (sizeof(S) == 8) return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
    else if constexpr (sizeof(S) == 4) return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
    else return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(r, vo, so, 0));
}
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
// AUX 2: non-temporal
template <typename S, int AUX = 0>
__device__ __forceinline__ void buf_st(S v, Rsrc r, uint32_t vo, uint32_t so) {
    if constexpr (sizeof(S) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, v), r, vo, so, AUX);
    else if constexpr (sizeof(S) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, vo, so, AUX);
    else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, vo, so, AUX);
}

// a wave-uniform value recomputed from here on instead of being kept (the
// scalar registers do not hold every derived offset at once)
__device__ __forceinline__ void renew(int32_t &v) { asm volatile("" : "+s"(v)); }

// Components L0 .. L0 + NL - 1 of a node; z uniform over the wave, (x, y) per
// lane.
template <int NL, typename S, typename T>
__device__ __forceinline__ void pull_row(PullCtx<S, T> c, int x, int y, int z, int L0, T (&d)[NL][Q]) {
    constexpr uint32_t es = sizeof(S);
    renew(c.nx);
    renew(c.RS);
    renew(c.PS);
    const uint32_t nxb = (uint32_t)c.nx * es, RSb = (uint32_t)c.RS * es, PSb = (uint32_t)c.PS * es;
    // bases two rows before plane z (c_z <= 0: plane z + 1 is one plane further)
    // and before plane z - 1 (c_z > 0), so that no offset is negative
    const S *pl = c.src + (int64_t)(z + 1) * c.PS - 2 * (int64_t)c.RS;
    const Rsrc r0 = rsrc_of(pl), r1 = rsrc_of(pl - c.PS);
    const bool lo = x == 0, hi = x == c.nx - 1;
    const uint32_t own = (uint32_t)(y + 2) * RSb + (uint32_t)x * es;
    const uint32_t vm = lo ? own + (nxb - es) : own - es, vp = hi ? own - (nxb - es) : own + es;
    const bool wm = c.wx && lo, wp = c.wx && hi;
#pragma unroll
    for (int k = 0; k < Q; k++) {
        const int i = SLOTS.dir[k];
        const T w = T(wgt(i));
        uint32_t vo = (cx(i) > 0 ? vm : cx(i) < 0 ? vp : own) + (cz(i) < 0 ? PSb : 0u);
        if (cx(i)) {
            // across an x-wall: the node's own slot opp(i), in plane z
            const uint32_t up = (uint32_t)(slot(0, opp(i)) - slot(0, i)) * nxb + (cy(i) > 0 ? RSb : cy(i) < 0 ? 0u - RSb : 0u) +
                               (cz(i) > 0 ? PSb : 0u);
            vo = (cx(i) > 0 ? wm : wp) ? own + up : vo;
        }
        const uint32_t so = (uint32_t)(1 - cy(i)) * RSb + (uint32_t)slot(L0, i) * nxb;
#pragma unroll
        for (int l = 0; l < NL; l++) {
            const S v = buf_ld<S>(cz(i) > 0 ? r1 : r0, vo, so + (uint32_t)(l * SLOTS.n[i]) * nxb);
            d[l][i] = ld_dev<S, T>(&v, w * (L0 + l ? c.scale[1] : c.scale[0]));
        }
    }
}

// FP16 storage: a pulled population is a product (number times scale), which the
// compiler may round, or fuse into the sums it enters.  Of two opposite ones the
// second (even i) is rounded here, so that component_modes always fuses the first,
// whichever of its outputs are read: a node's density must not depend on whether
// it is a tile's own node or a neighbour tile's halo.
template <typename S, typename T>
__device__ __forceinline__ void settle_pairs(T (&d)[Q]) {
    if constexpr (Rel<S>::value) {
#pragma unroll
        for (int i = 2; i < Q; i += 2) asm("" : "+v"(d[i]));
    }
}

// any node
template <typename S, typename T>
__device__ __forceinline__ void pull_node(const PullCtx<S, T> &c, int x, int y, int z, T (&d)[2][Q]) {
    const S *own = c.src + (int64_t)(z + 1) * c.PS + (int64_t)(y + 1) * c.RS + x;
    const bool lo = x == 0, hi = x == c.nx - 1;
    const int32_t dm = lo ? c.nx - 1 : -1, dp = hi ? 1 - c.nx : 1;
#pragma unroll
    for (int i = 0; i < Q; i++) {
        const T w = T(wgt(i));
        int32_t off = slot(0, i) * c.nx - cy(i) * c.RS - cz(i) * c.PS + (cx(i) > 0 ? dm : cx(i) < 0 ? dp : 0);
        if (cx(i)) off = c.wx && (cx(i) > 0 ? lo : hi) ? slot(0, opp(i)) * c.nx : off;
        d[0][i] = ld_dev<S, T>(own + off, w * c.scale[0]);
        d[1][i] = ld_dev<S, T>(own + off + SLOTS.n[i] * c.nx, w * c.scale[1]);
    }
}

// Density deviations and momenta of the pulled populations of a node.
template <typename T>
struct NodeM {
    T rd[2];
    T j[2][3];
};

template <typename T>
__device__ __forceinline__ void node_moments(const T (&d)[2][Q], NodeM<T> &s) {
#pragma unroll
    for (int l = 0; l < 2; l++) {
        T r = T(0), jx = T(0), jy = T(0), jz = T(0);
#pragma unroll
        for (int i = 0; i < Q; i++) {
            r += d[l][i];
            if (cx(i) > 0) jx += d[l][i]; else if (cx(i) < 0) jx -= d[l][i];
            if (cy(i) > 0) jy += d[l][i]; else if (cy(i) < 0) jy -= d[l][i];
            if (cz(i) > 0) jz += d[l][i]; else if (cz(i) < 0) jz -= d[l][i];
        }
        s.rd[l] = r; s.j[l][0] = jx; s.j[l][1] = jy; s.j[l][2] = jz;
    }
}

// ------------------------------------------------------- block reductions
// x + (x moved across lanes by the DPP pattern CTRL), FP64 as two 32-bit moves
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const int plo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, false);
    const int phi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, false);
    return x + __hiloint2double(phi, plo);
}

// x + (x of the lane 16 or 32 apart), the lower lane's value first in every
// lane, FP64 as two 32-bit swaps (v_permlane16_swap / v_permlane32_swap:
// rows 0-1 and 2-3, or the two halves of the wave, exchanged)
__device__ __forceinline__ double add_row_pair(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ __forceinline__ double add_half_pair(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}

// Sum over the 64 lanes of a wave, in a fixed order and bitwise the same in
// every lane: lane pairs, then quads, 8-lane halves and 16-lane rows are
// combined with DPP permutations (quad swaps, half-row and row mirrors; each
// step adds two equal partial sums in either order, so all lanes agree), then
// rows 0 + 1 and 2 + 3 and the two halves with lane swaps (lower part first).
// Everything stays in vector registers.  All lanes of the wave must be active.
template <int NV>
__device__ __forceinline__ void wave_sum(double (&v)[NV]) {
#pragma unroll
    for (int k = 0; k < NV; k++) {
        double x = v[k];
        x = dpp_add<0xB1>(x);   // quad_perm [1,0,3,2]
        x = dpp_add<0x4E>(x);   // quad_perm [2,3,0,1]
        x = dpp_add<0x141>(x);  // row_half_mirror
        x = dpp_add<0x140>(x);  // row_mirror
        x = add_row_pair(x);
        v[k] = add_half_pair(x);
    }
}

// fixed-order sum over the workgroup, result in every thread
template <int B, int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double *red /* [B/64][NV] */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_sum<NV>(v);
    __syncthreads();  // earlier readers of red are done
    if (lane == 0)
        for (int k = 0; k < NV; k++) red[wave * NV + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; k++) {
        double s = 0.0;
        for (int w = 0; w < B / 64; w++) s += red[w * NV + k];
        v[k] = s;
    }
}

// Workgroups are dispatched to the 8 XCDs round-robin; give each XCD a
// contiguous run of logical tiles so halo rows and planes shared by
// neighbouring tiles are read through the same L2.
__device__ __forceinline__ int xcd_logical(int b, int G) {
    const int q = G >> 3, r = G & 7, xcd = b & 7, slot = b >> 3;
    return xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}

// ================================================================ k_main
// Workgroup = ty full x-rows of one replica, marching over cz z-planes.
// Density deviations of the tile plus a one-node halo (rows y0-1 and
// y0+rows, planes z-1 and z+1) sit in a 4-plane LDS ring; halo densities are
// recomputed from pulled populations, so no density field goes through HBM.
// The density and momenta of the next plane stay in registers while the
// current plane collides.  The sphere enters only through the solid flags
// and wetting-layer densities of its bounding box; every FP64 particle
// computation lives in the bounding-box kernels.
// FP32 arithmetic with all relaxation times 1 (FP32 or FP16 storage): both
// components unrolled and the kernel held to 128 VGPRs (four waves per SIMD).
// Other forms keep the component loop rolled and at least three waves per SIMD
// (FP32) or two (FP64).
template <typename S, typename T, bool TAU1>
constexpr bool main_fast_form = sizeof(T) == 4 && TAU1;
template <typename S, typename T, bool TAU1>
constexpr bool main_unroll = sizeof(T) == 4 && TAU1;

// GROUP: fluids may hold several spheres (their boxes are searched too); a
// separate instantiation, so the single-sphere form keeps its registers.
// NOISE: some replica of the launch has kT > 0.  Every node then draws its
// normals; a replica with kT = 0 has zero amplitudes and takes none of them
// (products with zero).  Without it no normals are drawn.  Being a compile-
// time choice, the noise-free form costs the noisy one nothing.
template <typename S, typename T, int B, bool TAU1, bool GROUP, bool NOISE>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(main_fast_form<S, T, TAU1> ? 4 : sizeof(T) == 4 ? 3 : 2)))
void k_main(MainArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    T *lds = reinterpret_cast<T *>(smem);

    const int wg = xcd_logical(blockIdx.x, gridDim.x);
    const int r = find_rep(a.wg_begin, a.nrep, wg);
    const RepDesc D = a.desc[r];  // by value: no reload after stores
    RepState *stp = a.state + r;
    const Geo g = geo_of(D);
    const int nx = g.nx, ty = D.ty, zc = D.cz;
    const int local = wg - D.wg_begin;
    const int yt = local % D.nty, ch = local / D.nty;
    const int y0 = yt * ty, rows = min(ty, g.ny - y0);
    const int z0 = ch * zc, z1 = min(z0 + zc, g.nz);
    const int t = threadIdx.x;
    const int nin = nx * rows;
    // this lane's node: x and, in the upper half, its row of the tile (0x4000 and
    // more: none).  Kept packed, and what follows from it formed per plane, since
    // hoisted coordinates, neighbours and face masks cost 20 VGPRs.
    uint32_t pos = t < nin ? (uint32_t)(t % nx) | (uint32_t)(t / nx) << 16 : 0x40000000u;
    const int pr = (ty + 2) * nx;  // LDS elements per plane and component

    // Non-temporal stores where the populations cannot stay in the 256 MB cache
    // before memory (both buffers over 300 MB where a row's slots fill whole 128-byte
    // lines, over 350 MB where they fill 64-byte halves); FP32 and FP64.  Plain and
    // non-temporal, us: 192 ensemble channels (9.9 GB) 2437 and 2265, 64 x 64 x 256
    // (319 MB) 86.6 and 83.1, 128^3 160 and 152, 64 x 64 x 200 FP64 211 and 194.
    // Gain of a step, in one and in nine replicas of rows of nx nodes, by the size of
    // both buffers (MB):
    //              260          300          325          350          430          700
    //   FP32 64    0.91 0.91    0.99 0.98    1.02 1.02    1.07 1.05    1.02 1.02    1.05 1.05
    //        32    0.87 0.85    1.00 0.98    1.04 1.03    1.07 1.06    1.02 1.03    1.05 1.05
    //   (halves)
    //        48    0.85 0.85    0.97 0.94    1.01 1.00    1.03 1.00    1.03 1.03    1.05 1.05
    //        16    0.79 0.78    0.95 0.93    0.98 0.98    1.02 1.01    1.01 1.01    1.04 1.04
    //        80    0.87 0.86    0.95 0.91    1.00 0.92    1.03 1.00    1.01 1.01    1.04 1.04
    //       112    0.84 0.85    0.97 0.91    0.99 0.94    0.99 0.95    1.02 1.04    1.04 1.05
    //   FP64 40    0.98 1.00    1.02 1.00    1.04 1.03    1.04 1.04    1.06 1.04    1.04 1.04
    // Rows of other lengths write lines in parts (60 x 60 x 900: 290 and 326 us), and
    // FP16 gains nothing (192 x 192 x 1024: 1937 and 1917; 96 x 96 x 512: 323 and 328).
    const bool stream = sizeof(S) >= 4 && a.stream && ((nx * (int)sizeof(S)) & (a.stream - 1)) == 0;
    const bool hp = D.has_particle;
    const int nsph = GROUP ? D.n_sph : 1;
    const PullCtx<S, T> pc = pull_ctx<S, T>(a.src, D, g);
    const T dl[2] = {T(stp->delta[0]), T(stp->delta[1])};
    const double dld[2] = {stp->delta[0], stp->delta[1]};
    const uint32_t step = (uint32_t)stp->step;
    const int32_t org[3] = {stp->org[0], stp->org[1], stp->org[2]};
    const int Sx = D.S, S3 = Sx * Sx * Sx;
    const uint32_t *__restrict__ pmask = a.pmask + D.bbox_off;
    const double *__restrict__ vrho = a.vrho + D.bbox_off * 2;
    double *__restrict__ rho_n = a.rho_n + D.bbox_off * 2;
    S *__restrict__ dst = reinterpret_cast<S *>(a.dst) + D.pop_off;
    const double rho0d[2] = {D.rho0[0], D.rho0[1]};
    const T G = sizeof(T) == 4 ? T(D.G32) : T(D.G);
    const T af[3] = {sizeof(T) == 4 ? T(D.af32[0]) : T(D.af[0]), sizeof(T) == 4 ? T(D.af32[1]) : T(D.af[1]),
                     sizeof(T) == 4 ? T(D.af32[2]) : T(D.af[2])};
    const uint32_t key0 = D.key0, key1 = D.key1;
    const Coef<T> cf = make_coef_dev<T>(D);
    uint32_t k0 = key0, k1 = key1;
    PullCtx<S, T> pcl = pc;

    // four plane slots: the fill of the next plane never lands on a slot the
    // collision of the current plane still reads, so one barrier per plane
    auto L = [&](int zp, int l, int row, int xx) -> T & {
        const int slot = zp & 3;
        return lds[(slot * 2 + l) * pr + (row + 1) * nx + xx];
    };

    // whether plane z meets the sphere's box (uniform; with several spheres: may)
    auto box_plane = [&](int z) -> bool {
        int bz = z - org[2];
        if (!g.wz) bz = bz < 0 ? bz + g.nz : (bz >= g.nz ? bz - g.nz : bz);
        return hp && ((GROUP && nsph > 1) || (uint32_t)bz < (uint32_t)Sx);
    };

    // density deviation of a box node: pulled (plus the mass correction), or
    // the wetting-layer value on particle nodes; fluid nodes also return
    // their moments (have: the node's populations, if they are loaded already)
    auto node_density = [&](int xx, int yy, int zz, bool zbox, const T(*have)[Q], NodeM<T> &s, T &rA, T &rB) -> bool {
        int b = -1;
        if (zbox) b = bbox_index(xx, yy, zz, org, Sx, g);
        if (b < 0 || !(pmask[b] & MASK_SOLID)) {
            // the group's other spheres (their boxes are disjoint from this
            // one's and from each other, so at most one holds the node)
            int64_t vi = -1;
            int vs = 0;
            if (GROUP && nsph > 1 && b < 0) {
                for (int e = 1; e < nsph; e++) {
                    const RepDesc *De = a.desc + r + e;
                    const int Se = De->S;
                    const int be = bbox_index(xx, yy, zz, a.state[r + e].org, Se, g);
                    if (be < 0) continue;
                    if (a.pmask[De->bbox_off + be] & MASK_SOLID) {
                        vi = 2 * De->bbox_off + be;
                        vs = Se * Se * Se;
                    }
                    break;
                }
            }
            if (vi < 0) {
                T d[2][Q];
                if constexpr (TAU1) {
                    if (!have) pull_row<2>(pcl, xx, yy, zz, 0, d);
#pragma unroll
                    for (int i = 0; i < Q && have; i++) {
                        d[0][i] = have[0][i];
                        d[1][i] = have[1][i];
                    }
                    node_moments(d, s);
                } else {
                    pull_row<2>(pcl, xx, yy, zz, 0, d);
                    settle_pairs<S>(d[0]);
                    settle_pairs<S>(d[1]);
                    T unused[Q];
                    component_modes(d[0], s.rd[0], s.j[0], unused);
                    component_modes(d[1], s.rd[1], s.j[1], unused);
                }
                s.rd[0] += dl[0];
                s.rd[1] += dl[1];
                rA = s.rd[0];
                rB = s.rd[1];
                return true;
            }
            rA = T(a.vrho[vi] + dld[0] - rho0d[0]);
            rB = T(a.vrho[vi + vs] + dld[1] - rho0d[1]);
            return false;
        }
        rA = T(vrho[b] + dld[0] - rho0d[0]);
        rB = T(vrho[S3 + b] + dld[1] - rho0d[1]);
        return false;
    };

    NodeM<T> nxt;
    bool nxt_fluid = false;

    // FP32, all relaxation times 1: the next plane's populations of this lane's
    // node are loaded while the current plane collides (38 registers, which the
    // packed position leaves room for at four waves per SIMD), so that memory is
    // busy in the collision phase too.  Measured without and with: 60 x 60 x 900
    // 296 -> 290 us, 192 ensemble channels 2464 -> 2400, 6 x (32 x 32 x 128) 61.1 ->
    // 58.8, 64 x 64 x 256 86.7 -> 85.4.  FP16 storage loses by it (192 x 192 x 1024:
    // 1912 -> 2082 us; bound by the vector ALU, and each 16-bit number held takes a
    // register), and the general and FP64 forms have no registers left.
    constexpr bool PREF = main_fast_form<S, T, TAU1> && sizeof(S) == 4;
    T pre[2][Q];
    auto prefetch = [&](int zp) {
        const int zz = mirror1(zp, g.nz, g.wz);
        const int x = (int)(pos & 0xffffu), yl = (int)(pos >> 16);
        if (yl < 0x4000) pull_row<2>(pcl, x, y0 + yl, zz, 0, pre);
        __builtin_amdgcn_sched_barrier(0);
    };
    // fill LDS plane zp (unmapped index); the interior node's moments go to nxt
    auto fill = [&](int zp) {
        const int zz = mirror1(zp, g.nz, g.wz);
        const bool zbox = box_plane(zz);
        const int x = (int)(pos & 0xffffu), yl = (int)(pos >> 16);
        if (yl < 0x4000) {
            T rA, rB;
            nxt_fluid = node_density(x, y0 + yl, zz, zbox, PREF ? pre : nullptr, nxt, rA, rB);
            L(zp, 0, yl, x) = rA;
            L(zp, 1, yl, x) = rB;
        }
        for (int h = t - nin; h < 2 * nx; h += B) {
            if (h < 0) continue;
            const int row = h < nx ? -1 : rows;
            const int xx = h < nx ? h : h - nx;
            const int yy = mirror1(y0 + row, g.ny, g.wy);
            NodeM<T> hd;
            T rA, rB;
            node_density(xx, yy, zz, zbox, nullptr, hd, rA, rB);
            L(zp, 0, row, xx) = rA;
            L(zp, 1, row, xx) = rB;
        }
    };

    // Plane zp is filled while the plane filled before it collides.  Odd
    // z-chunks march downwards, so two neighbouring chunks read the halo
    // planes they share at the same time (both at their start or both at
    // their end) and the second read hits L2.
    const int dir = (ch & 1) ? -1 : 1;
    const int zfirst = dir > 0 ? z0 - 1 : z1;
    const int nplanes = z1 - z0 + 2;
    if constexpr (PREF) prefetch(zfirst);
    for (int k = 0; k < nplanes; k++) {
        // keep uniform values derived from these roots inside the loop (scalar
        // recomputation is cheaper than spilling hoisted copies)
        asm volatile("" : "+s"(k0), "+s"(k1), "+s"(pcl.nx), "+s"(pcl.RS), "+s"(pcl.PS));
        asm volatile("" : "+v"(pos));
        const int zp = zfirst + dir * k;
        const NodeM<T> cur = nxt;
        const bool cur_fluid = nxt_fluid;
        fill(zp);
        __syncthreads();
        if constexpr (PREF)
            if (k + 1 < nplanes) prefetch(zp + dir);
        if (k < 2) continue;
        const int z = zp - dir;
        const int x = (int)(pos & 0xffffu), yl = (int)(pos >> 16), y = y0 + yl;
        if (yl < 0x4000 && cur_fluid) {
            const int xm = mirror1(x - 1, nx, g.wx), xp = mirror1(x + 1, nx, g.wx);
            const bool ylo = y == 0, yhi = y == g.ny - 1;
            const T(&rd)[2] = cur.rd;
            const T(&j)[2][3] = cur.j;
            // Shan-Chen: F_l = -G rho_l sum_i w_i rho~_l'(x + c_i) c_i + rho_l a_f
            T grad[2][3] = {{T(0), T(0), T(0)}, {T(0), T(0), T(0)}};
#pragma unroll
            for (int i = 1; i < Q; i++) {
                const int xx = cx(i) > 0 ? xp : (cx(i) < 0 ? xm : x);
                const T w = T(wgt(i));
#pragma unroll
                for (int l = 0; l < 2; l++) {
                    const T v = w * L(z + cz(i), l, yl + cy(i), xx);
                    if (cx(i)) grad[l][0] += cx(i) > 0 ? v : -v;
                    if (cy(i)) grad[l][1] += cy(i) > 0 ? v : -v;
                    if (cz(i)) grad[l][2] += cz(i) > 0 ? v : -v;
                }
            }
            const T rl[2] = {cf.rho0[0] + rd[0], cf.rho0[1] + rd[1]};
            if (!(rl[0] > T(0)) || !(rl[1] >= T(0))) atomicOr(&stp->flags, FLAG_UNSTABLE);
            if (box_plane(z)) {  // densities near the spheres, for the link kernel
                const int b = bbox_index(x, y, z, org, Sx, g);
                if (b >= 0) {
                    rho_n[b] = (double)rl[0];
                    rho_n[S3 + b] = (double)rl[1];
                } else if (GROUP && nsph > 1) {
                    for (int e = 1; e < nsph; e++) {
                        const RepDesc *De = a.desc + r + e;
                        const int Se = De->S;
                        const int be = bbox_index(x, y, z, a.state[r + e].org, Se, g);
                        if (be < 0) continue;
                        double *rn = a.rho_n + 2 * De->bbox_off;
                        rn[be] = (double)rl[0];
                        rn[Se * Se * Se + be] = (double)rl[1];
                        break;
                    }
                }
            }
            T F[2][3];
#pragma unroll
            for (int q = 0; q < 3; q++) {
                if constexpr (TAU1) {  // (rounded as the compiler takes it; below: stated)
                    F[0][q] = -G * rl[0] * grad[1][q] + rl[0] * af[q];
                    F[1][q] = -G * rl[1] * grad[0][q] + rl[1] * af[q];
                } else {
                    F[0][q] = fma_of(-G * rl[0], grad[1][q], rl[0] * af[q]);
                    F[1][q] = fma_of(-G * rl[1], grad[0][q], rl[1] * af[q]);
                }
            }
            const uint32_t node = (uint32_t)(x + nx * (y + g.ny * z));
            T u[3], xid[3];
            T zz[36];
            if constexpr (NOISE) noise_block<T>(node, step, 8u, k0, k1, zz + 32);
            else zz[32] = zz[33] = zz[34] = T(0);
            common_velocity(rd, j, F, zz, cf, u, xid);
            const bool zlo = z == 0, zhi = z == g.nz - 1;
            const bool yzface = ylo || yhi || zlo || zhi;
            S *dplane = dst + (int64_t)(z + 1) * pcl.PS;
            const Rsrc drs = rsrc_of(dplane);
            const uint32_t own = ((uint32_t)(y + 1) * (uint32_t)pcl.RS + (uint32_t)x) * (uint32_t)sizeof(S);
            constexpr int kCompUnroll = main_unroll<S, T, TAU1> ? 2 : 1;
#pragma unroll kCompUnroll
            for (int l = 0; l < 2; l++) {
                // this component's values (selected, so nothing is indexed by l)
                const T rdl = l ? rd[1] : rd[0];
                const T jl[3] = {l ? j[1][0] : j[0][0], l ? j[1][1] : j[0][1], l ? j[1][2] : j[0][2]};
                const T Fl[3] = {l ? F[1][0] : F[0][0], l ? F[1][1] : F[0][1], l ? F[1][2] : F[0][2]};
                const T r0l = l ? cf.rho0[1] : cf.rho0[0];
                const T sig = l ? T(-1) : T(1);
                // general relaxation: modes 4..18 of the populations, pulled once more
                // (from the caches); carried along since the fill they cost 30
                // registers.  The loads are issued before the normals are drawn.
                T dl1[1][TAU1 ? 1 : Q];
                if constexpr (!TAU1) {
                    pull_row<1>(pcl, x, y, z, l, dl1);
                    if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
                }
                T zl[16];
                if constexpr (NOISE) {
#pragma unroll
                    for (int b = 0; b < 4; b++)
                        noise_block<T>(node, step, (uint32_t)(4 * l + b), k0, k1, zl + 4 * b);
                } else {
#pragma unroll
                    for (int k = 0; k < 16; k++) zl[k] = T(0);
                }
                T out[Q];
                if constexpr (TAU1) {
                    relax_tau1(r0l, sig, rdl, jl, Fl, u, xid, zl, cf, out);
                } else {
                    T ml[Q], rdm, jm[3];
                    settle_pairs<S>(dl1[0]);
                    component_modes(dl1[0], rdm, jm, ml);
                    // each mode a number of its own: fused into the relaxation the
                    // sums would round differently from form to form
#pragma unroll
                    for (int k = 4; k < Q; k++) asm("" : "+v"(ml[k]));
                    relax_component(r0l, sig, rdl, jl, ml, Fl, u, xid, zl, cf, out);
                }
                const T sc = Rel<S>::value ? r0l : T(1);
                int32_t nxs = nx;
                renew(nxs);
                const uint32_t nxb = (uint32_t)nxs * (uint32_t)sizeof(S);
                // the values are final here: formed inside the two branches below, FP64
                // sums would be fused differently from one form of the kernel to another
                if constexpr (sizeof(T) == 8) {
#pragma unroll
                    for (int i = 0; i < Q; i++) asm("" : "+v"(out[i]));
                }
                auto store = [&](auto aux) {
#pragma unroll
                    for (int i = 0; i < Q; i++) {
                        const T inv = Rel<S>::value ? T(1) / (T(wgt(i)) * sc) : T(1);
                        S v;
                        st_dev<S, T>(&v, out[i], inv);
                        buf_st<S, decltype(aux)::value>(v, drs, own, (uint32_t)slot(l, i) * nxb);
                    }
                };
                if (stream) store(std::integral_constant<int, 2>{});
                else store(std::integral_constant<int, 0>{});
                // A link that leaves the box through a y- or z-face also writes its
                // value where the receiver pulls it from: the wall ghost x + c_i,
                // slot opp(i) (half-way bounce-back), or the periodic image of x,
                // slot i.  (Through an x-face alone it is pulled from the node's
                // own slot, and across an x-wall whatever the other axes are.)
                if (yzface) {
                    const bool xlo = x == 0, xhi = x == nx - 1;
#pragma unroll
                    for (int i = 1; i < Q; i++) {
                        if (cy(i) == 0 && cz(i) == 0) continue;
                        const T inv = Rel<S>::value ? T(1) / (T(wgt(i)) * sc) : T(1);
                        const bool ex = cx(i) > 0 ? xhi : (cx(i) < 0 ? xlo : false);
                        const bool ey = cy(i) > 0 ? yhi : (cy(i) < 0 ? ylo : false);
                        const bool ez = cz(i) > 0 ? zhi : (cz(i) < 0 ? zlo : false);
                        if ((ey || ez) && !(ex && g.wx)) {
                            const bool bounce = (ey && g.wy) || (ez && g.wz);
                            const int32_t dx = ex ? cx(i) * (1 - nx) : cx(i);
                            const int64_t so =
                                bounce ? (int64_t)(slot(l, opp(i)) * pcl.nx + cy(i) * pcl.RS + dx) + (int64_t)cz(i) * pcl.PS
                                       : (int64_t)(slot(l, i) * pcl.nx) - (int64_t)(ey ? cy(i) * g.ny : 0) * pcl.RS -
                                             (int64_t)(ez ? cz(i) * g.nz : 0) * pcl.PS;
                            S *base = dplane;
                            st_dev<S, T>(reinterpret_cast<S *>(reinterpret_cast<char *>(base + so) + own), out[i], inv);
                        }
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------- sphere-box helpers
// Sum of NV values over per-workgroup partials [count][PART] starting at k0,
// in a fixed order independent of the launch: lane l adds partials l, l + 64,
// ..., then a butterfly over the wave.  Every lane of every wave holds the
// same result, so no LDS or barrier is needed.
// A lane's partials are loaded CH at a time before they are added (in the
// same order), so a long list costs 1/CH of the dependent round trips.
template <int NV>
__device__ __forceinline__ void sum_partials(const double *part, int count, int k0, double (&v)[NV]) {
    constexpr int CH = NV > 16 ? 2 : 4;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < NV; k++) v[k] = 0.0;
    for (int w0 = lane; w0 < count; w0 += CH * 64) {
        double c[CH][NV];
#pragma unroll
        for (int j = 0; j < CH; j++) {
            const int w = w0 + 64 * j;
            const double *p = part + (int64_t)(w < count ? w : 0) * PART + k0;
#pragma unroll
            for (int k = 0; k < NV; k++) c[j][k] = p[k];
        }
#pragma unroll
        for (int j = 0; j < CH; j++) {
            if (w0 + 64 * j >= count) break;
#pragma unroll
            for (int k = 0; k < NV; k++) v[k] += c[j][k];
        }
    }
    wave_sum<NV>(v);
}

// Neighbourhood of a box node p for the particle predicate: for p itself
// (bit 0) and each neighbour p + c_i (bit i), whether it lies inside the
// lattice (not a wall layer) and whether it is a particle node of the
// sphere at Xc.  The squared minimum-image separations along each axis are
// formed once for the positions p + {-1, 0, 1} (wrapped on periodic axes) and
// combined in the order pnode uses, so every decision is bitwise the one
// pnode takes for that node.  Held as two bit masks, not as arrays, so that
// nothing of it is kept in scratch memory.
struct Nbr {
    uint32_t ok;      // bit i: p + c_i inside the lattice
    uint32_t solid;   // bit i: p + c_i a particle node
};

__device__ __forceinline__ void nbr_of(const int (&p)[3], const double *Xc, double R2, const Geo &g,
                                       Nbr &nb) {
#pragma clang fp contract(off)
    const int n3[3] = {g.nx, g.ny, g.nz};
    const bool w3[3] = {g.wx, g.wy, g.wz};
    double sq[3][3];
    bool in[3][3];
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            int q = p[ax] + k - 1;
            in[ax][k] = w3[ax] ? (q >= 0 && q < n3[ax]) : true;
            if (!w3[ax]) q = q < 0 ? q + n3[ax] : (q >= n3[ax] ? q - n3[ax] : q);
            const double d = sepd((double)q - Xc[ax], n3[ax], w3[ax]);
            sq[ax][k] = d * d;
        }
    }
    nb.ok = 0u;
    nb.solid = 0u;
#pragma unroll
    for (int i = 0; i < Q; i++) {
        double d2 = sq[0][cx(i) + 1] + sq[1][cy(i) + 1];
        d2 = d2 + sq[2][cz(i) + 1];
        if (in[0][cx(i) + 1] && in[1][cy(i) + 1] && in[2][cz(i) + 1]) nb.ok |= 1u << i;
        if (d2 < R2) nb.solid |= 1u << i;
    }
}

__device__ __forceinline__ bool nbr_ok(const Nbr &nb, int i) { return (nb.ok >> i) & 1u; }

__device__ __forceinline__ bool pnode_nb(const Nbr &nb, int i) { return (nb.solid >> i) & 1u; }

// storage form of a deviation (as st_dev writes it) and the value a pull of
// it returns (as ld_dev reads it with the pull's scale)
template <typename S, typename T>
__device__ __forceinline__ T store_round(double v, T inv_scale, T scale, S &sv) {
    if constexpr (Rel<S>::value) {
        sv = (S)(float)(T(v) * inv_scale);
        return T((float)sv) * scale;
    } else {
        sv = (S)T(v);
        return T(sv);
    }
}

// Four lanes per box node.  k_links and k_particle are chains of a few
// thousand nodes on a chip of 1024 SIMDs, so what they take is the number of
// instructions one wave issues, one after another, and the round trips it
// waits for.  Lane q of a node's quad takes the directions i = 5 q + m,
// m = 0 .. 4 (i = 19: none): a quarter of the loads, predicates and link terms
// each, in code that is the same for every direction (the velocities come from
// bit tables) and a fifth as long.  With one lane per node every surface wave
// issued 1.7 k (k_links) and 2.2 k (k_particle) vector instructions.
// 64 x 64 x 256 channel (R = 8): k_links 12.6 -> 6.5 us, k_particle 23.3 -> 11.6;
// 16 x 16 x 32 (R = 3): 11.7 -> 5.7 and 16.8 -> 10.7 us.  192 spheres, where the
// chip is full and the quads' common work counts: both together 145 -> 176 us of
// a 2.4 ms step.
constexpr int QM = 5;
constexpr uint32_t dir_bits(int ax, int m) {  // c + 1 of the four directions 5 q + m, two bits each
    uint32_t v = 0;
    for (int q = 0; q < 4; q++) {
        const int i = QM * q + m;
        const int c = i >= Q ? 0 : ax == 0 ? cx(i) : ax == 1 ? cy(i) : cz(i);
        v |= (uint32_t)(c + 1) << (2 * q);
    }
    return v;
}
constexpr uint32_t slot_bits(bool against, int m) {  // their slots (or their opposites'), one byte each; bit 7: n = 3
    uint32_t v = 0;
    for (int q = 0; q < 4; q++) {
        const int i = QM * q + m < Q ? QM * q + m : 0;
        const SlotOf s = slot_of(against ? opp(i) : i);
        v |= (uint32_t)(s.s | (s.n == 3 ? 0x80 : 0)) << (8 * q);
    }
    return v;
}
struct QDir {
    int c[3];
    int i;          // direction
    int s, so, n;   // its slot and its opposite's (component A), step to component B
    bool valid;     // a moving direction (i = 1 .. 18)
};
template <int M>
__device__ __forceinline__ QDir quad_dir(int q) {
    QDir d;
    constexpr uint32_t bx = dir_bits(0, M), by = dir_bits(1, M), bz = dir_bits(2, M);
    d.c[0] = (int)((bx >> (2 * q)) & 3u) - 1;
    d.c[1] = (int)((by >> (2 * q)) & 3u) - 1;
    d.c[2] = (int)((bz >> (2 * q)) & 3u) - 1;
    d.i = QM * q + M;
    constexpr uint32_t bs = slot_bits(false, M), bo = slot_bits(true, M);
    d.s = (int)((bs >> (8 * q)) & 63u);
    d.so = (int)((bo >> (8 * q)) & 63u);
    d.n = (bs >> (8 * q)) & 0x80u ? 3 : 1;
    d.valid = M == 0 ? q != 0 : M == QM - 1 ? q != 3 : true;
    return d;
}
// the direction against d (its number is not needed)
__device__ __forceinline__ QDir against(const QDir &d) {
    return {{-d.c[0], -d.c[1], -d.c[2]}, -1, d.so, d.s, d.n, d.valid};
}
// w_i of direction 5 q + M
template <int M>
__device__ __forceinline__ double quad_w(int q) {
    if (M == 0) return q == 0 ? 1.0 / 3.0 : q == 1 ? 1.0 / 18.0 : 1.0 / 36.0;
    if (M == 1) return q <= 1 ? 1.0 / 18.0 : 1.0 / 36.0;
    return q == 0 ? 1.0 / 18.0 : 1.0 / 36.0;
}
// f(integral_constant<int, m>) for m = 0 .. 4
template <typename F>
__device__ __forceinline__ void for_quad_dirs(F &&f) {
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{});
}

// sum over the quad, the same bits in its four lanes
__device__ __forceinline__ int quad_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);
    return x;
}
__device__ __forceinline__ uint32_t quad_or(uint32_t x) {
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false);
    return x;
}
// the value of lane SRC of the quad
template <int SRC>
__device__ __forceinline__ float quad_bcast(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), SRC * 0x55, 0xf, 0xf, false));
}
template <int SRC>
__device__ __forceinline__ double quad_bcast(double x) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), SRC * 0x55, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), SRC * 0x55, 0xf, 0xf, false));
}

// sum of a node's 20 values (5 per lane) in the order of its directions, in
// every lane: lane 0 adds its five, lane 1 goes on from there, ...
__device__ __forceinline__ double chain_sum(const double (&v)[QM]) {
    double x = 0.0;
    auto five = [&] {
#pragma unroll
        for (int m = 0; m < QM; m++) x += v[m];
    };
    five();
    x = quad_bcast<0>(x);
    five();
    x = quad_bcast<1>(x);
    five();
    x = quad_bcast<2>(x);
    five();
    return quad_bcast<3>(x);
}

// Box node b of the box at org (edge S): its box coordinates and lattice
// position; false beyond the box, in a wall layer, or more than a period away: a
// diverging sphere may pass several periods in a step, and the steps queued behind
// that one still run (they find no node of it).
__host__ __device__ __forceinline__ bool box_node(int b, const int32_t *org, int S, const Geo &g, int (&bb)[3], int (&p)[3]) {
    const uint32_t ub = (uint32_t)b, uS = (uint32_t)S;
    const uint32_t row = ub / uS;
    bb[0] = (int)(ub - row * uS);
    bb[2] = (int)(row / uS);
    bb[1] = (int)(row - (uint32_t)bb[2] * uS);
    const int n3[3] = {g.nx, g.ny, g.nz};
    const bool w3[3] = {g.wx, g.wy, g.wz};
    bool in = bb[2] < S;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        int v = (int)((uint32_t)org[a] + (uint32_t)bb[a]);
        if (!w3[a]) v = v < 0 ? v + n3[a] : (v >= n3[a] ? v - n3[a] : v);
        in = in && (uint32_t)v < (uint32_t)n3[a];
        p[a] = v;
    }
    return in;
}

// lattice position p + c; false across a wall
__device__ __forceinline__ bool step_to(const int (&p)[3], const int (&c)[3], const Geo &g, int (&q)[3]) {
    bool ok = true;
    const int n3[3] = {g.nx, g.ny, g.nz};
    const bool w3[3] = {g.wx, g.wy, g.wz};
#pragma unroll
    for (int a = 0; a < 3; a++) {
        int v = p[a] + c[a];
        if (v < 0 || v >= n3[a]) {
            if (w3[a]) ok = false;
            v = v < 0 ? v + n3[a] : v - n3[a];
        }
        q[a] = v;
    }
    return ok;
}

// box index of box coordinates bb + c, -1 outside the box
__device__ __forceinline__ int box_at(const int (&bb)[3], const int (&c)[3], int S) {
    const int x = bb[0] + c[0], y = bb[1] + c[1], z = bb[2] + c[2];
    const bool in = (uint32_t)x < (uint32_t)S && (uint32_t)y < (uint32_t)S && (uint32_t)z < (uint32_t)S;
    return in ? (z * S + y) * S + x : -1;
}

// element offset, from the node's own row (slot 0 at its x), of the slot it
// pulls direction d from (component A): pull_slot with a direction per lane
__device__ __forceinline__ int pull_off(int x, const QDir &d, const Geo &g) {
    const int sx = x - d.c[0];
    const bool out = sx < 0 || sx >= g.nx;
    const int wr = sx < 0 ? g.nx : (out ? -g.nx : 0);
    const int off = d.s * g.nx - d.c[1] * row_stride(g) - d.c[2] * plane_stride(g) - d.c[0] + wr;
    return (out && g.wx) ? d.so * g.nx : off;
}

// Sum of 64 numbers v[0 .. 63] by the 16 threads s = 0 .. 15 of a DPP row, as
// the balanced tree of neighbouring pairs (the tree of wave_sum); the result is
// in each of them.
__device__ __forceinline__ double row_sum64(const double *v, int s) {
    double x = (v[4 * s] + v[4 * s + 1]) + (v[4 * s + 2] + v[4 * s + 3]);
    x = dpp_add<0xB1>(x);
    x = dpp_add<0x4E>(x);
    x = dpp_add<0x141>(x);
    return dpp_add<0x140>(x);
}

// =============================================================== k_links
// Four lanes per node of the box of X^n.  A node p fluid at X^n with links
// to the sphere (p + c_i a particle node) applies the moving-wall
// bounce-back f_opp(i)(p) = f*_i(p) - 6 w_i rho_l(p) (c_i . u_b), u_b the
// rigid velocity at the link midpoint, and writes it into the slot p pulls
// from (opp(i) at p + c_i) for the next step; it sums the exchanged momentum
// sum_l (2 f*_i - 6 w_i rho_l c_i . u_b) c_i and its torque about X^n, the
// bounce-back mass flux and the reaction of the wetting layer on the sphere.
// Every fluid node near the sphere then forms its step-(n+1) populations
// (plain pulls, its own bounced values on links) and stores their densities
// and momentum for the particle kernel, which reads them within sqrt(2) of
// particle nodes at X^n or X^{n+1} (|U| < 1/2 per axis): nodes beyond R + 3 do
// nothing.  Particle nodes are read from the flags k_particle left.
// Every load is issued before the first is used (no load depends on a flag).
template <typename S, typename T>
__global__ __launch_bounds__(K3_THREADS) void k_links(LinkArgs a) {
    __shared__ double red[15 * K3_NODES];
    const int r = find_rep(a.k3_begin, a.nrep, blockIdx.x);
    const RepDesc &D = a.desc[r];
    const RepState &st = a.state[r];
    if (!D.has_particle) return;
    const Geo g = geo_of(D);
    const int t = threadIdx.x, q = t & 3;
    const int local = blockIdx.x - D.k3_begin;
    const int Sx = D.S, S3 = Sx * Sx * Sx;
    const int32_t org[3] = {st.org[0], st.org[1], st.org[2]};
    const double X[3] = {st.X[0], st.X[1], st.X[2]}, U[3] = {st.U[0], st.U[1], st.U[2]};
    const double W[3] = {st.W[0], st.W[1], st.W[2]};
    const double dlt[2] = {st.delta[0], st.delta[1]};
    const double rho0[2] = {D.rho0[0], D.rho0[1]};
    const double *vrho = a.vrho + D.bbox_off * 2;
    const double *rho_n = a.rho_n + D.bbox_off * 2;
    const uint32_t *pmask = a.pmask + D.bbox_off;
    double *raw = a.raw + D.bbox_off * RAW;
    S *buf = reinterpret_cast<S *>(a.buf) + D.pop_off;
    const int b = local * K3_NODES + (t >> 2);
    int bb[3], p[3];
    const bool in = box_node(b, org, Sx, g, bb, p);
    const double dd[3] = {sepd(p[0] - X[0], g.nx, g.wx), sepd(p[1] - X[1], g.ny, g.wy),
                          sepd(p[2] - X[2], g.nz, g.wz)};
    const double far = D.radius + 3.0;
    const bool near = in && dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2] < far * far;
    double vec[3] = {0.0, 0.0, 0.0}, mass[2] = {0.0, 0.0};
    int nlinks = 0;
    bool solid = false;
    if (near) {
        const int64_t own = slot_at(p[0], p[1], p[2], 0, g);
        const S *row = buf + own;
        const double rl[2] = {rho_n[b], rho_n[S3 + b]}, vw[2] = {vrho[b], vrho[S3 + b]};
        solid = pmask[b] & MASK_SOLID;
        // per direction i of this lane: the neighbour p + c_i, the population pulled
        // from it (direction opp(i)) and the node's own post-collision value
        // leaving along c_i
        S dv[2][QM], fv[2][QM];
        uint32_t pm[QM];
        double rn[2][QM];             // densities of the neighbours
        bool ok[QM];
        for_quad_dirs([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const QDir d = quad_dir<m>(q);
            const int off = d.i < Q ? pull_off(p[0], against(d), g) : 0;
            const int ownoff = d.s * g.nx;
            int np[3];
            const int nbi = box_at(bb, d.c, Sx);
            ok[m] = d.valid && nbi >= 0 && step_to(p, d.c, g, np);
            const int nb = nbi >= 0 ? nbi : b;
#pragma unroll
            for (int l = 0; l < 2; l++) {
                dv[l][m] = row[off + l * d.n * g.nx];
                fv[l][m] = row[ownoff + l * d.n * g.nx];
                rn[l][m] = rho_n[l * S3 + nb];
            }
            pm[m] = pmask[nb];
        });
        // rigid velocity at the link midpoint p + c_i/2: c_i . u_b = c_i . (U + W x d)
        // with d = p - X, since c_i . (W x c_i) = 0; the torque of the summed
        // link momentum P about X is d x P for the same reason
        const double V[3] = {U[0] + W[1] * dd[2] - W[2] * dd[1], U[1] + W[2] * dd[0] - W[0] * dd[2],
                             U[2] + W[0] * dd[1] - W[1] * dd[0]};
        T v[2][QM];                   // population opp(i) of step n + 1
        double mx[3][QM], mf[2][QM];  // momentum along c_i, mass flux
        for_quad_dirs([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const QDir d = quad_dir<m>(q);
            const double w = quad_w<m>(q);
            const bool sn = ok[m] && (pm[m] & MASK_SOLID);
            double amp = 0.0;
            mf[0][m] = mf[1][m] = 0.0;
#pragma unroll
            for (int l = 0; l < 2; l++)
                v[l][m] = ld_dev<S, T>(&dv[l][m], Rel<S>::value ? T(w) * T(rho0[l]) : T(1));
            if (sn && !solid) {  // link
                const double cu = d.c[0] * V[0] + d.c[1] * V[1] + d.c[2] * V[2];
                S *to = buf + own + pull_off(p[0], against(d), g);
#pragma unroll
                for (int l = 0; l < 2; l++) {
                    const double wr = w * rho0[l];
                    const double fs = wr + (double)ld_dev<S, T>(&fv[l][m], Rel<S>::value ? T(wr) : T(1));
                    const double corr = 6.0 * w * rl[l] * cu;
                    amp += 2.0 * fs - corr;
                    mf[l][m] = -corr;
                    S sv;
                    v[l][m] = store_round<S, T>(fs - corr - wr, Rel<S>::value ? T(1.0 / wr) : T(1),
                                                Rel<S>::value ? T(w) * T(rho0[l]) : T(1), sv);
                    to[l * d.n * g.nx] = sv;
                }
                nlinks++;
            }
            if (solid && ok[m] && !sn) {
                // reaction of the wetting layer: the Shan-Chen force on the fluid
                // neighbour x = s + c is -sw c (sw = -G w rho_l(x) rho~_l'(s)); its torque
                // about X is d_s x (-sw c)
                amp = D.G * w * (rn[0][m] * (vw[1] + dlt[1]) + rn[1][m] * (vw[0] + dlt[0]));
            }
#pragma unroll
            for (int x = 0; x < 3; x++) mx[x][m] = amp * d.c[x];
        });
#pragma unroll
        for (int x = 0; x < 3; x++) vec[x] = chain_sum(mx[x]);
        mass[0] = chain_sum(mf[0]);
        mass[1] = chain_sum(mf[1]);
        if (!solid) {
            // densities and momentum of step n+1, the populations taken from the
            // quad's lanes in the order node_moments adds them
            double mo[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int l = 0; l < 2; l++) {
                T rd = T(0), j[3] = {T(0), T(0), T(0)};
#pragma unroll
                for (int i = 0; i < Q; i++) {
                    const int from = opp(i) / QM;  // the lane that holds population i
                    const T x = v[l][opp(i) % QM];
                    const T u = from == 0 ? quad_bcast<0>(x) : from == 1 ? quad_bcast<1>(x)
                              : from == 2 ? quad_bcast<2>(x) : quad_bcast<3>(x);
                    rd += u;
                    if (cx(i) > 0) j[0] += u; else if (cx(i) < 0) j[0] -= u;
                    if (cy(i) > 0) j[1] += u; else if (cy(i) < 0) j[1] -= u;
                    if (cz(i) > 0) j[2] += u; else if (cz(i) < 0) j[2] -= u;
                }
                mo[l] = rho0[l] + (double)rd;
#pragma unroll
                for (int x = 0; x < 3; x++) mo[2 + x] += (double)j[x];
            }
            raw[q * S3 + b] = q == 0 ? mo[0] : q == 1 ? mo[1] : q == 2 ? mo[2] : mo[3];
            if (q == 0) raw[4 * S3 + b] = mo[4];
        }
    }
    nlinks = quad_sum(nlinks);
    {
        // lane q of the quad writes its quarter of the node's 15 values
        const double tq[3] = {dd[1] * vec[2] - dd[2] * vec[1], dd[2] * vec[0] - dd[0] * vec[2],
                              dd[0] * vec[1] - dd[1] * vec[0]};
        double *c = red + (t >> 2);
        if (q < 3) {
            const double f = q == 0 ? vec[0] : q == 1 ? vec[1] : vec[2];
            const double m = near ? (q == 0 ? tq[0] : q == 1 ? tq[1] : tq[2]) : 0.0;
            c[q * 64] = solid ? 0.0 : f;
            c[(3 + q) * 64] = solid ? 0.0 : m;
            c[(8 + q) * 64] = solid ? f : 0.0;
            c[(11 + q) * 64] = solid ? m : 0.0;
        } else {
            c[6 * 64] = mass[0];
            c[7 * 64] = mass[1];
            c[14 * 64] = (double)nlinks;
        }
    }
    __syncthreads();
    const double s = row_sum64(red + (t < 240 ? t >> 4 : 0) * 64, t & 15);
    if (t < 240 && (t & 15) == 0) a.part1[D.part3_off + (int64_t)local * PART + (t >> 4)] = s;
}

// ============================================================ k_particle
// Four lanes per node of the box of X^{n+1}.  Every workgroup sums the link
// partials (fixed order) and advances the sphere: leap-frog Newton-Euler under
// F = links - wetting reaction + F_ext + pending event momentum.  Each node
// then takes its flag at X^{n+1} (the FP64 predicate; the flags at X^n are the
// ones the last step left), and
//  * covered (fluid at X^n, particle at X^{n+1}): adds its momentum and
//    mass to the event sums;
//  * uncovered (particle at X^n, fluid at X^{n+1}): gets f_eq(rho_bar, u_b)
//    written into the slots it pulls from, rho_bar the mean density of its
//    neighbours fluid at both times;
//  * particle node at X^{n+1}: gets the wetting-layer density, mean of its
//    fluid neighbours +/- Delta rho (the mass correction delta is added
//    where it is read).
// Each workgroup leaves its event sums as a partial.  The last one to finish
// (per fluid) combines them, with the global mass correction and the new state
// of step n+1.  The partials go out as device-scope stores and come back as
// device-scope loads, each workgroup waiting for its own before it counts
// itself: a release fence instead writes back the L2 of its XCD (2-3 us, and
// with thousands of workgroups more than a separate launch).

// Motion of step n+1 of one sphere, in LDS.
struct Motion {
    double F[3], Tq[3], Un[3], Wn[3], Xn[3];
    int org[3];
};

// Scratch of a box workgroup: link sums, motion, event totals.
struct BoxShared {
    double grp[16][16];
    double sum[16];
    double tot[20];
    uint32_t evw[64];      // workgroups with events, a window of 2048
    double cnt[K3_THREADS / 64];
    Motion mo;
    int32_t org[MAX_GROUP][3];
    int last;
};

// Link sums of one sphere (15 values) into sh.sum, the order of sum_partials:
// column l = 0 .. 63 adds partials l, l + 64, ..., then the balanced tree over
// the columns (thread t: value t % 16, columns 4 (t / 16) .. + 3).  Ends with a
// barrier.
__device__ __forceinline__ void link_sums(const double *part1, int count, BoxShared &sh, int t) {
    const int k = t & 15, gq = t >> 4;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (k < 15) {
        const double *p = part1 + (int64_t)(4 * gq) * PART + k;
        for (int w = 4 * gq; w < count; w += 192, p += 192 * PART) {
            double c[3][4];
#pragma unroll
            for (int m = 0; m < 3; m++)
#pragma unroll
                for (int j = 0; j < 4; j++) c[m][j] = w + 64 * m + j < count ? p[(64 * m + j) * PART] : 0.0;
#pragma unroll
            for (int m = 0; m < 3; m++)
#pragma unroll
                for (int j = 0; j < 4; j++) s[j] += c[m][j];
        }
    }
    __syncthreads();  // earlier readers of sh.grp are done
    sh.grp[gq][k] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    if (t < 15) {
        double v[16];
#pragma unroll
        for (int j = 0; j < 16; j++) v[j] = sh.grp[j][t];
#pragma unroll
        for (int h = 1; h < 16; h *= 2)
#pragma unroll
            for (int j = 0; j < 16; j += 2 * h) v[j] += v[j + h];
        sh.sum[t] = v[0];
    }
    __syncthreads();
}

// Leap-frog Newton-Euler step of one sphere from the link sums of step n
// (momentum exchange minus wetting-layer reaction, plus F_ext and the
// pending event momentum), and the bounding-box origin of X^{n+1}: one thread
// per axis.  Every caller evaluates it on the same inputs, so all agree
// bitwise.  Ends with a barrier.
struct Axis {  // what it reads of one axis; loaded before the link sums
    double X, U, W, Fext, Pev, Lev, mp, Ip;
};
__device__ __forceinline__ Axis axis_of(const RepDesc &D, const RepState *st, int t) {
    const int x = t < 3 ? t : 0;
    return {st->X[x], st->U[x], st->W[x], D.Fext[x], st->Pev[x], st->Lev[x], D.mp, D.Ip};
}
__device__ __forceinline__ void newton_euler(const RepDesc &D, const Axis &ax, const Geo &g, BoxShared &sh, int t) {
    if (t < 3) {
        const double (&sum)[16] = sh.sum;
        const int n = t == 0 ? g.nx : t == 1 ? g.ny : g.nz;
        const bool wall = t == 0 ? g.wx : t == 1 ? g.wy : g.wz;
        const double U = ax.U, W = ax.W;
        const double F = sum[t] - sum[8 + t] + ax.Fext + ax.Pev;
        const double Tq = sum[3 + t] - sum[11 + t] + ax.Lev;
        const double Un = D.fixed_velocity ? U : U + F / ax.mp;
        double Xn = ax.X + Un;
        if (!wall) {
            if (Xn >= n) Xn -= n;
            else if (Xn < 0.0) Xn += n;
        }
        sh.mo.F[t] = F;
        sh.mo.Tq[t] = Tq;
        sh.mo.Un[t] = Un;
        sh.mo.Wn[t] = D.fixed_velocity ? W : W + Tq / ax.Ip;
        sh.mo.Xn[t] = Xn;
        sh.mo.org[t] = box_start(Xn - D.radius);  // box of X^{n+1}
    }
    __syncthreads();
}

// device-scope access to the event partials (see above)
__device__ __forceinline__ void put_dev(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_dev(const double *p) {
    return __hip_atomic_load(const_cast<double *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Event totals of one sphere into sh.tot, the order of sum_partials.  Slot 9
// (particle nodes) and slot 20 (events in this workgroup) are in every partial;
// the other slots are read from the workgroups that had events and are zero
// elsewhere (adding zero changes nothing).  col: 20 x 64 columns.  Ends with a
// barrier.
__device__ __forceinline__ void event_totals(const double *part3, int count, BoxShared &sh, double *col, int t) {
    double cnt = 0.0;
    bool any = false;
    __syncthreads();
    for (int w0 = 0; w0 < count; w0 += 2048) {
        if (t < 64) sh.evw[t] = 0u;
        __syncthreads();
        bool mine = false;
        for (int w = w0 + t; w < min(count, w0 + 2048); w += K3_THREADS) {
            cnt += get_dev(part3 + (int64_t)w * PART + 9);
            if (get_dev(part3 + (int64_t)w * PART + 20) != 0.0) {
                atomicOr(&sh.evw[(w - w0) >> 5], 1u << ((w - w0) & 31));
                mine = true;
            }
        }
        if (!__syncthreads_or(mine)) continue;
        if (!any)
            for (int e = t; e < 20 * 64; e += K3_THREADS) col[e] = 0.0;
        any = true;
        __syncthreads();
        if (t < 64)  // words with a bit set, in ascending order
            for (uint64_t words = __ballot(sh.evw[t] != 0u); words; words &= words - 1) {
                const int k = __builtin_ctzll(words);
                for (uint32_t e = sh.evw[k]; e; e &= e - 1) {
                    const int w = w0 + 32 * k + __builtin_ctz(e);
                    if (t < 20 && t != 9) col[t * 64 + (w & 63)] += get_dev(part3 + (int64_t)w * PART + t);
                }
            }
        __syncthreads();
    }
    // whole numbers: exact in any order
    double c[1] = {cnt};
    wave_sum<1>(c);
    if ((t & 63) == 0) sh.cnt[t >> 6] = c[0];
    if (any) {
        const double a = row_sum64(col + (t >> 4) * 64, t & 15);
        const double b = row_sum64(col + (16 + ((t >> 4) & 3)) * 64, t & 15);
        if ((t & 15) == 0) sh.tot[t >> 4] = a;
        if ((t & 15) == 0 && t < 64) sh.tot[16 + (t >> 4)] = b;
    } else if (t < 20) {
        sh.tot[t] = 0.0;
    }
    __syncthreads();
    if (t == 0) sh.tot[9] = (sh.cnt[0] + sh.cnt[1]) + (sh.cnt[2] + sh.cnt[3]);
    __syncthreads();
}

// slot of step n in a U-series ring
__device__ __forceinline__ int64_t ring_slot(int64_t n, int cap) {
    return n < ((int64_t)1 << 31) ? (int64_t)((uint32_t)n % (uint32_t)cap) : n % cap;
}

// A replica without a sphere: record U = 0 and advance the step counter.
__device__ __forceinline__ void advance_empty(const ParticleArgs &a, const RepDesc &D, RepState *st) {
    const int64_t n = st->step;
    double *s = a.series + D.series_off + 3 * ring_slot(n, D.series_cap);
    s[0] = s[1] = s[2] = 0.0;
    st->delta[0] = st->delta[1] = 0.0;
    st->step = n + 1;
}

// Motion of step n+1 of one sphere (threads 0 .. 2, one per axis): position,
// velocities, forces, bounding-box origin, pending event momentum, the U series
// entry and (thread 0) the event counters.  Returns in each of these threads
// whether the sphere went unstable (|U| >= 1/2, a non-finite force) or reached a
// wall on its axis.
__device__ __forceinline__ bool publish_motion(const ParticleArgs &a, const RepDesc &D, RepState *st, const Geo &g,
                                               const BoxShared &sh, int t) {
    if (t >= 3) return false;
    const Motion &mo = sh.mo;
    const int64_t n = st->step;
    const int nn = t == 0 ? g.nx : t == 1 ? g.ny : g.nz;
    const bool wall = t == 0 ? g.wx : t == 1 ? g.wy : g.wz;
    const double Xold = st->X[t];
    st->Xp[t] = Xold;
    st->X[t] = mo.Xn[t];
    st->U[t] = mo.Un[t];
    st->W[t] = mo.Wn[t];
    st->F[t] = mo.F[t];
    st->T[t] = mo.Tq[t];
    st->Pev[t] = sh.tot[t] - sh.tot[10 + t];
    st->Lev[t] = sh.tot[3 + t] - sh.tot[13 + t];
    st->org[t] = mo.org[t];
    a.series[D.series_off + 3 * ring_slot(n, D.series_cap) + t] = mo.Un[t];
    if (t == 2) st->uz_sum += mo.Un[2];
    if (t == 0) {
        st->n_cov += (int64_t)sh.tot[8];
        st->n_unc += (int64_t)sh.tot[18];
        st->n_links = (int64_t)sh.sum[14];
    }
    return !(fabs(mo.Un[t]) < 0.5) || !isfinite(mo.F[t]) ||
           (wall && (mo.Xn[t] - D.radius < -0.5 || mo.Xn[t] + D.radius > nn - 0.5));
}

// Publish step n+1 of one replica with a single sphere from the link sums,
// the motion and the event totals (one workgroup): global mass correction
// delta_l = -(bounce-back flux - covered + uncovered mass)_l / |Phi^{n+1}|,
// then the sphere's motion, the step counter and the stability flag.
__device__ __forceinline__ void publish_step(const ParticleArgs &a, const RepDesc &D, RepState *st, const Geo &g,
                                             const BoxShared &sh, int t) {
    if (t >= 64) return;
    const double nf = (double)D.N - sh.tot[9];
    const bool bad = publish_motion(a, D, st, g, sh, t);
    const bool any = __any(bad);
    if (t < 2) st->delta[t] = -(sh.sum[6 + t] - sh.tot[6 + t] + sh.tot[16 + t]) / nf;
    if (t == 0) {
        st->n_fluid = nf;
        if (any) st->flags |= FLAG_UNSTABLE;
        st->step = st->step + 1;
        st->k3_done = 0;
    }
}

// Publish step n+1 of a group of spheres in one fluid (one workgroup).  The
// mass correction is global: the bounce-back, covered and uncovered fluxes and
// the particle nodes of every sphere are summed before delta_l and |Phi^{n+1}|
// are formed.  Each sphere then takes its own Newton-Euler step, and every
// entry of the group receives the shared fields (delta, fluid nodes, step,
// flags).  Two boxes that now share a node set FLAG_CONTACT on the group.
__device__ __forceinline__ void publish_group(const ParticleArgs &a, int prim, const Geo &g, BoxShared &sh,
                                              double *col, int t) {
    const RepDesc *P = a.desc + prim;
    const int K = P->n_sph;
    double dm[2] = {0.0, 0.0}, nsol = 0.0;
    uint32_t flags = 0u;
    for (int e = prim; e < prim + K; e++) {
        const RepDesc &De = a.desc[e];
        RepState *se = a.state + e;
        flags |= se->flags;
        const Axis ax = axis_of(De, se, t);
        link_sums(a.part1 + De.part3_off, De.k3_count, sh, t);
        event_totals(a.part3 + De.part3_off, De.k3_count, sh, col, t);
        newton_euler(De, ax, g, sh, t);
        for (int l = 0; l < 2; l++) dm[l] += sh.sum[6 + l] - sh.tot[6 + l] + sh.tot[16 + l];
        nsol += sh.tot[9];
        if (t < 64) {
            const bool bad = publish_motion(a, De, se, g, sh, t);
            if (__any(bad)) flags |= FLAG_UNSTABLE;
        }
        if (t < 3) sh.org[e - prim][t] = sh.mo.org[t];
    }
    __syncthreads();
    if (t != 0) return;
    const double nf = (double)P->N - nsol;
    const int32_t n3[3] = {g.nx, g.ny, g.nz};
    for (int e = 0; e < K; e++)
        for (int f = e + 1; f < K; f++)
            if (boxes_overlap(sh.org[e], a.desc[prim + e].S, sh.org[f], a.desc[prim + f].S, n3, P->walls))
                flags |= FLAG_CONTACT;
    const int64_t step = a.state[prim].step + 1;
    for (int e = prim; e < prim + K; e++) {
        RepState *se = a.state + e;
        se->delta[0] = -dm[0] / nf;
        se->delta[1] = -dm[1] / nf;
        se->n_fluid = nf;
        se->flags = flags;
        se->step = step;
    }
    a.state[prim].k3_done = 0;
}

template <typename S, typename T>
__global__ __launch_bounds__(K3_THREADS) void k_particle(ParticleArgs a) {
    __shared__ BoxShared sh;
    __shared__ double ev[20 * K3_NODES];
    const int r = find_rep(a.k3_begin, a.nrep, blockIdx.x);
    const RepDesc &D = a.desc[r];
    RepState *st = a.state + r;
    const int t = threadIdx.x, q = t & 3;
    const int local = blockIdx.x - D.k3_begin;
    if (!D.has_particle) {
        if (t == 0) advance_empty(a, D, st);
        return;
    }
    const Geo g = geo_of(D);
    const int32_t orgo[3] = {st->org[0], st->org[1], st->org[2]};
    const Axis ax = axis_of(D, st, t);
    // 1. link momentum exchange and wetting-layer reaction of step n
    link_sums(a.part1 + D.part3_off, D.k3_count, sh, t);
    // 2. Newton-Euler, leap-frog
    newton_euler(D, ax, g, sh, t);
    const double Xn[3] = {sh.mo.Xn[0], sh.mo.Xn[1], sh.mo.Xn[2]};
    const int org[3] = {sh.mo.org[0], sh.mo.org[1], sh.mo.org[2]};
    const int Sx = D.S, S3 = Sx * Sx * Sx;
    const double *raw = a.raw + D.bbox_off * RAW;
    double *vrho = a.vrho + D.bbox_off * 2;
    const uint32_t *pold = a.pmask_old + D.bbox_off;
    uint32_t *pnew = a.pmask + D.bbox_off;
    S *buf = reinterpret_cast<S *>(a.buf) + D.pop_off;

    // 3. events and wetting layer
    const int b = local * K3_NODES + (t >> 2);
    int bb[3], p[3];
    const bool in = box_node(b, org, Sx, g, bb, p);
    // box coordinates in the box of X^n
    int bo[3];
    const int n3[3] = {g.nx, g.ny, g.nz};
    const bool w3[3] = {g.wx, g.wy, g.wz};
#pragma unroll
    for (int x = 0; x < 3; x++) {
        int s = org[x] - orgo[x];
        if (!w3[x]) s = 2 * s > n3[x] ? s - n3[x] : (2 * s < -n3[x] ? s + n3[x] : s);
        bo[x] = bb[x] + s;
    }
    const int zero[3] = {0, 0, 0};
    const int ob = box_at(bo, zero, Sx);
    const bool so = in && ob >= 0 && (pold[ob < 0 ? 0 : ob] & MASK_SOLID);  // particle node at X^n
    const bool sn = in && pnode(p[0], p[1], p[2], Xn, D.R2, g);             // at X^{n+1}
    const bool unc = so && !sn, cov = in && !so && sn;

    // neighbours of lattice node c (old-box coordinates cb) along this lane's
    // directions that are fluid at X^{n+1}: those fluid at X^n too (kept) and
    // those uncovered now (fresh), as bits m; their post-streaming densities are
    // loaded beside the flags (meaningful for kept ones only)
    auto flags_of = [&](const int (&c)[3], const int (&cb)[3], uint32_t &kept, uint32_t &fresh, double (&v)[2][QM]) {
        kept = fresh = 0u;
        uint32_t pm[QM];
        int idx[QM];
        for_quad_dirs([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const QDir d = quad_dir<m>(q);
            idx[m] = d.valid ? box_at(cb, d.c, Sx) : -1;
            const int at = idx[m] < 0 ? 0 : idx[m];
            pm[m] = pold[at];
            v[0][m] = raw[at];
            v[1][m] = raw[S3 + at];
        });
        for_quad_dirs([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const QDir d = quad_dir<m>(q);
            int np[3];
            if (!d.valid || !step_to(c, d.c, g, np) || pnode(np[0], np[1], np[2], Xn, D.R2, g)) return;
            if (idx[m] < 0) return;
            if (pm[m] & MASK_SOLID) fresh |= 1u << m;
            else kept |= 1u << m;
        });
    };
    // sums of the kept neighbours' densities, in the four lanes of the quad
    auto sum_kept = [&](uint32_t kept, const double (&v)[2][QM], double (&s)[2]) {
#pragma unroll
        for (int l = 0; l < 2; l++) {
            double x[QM];
#pragma unroll
            for (int m = 0; m < QM; m++) x[m] = (kept >> m) & 1u ? v[l][m] : 0.0;
            s[l] = chain_sum(x);
        }
    };
    // their mean (rho0 when there is none): the density of an uncovered node
    auto mean_kept = [&](uint32_t kept, const double (&v)[2][QM], double (&m2)[2]) {
        sum_kept(kept, v, m2);
        const int cnt = quad_sum(__builtin_popcount(kept));
#pragma unroll
        for (int l = 0; l < 2; l++) m2[l] = cnt > 0 ? m2[l] / cnt : D.rho0[l];
    };
    uint32_t kept = 0, fresh = 0;
    double v[2][QM];
    const bool work = sn || unc;  // the same in the four lanes of a quad
    if (work) flags_of(p, bo, kept, fresh, v);
    double self[2] = {0.0, 0.0};
    if (unc) mean_kept(kept, v, self);
    // Densities of a particle node's fresh neighbours: each is the mean over that
    // neighbour's own kept neighbours, formed by the whole quad.
    double fs[2] = {0.0, 0.0};
    if (sn && quad_or(fresh)) {
        // (in the order of the directions)
#pragma unroll 1
        for (int s = 0; s < 4; s++) {
            if (!quad_or(q == s ? fresh : 0u)) continue;
#pragma unroll 1
            for (int m = 0; m < QM; m++) {
                // lane s's direction 5 s + m of the quad's node, in every lane of the quad
                const int i = QM * s + m;
                const bool has = quad_or(q == s ? (fresh >> m) & 1u : 0u) != 0u;
                if (!has) continue;
                const int c[3] = {cx(i), cy(i), cz(i)};
                int np[3], nb[3];
                step_to(p, c, g, np);
#pragma unroll
                for (int x = 0; x < 3; x++) nb[x] = bo[x] + c[x];
                uint32_t k2, f2;
                double v2[2][QM], m2[2];
                flags_of(np, nb, k2, f2, v2);
                mean_kept(k2, v2, m2);
                fs[0] += m2[0];
                fs[1] += m2[1];
            }
        }
    }
    if (sn) {
        // wetting layer: mean density of the neighbours fluid at X^{n+1}
        double s[2];
        sum_kept(kept, v, s);
        const double s0 = s[0] + fs[0], s1 = s[1] + fs[1];
        const int cnt = quad_sum(__builtin_popcount(kept | fresh));
        if (q == 0) vrho[b] = cnt > 0 ? s0 / cnt + D.drho : 0.0;
        if (q == 1) vrho[S3 + b] = cnt > 0 ? s1 / cnt - D.drho : 0.0;
    }
    if (q == 0 && b < S3) pnew[b] = sn ? MASK_SOLID : 0u;
    const int nsolid = __syncthreads_count(sn && q == 0);
    const bool events = __syncthreads_or(unc || (cov && ob >= 0));
    double *pp = a.part3 + D.part3_off + (int64_t)local * PART;
    if (events) {
        if (unc) {  // f_eq of its neighbours' mean density and u_b
            const double rr[3] = {sepd(p[0] - Xn[0], g.nx, g.wx), sepd(p[1] - Xn[1], g.ny, g.wy),
                                  sepd(p[2] - Xn[2], g.nz, g.wz)};
            const double *Un = sh.mo.Un, *Wn = sh.mo.Wn;
            const double u[3] = {Un[0] + Wn[1] * rr[2] - Wn[2] * rr[1], Un[1] + Wn[2] * rr[0] - Wn[0] * rr[2],
                                 Un[2] + Wn[0] * rr[1] - Wn[1] * rr[0]};
            const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
            S *row = buf + slot_at(p[0], p[1], p[2], 0, g);
            for_quad_dirs([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                const QDir d = quad_dir<m>(q);
                if (d.i >= Q) return;
                const double w = quad_w<m>(q);
                const double cu = d.c[0] * u[0] + d.c[1] * u[1] + d.c[2] * u[2];
                const double e = 1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu;
                S *to = row + pull_off(p[0], d, g);
#pragma unroll
                for (int l = 0; l < 2; l++) {
                    const double wr = w * D.rho0[l];
                    st_dev<S, T>(to + l * d.n * g.nx, T(w * self[l] * e - wr), Rel<S>::value ? T(1.0 / wr) : T(1));
                }
            });
        }
        if (q == 0) {
            double o[20];
#pragma unroll
            for (int k = 0; k < 20; k++) o[k] = 0.0;
            if (unc || (cov && ob >= 0)) {
                const double rr[3] = {sepd(p[0] - Xn[0], g.nx, g.wx), sepd(p[1] - Xn[1], g.ny, g.wy),
                                      sepd(p[2] - Xn[2], g.nz, g.wz)};
                double j[3], m2[2];
                if (cov) {
                    for (int x = 0; x < 3; x++) j[x] = raw[(2 + x) * S3 + ob];
                    m2[0] = raw[ob];
                    m2[1] = raw[S3 + ob];
                } else {
                    const double *Un = sh.mo.Un, *Wn = sh.mo.Wn;
                    const double tot = self[0] + self[1];
                    j[0] = tot * (Un[0] + Wn[1] * rr[2] - Wn[2] * rr[1]);
                    j[1] = tot * (Un[1] + Wn[2] * rr[0] - Wn[0] * rr[2]);
                    j[2] = tot * (Un[2] + Wn[0] * rr[1] - Wn[1] * rr[0]);
                    m2[0] = self[0];
                    m2[1] = self[1];
                }
                const double e9[9] = {j[0], j[1], j[2], rr[1] * j[2] - rr[2] * j[1], rr[2] * j[0] - rr[0] * j[2],
                                      rr[0] * j[1] - rr[1] * j[0], m2[0], m2[1], 1.0};
#pragma unroll
                for (int k = 0; k < 9; k++) {
                    o[k] = cov ? e9[k] : 0.0;
                    o[10 + k] = cov ? 0.0 : e9[k];
                }
            }
#pragma unroll
            for (int k = 0; k < 20; k++) ev[k * K3_NODES + (t >> 2)] = o[k];
        }
        __syncthreads();
        // rows 0 .. 15, then 16 .. 19
        double s = row_sum64(ev + (t >> 4) * K3_NODES, t & 15);
        if ((t & 15) == 0 && (t >> 4) != 9) put_dev(pp + (t >> 4), s);
        s = row_sum64(ev + (16 + ((t >> 4) & 3)) * K3_NODES, t & 15);
        if (t < 64 && (t & 15) == 0) put_dev(pp + 16 + (t >> 4), s);
    }
    if (t == 0) {
        put_dev(pp + 9, (double)nsolid);
        put_dev(pp + 20, events ? 1.0 : 0.0);
    }
    // the partials have left for device-visible memory before the count below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // the counter of the group's primary entry counts the workgroups of every
    // sphere in the fluid (a single sphere: its own)
    RepState *sp = a.state + D.primary;
    if (t == 0)
        sh.last = __hip_atomic_fetch_add(&sp->k3_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                  (unsigned)(D.k3_total - 1);
    __syncthreads();
    if (!sh.last) return;
    // the next launch sees the stores below: kernel boundaries order them
    if (D.n_sph > 1) {
        publish_group(a, D.primary, g, sh, ev, t);
        return;
    }
    // last workgroup: event sums (fixed order), then the new state
    event_totals(a.part3 + D.part3_off, D.k3_count, sh, ev, t);
    publish_step(a, D, st, g, sh, t);
}

// ================================================================ k_init
// f(0) = w_i rho_l(x) with rho_l = rho0_l + amp (2u - 1), u from Philox with
// counter (node, 0, 0, 1), word l, written into the slots x pulls from; the
// planes z >= init_split (when set) start from the swapped pair rho0_{1-l}.
template <typename S>
__global__ __launch_bounds__(256) void k_init(InitArgs a) {
    __shared__ double red[4 * 2];
    const int wg = blockIdx.x;
    const int r = find_rep(a.init_begin, a.nrep, wg);
    const RepDesc &D = a.desc[r];
    const Geo g = geo_of(D);
    const int64_t n = (int64_t)(wg - a.init_begin[r]) * 256 + threadIdx.x;
    double m[2] = {0.0, 0.0};
    if (n < g.N) {
        const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny);
        const int z = (int)(n / ((int64_t)g.nx * g.ny));
        bool solid = false;  // inside any sphere of the replica
        for (int e = r; e < r + D.n_sph; e++)
            solid = solid || (a.desc[e].has_particle && pnode(x, y, z, a.state[e].X, a.desc[e].R2, g));
        uint32_t c0 = (uint32_t)n, c1 = 0u, c2 = 0u, c3 = 1u;
        philox4x32_10(c0, c1, c2, c3, D.key0, D.key1);
        const uint32_t w[2] = {c0, c1};
        S *dst = reinterpret_cast<S *>(a.buf) + D.pop_off;
        const bool swap = D.init_split > 0 && z >= D.init_split;  // other phase above the split
        for (int l = 0; l < 2; l++) {
            const double base = swap ? D.rho0[1 - l] : D.rho0[l];
            const double rho = base + D.init_amp * (2.0 * (((double)w[l] + 0.5) * 0x1p-32) - 1.0);
            if (solid) continue;
            m[l] = rho;
            for (int i = 0; i < Q; i++) {
                const double wr = wgt(i) * D.rho0[l];
                st_dev<S, double>(dst + pull_slot(x, y, z, l, i, g),
                                  wgt(i) * rho - wr, Rel<S>::value ? 1.0 / wr : 1.0);
            }
        }
    }
    block_sum<256, 2>(m, red);
    if (threadIdx.x == 0) {
        a.mass[2 * wg] = m[0];
        a.mass[2 * wg + 1] = m[1];
    }
}

// The entry of the group of primary entry prim whose sphere holds node
// (x, y, z) for the current step (b: its box index), or -1 for a fluid node.
__device__ __forceinline__ int solid_entry(int x, int y, int z, const RepDesc *desc, const RepState *state,
                                           const uint32_t *pmask, int prim, const Geo &g, int &b) {
    for (int e = prim; e < prim + desc[prim].n_sph; e++) {
        const RepDesc &D = desc[e];
        if (!D.has_particle) continue;
        b = bbox_index(x, y, z, state[e].org, D.S, g);
        if (b >= 0 && (pmask[D.bbox_off + b] & MASK_SOLID)) return e;
    }
    b = -1;
    return -1;
}

// ================================================================= k_ck
// Population part of a checkpoint: one array per component and direction over
// the lattice padded by one layer per side, population i of node x at padded
// position x - c_i, slot i; elements no node pulls from hold 0.  One thread per
// padded position, consecutive ones along x.
// Bound by HBM; the form is kept for checkpoints that outlive the process that
// wrote them.  All of a thread's loads are issued before its first store (the two
// buffers could be one for all the compiler knows, so that each store would
// otherwise hold up the next load), and each XCD takes a run of neighbouring
// blocks, whose ends share cache lines.  Save and restore, with their copies of the
// state and the wait: 192 x 192 x 512 FP16 1111 and 1130 us before, 708 and 752 now
// (583 for a copy of as many bytes); FP32 1375 and 1452, 1248 and 1278 (1190); 16 x
// 16 x 32 FP32 30.4 and 27.6, 26.6 and 24.4 (24.3 and 22.4).
template <typename S, bool SAVE>
__global__ __launch_bounds__(256) void k_ck(CkArgs a) {
    const int r = a.rep0 + blockIdx.y;
    const RepDesc &D = a.desc[r];
    const uint32_t k = (uint32_t)xcd_logical(blockIdx.x, gridDim.x) * 256u + threadIdx.x;  // ck_NP has 26 bits at most
    if (D.primary != r || k >= D.ck_NP) return;
    const Geo g = geo_of(D);
    const uint32_t row = k / (uint32_t)(g.nx + 2), plane = row / (uint32_t)(g.ny + 2);
    const int px = (int)(k - row * (uint32_t)(g.nx + 2)) - 1, py = (int)(row - plane * (uint32_t)(g.ny + 2)) - 1;
    const int pz = (int)plane - 1;
    S *pop = reinterpret_cast<S *>(a.pop) + D.pop_off;
    S *ck = reinterpret_cast<S *>(a.ck) + D.ck_off + k;
    S v[2][Q];
    uint32_t inside = 0;
#pragma unroll
    for (int i = 0; i < Q; i++) {
        const int x = px + cx(i), y = py + cy(i), z = pz + cz(i);
        const bool in = x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
        inside |= in ? 1u << i : 0u;
        const S *p = pop + (in ? pull_slot(x, y, z, 0, i, g) : 0);
#pragma unroll
        for (int l = 0; l < 2; l++)
            v[l][i] = SAVE ? p[l * SLOTS.n[i] * g.nx] : ck[(int64_t)(l * Q + i) * D.ck_NP];
    }
#pragma unroll
    for (int i = 0; i < Q; i++) {
        const bool in = inside >> i & 1u;
        S *p = pop + (in ? pull_slot(px + cx(i), py + cy(i), pz + cz(i), 0, i, g) : 0);
#pragma unroll
        for (int l = 0; l < 2; l++) {
            if constexpr (SAVE) ck[(int64_t)(l * Q + i) * D.ck_NP] = in ? v[l][i] : S(0);
            else if (in) p[l * SLOTS.n[i] * g.nx] = v[l][i];
        }
    }
}

// ============================================================= k_export
// f_{l i}(x, n) in FP64 for the nodes of planes [z_begin, z_end) of one
// replica (particle nodes: 0).
template <typename S, typename T>
__global__ __launch_bounds__(256) void k_export(ExportArgs a) {
    const RepDesc &D = a.desc[a.rep];
    const RepState &st = a.state[a.rep];
    const Geo g = geo_of(D);
    const int64_t plane = (int64_t)g.nx * g.ny;
    const int64_t cnt = plane * (a.z_end - a.z_begin);
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= cnt) return;
    const int x = (int)(k % g.nx), y = (int)((k / g.nx) % g.ny), z = a.z_begin + (int)(k / plane);
    const PullCtx<S, T> pc = pull_ctx<S, T>(a.src, D, g);
    int b;
    const bool solid = solid_entry(x, y, z, a.desc, a.state, a.pmask, D.primary, g, b) >= 0;
    T d[2][Q];
    if (!solid) pull_node(pc, x, y, z, d);
    for (int l = 0; l < 2; l++)
        for (int i = 0; i < Q; i++)
            a.out[(int64_t)(l * Q + i) * cnt + k] =
                solid ? 0.0 : wgt(i) * (D.rho0[l] + st.delta[l]) + (double)d[l][i];
}

// ============================================================= k_fields_a
// Density seen by the Shan-Chen force (wetting layer on particle nodes),
// total momentum and a solid flag per node, into scratch.
template <typename S, typename T>
__global__ __launch_bounds__(256) void k_fields_a(FieldArgs a) {
    const RepDesc &D = a.desc[a.rep];
    const RepState &st = a.state[a.rep];
    const Geo g = geo_of(D);
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= g.N) return;
    const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny);
    const int z = (int)(n / ((int64_t)g.nx * g.ny));
    double *rt = a.scratch, *jt = a.scratch + 2 * g.N, *sol = a.scratch + 8 * g.N;
    int b;
    const int e = solid_entry(x, y, z, a.desc, a.state, a.pmask, D.primary, g, b);
    if (e >= 0) {
        const int S3 = a.desc[e].S * a.desc[e].S * a.desc[e].S;
        const double *vrho = a.vrho + a.desc[e].bbox_off * 2;
        rt[n] = vrho[b] + st.delta[0];
        rt[g.N + n] = vrho[S3 + b] + st.delta[1];
        for (int q = 0; q < 3; q++) jt[q * g.N + n] = 0.0;
        sol[n] = 1.0;
        return;
    }
    const PullCtx<S, T> pc = pull_ctx<S, T>(a.src, D, g);
    T d[2][Q];
    pull_node(pc, x, y, z, d);
    double jtot[3] = {0.0, 0.0, 0.0};
    for (int l = 0; l < 2; l++) {
        T rd, jl[3], mm[Q];
        component_modes(d[l], rd, jl, mm);
        rt[l * g.N + n] = D.rho0[l] + st.delta[l] + (double)rd;
        for (int q = 0; q < 3; q++) jtot[q] += (double)jl[q];
    }
    for (int q = 0; q < 3; q++) jt[q * g.N + n] = jtot[q];
    sol[n] = 0.0;
}

// ============================================================== launchers
template <typename S, typename T, int B, bool GROUP>
void launch_main_b(const MainArgs &a, int grid, size_t lds, hipStream_t s) {
    if (a.tau1) {
        if (a.noise) hipLaunchKernelGGL((k_main<S, T, B, true, GROUP, true>), dim3(grid), dim3(B), lds, s, a);
        else hipLaunchKernelGGL((k_main<S, T, B, true, GROUP, false>), dim3(grid), dim3(B), lds, s, a);
    } else {
        if (a.noise) hipLaunchKernelGGL((k_main<S, T, B, false, GROUP, true>), dim3(grid), dim3(B), lds, s, a);
        else hipLaunchKernelGGL((k_main<S, T, B, false, GROUP, false>), dim3(grid), dim3(B), lds, s, a);
    }
}

template <typename S, typename T, bool GROUP>
hipError_t launch_main_g(const MainArgs &a, int grid, int block, size_t lds, hipStream_t s) {
    switch (block) {
    case 256: launch_main_b<S, T, 256, GROUP>(a, grid, lds, s); break;
    case 512: launch_main_b<S, T, 512, GROUP>(a, grid, lds, s); break;
    case 1024: launch_main_b<S, T, 1024, GROUP>(a, grid, lds, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename S, typename T>
hipError_t launch_main_t(const MainArgs &a, int grid, int block, size_t lds, hipStream_t s) {
    return a.groups ? launch_main_g<S, T, true>(a, grid, block, lds, s)
                    : launch_main_g<S, T, false>(a, grid, block, lds, s);
}

template <typename S, typename T>
hipError_t launch_links_t(const LinkArgs &a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((k_links<S, T>), dim3(grid), dim3(K3_THREADS), 0, s, a);
    return hipGetLastError();
}

template <typename S, typename T>
hipError_t launch_particle_t(const ParticleArgs &a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((k_particle<S, T>), dim3(grid), dim3(K3_THREADS), 0, s, a);
    return hipGetLastError();
}

template <typename S, typename T>
hipError_t launch_init_t(const InitArgs &a, int grid, hipStream_t s) {
    hipLaunchKernelGGL(k_init<S>, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename S, typename T>
hipError_t launch_export_t(const ExportArgs &a, int64_t count, hipStream_t s) {
    hipLaunchKernelGGL((k_export<S, T>), dim3((int)((count + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_ck_t(bool save, const CkArgs &a, int blocks, int nrep, hipStream_t s) {
    if (save) hipLaunchKernelGGL((k_ck<S, true>), dim3(blocks, nrep), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_ck<S, false>), dim3(blocks, nrep), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename S, typename T>
hipError_t launch_fields_a_t(const FieldArgs &a, int64_t N, hipStream_t s) {
    hipLaunchKernelGGL((k_fields_a<S, T>), dim3((int)((N + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

#define LBM_INSTANTIATE(SUFFIX, S, T)                                                              \
    hipError_t launch_main_##SUFFIX(const MainArgs &a, int grid, int block, size_t lds,          \
                                    hipStream_t s) {                                               \
        return launch_main_t<S, T>(a, grid, block, lds, s);                                        \
    }                                                                                              \
    hipError_t launch_links_##SUFFIX(const LinkArgs &a, int grid, hipStream_t s) {                 \
        return launch_links_t<S, T>(a, grid, s);                                                   \
    }                                                                                              \
    hipError_t launch_particle_##SUFFIX(const ParticleArgs &a, int grid, hipStream_t s) {          \
        return launch_particle_t<S, T>(a, grid, s);                                                \
    }                                                                                              \
    hipError_t launch_init_##SUFFIX(const InitArgs &a, int grid, hipStream_t s) {                  \
        return launch_init_t<S, T>(a, grid, s);                                                    \
    }                                                                                              \
    hipError_t launch_export_##SUFFIX(const ExportArgs &a, int64_t count, hipStream_t s) {         \
        return launch_export_t<S, T>(a, count, s);                                                 \
    }                                                                                              \
    hipError_t launch_ck_##SUFFIX(bool save, const CkArgs &a, int blocks, int nrep, hipStream_t s) { \
        return launch_ck_t<S>(save, a, blocks, nrep, s);                                           \
    }                                                                                              \
    hipError_t launch_fields_a_##SUFFIX(const FieldArgs &a, int64_t N, hipStream_t s) {            \
        return launch_fields_a_t<S, T>(a, N, s);                                                   \
    }

}  // namespace lbm
