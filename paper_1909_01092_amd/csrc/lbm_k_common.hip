// Precision-independent kernels (initial wetting layer, hydrodynamic velocity,
// column sums) and the dispatch on storage precision.
#include <algorithm>
#include "lbm_kernels_impl.h"

namespace lbm {

// Wetting-layer densities, bbox origin and fluid count of the initial state
// (one workgroup per replica).
__global__ __launch_bounds__(256) void k_init_layer(InitArgs a) {
    __shared__ double red[4];
    const int r = blockIdx.x;
    const RepDesc &D = a.desc[r];
    RepState *st = a.state + r;
    const Geo g = geo_of(D);
    if (!D.has_particle) {
        if (threadIdx.x == 0) st->n_fluid = (double)D.N;
        return;
    }
    const int n3[3] = {g.nx, g.ny, g.nz};
    const bool w3[3] = {g.wx, g.wy, g.wz};
    const double X[3] = {st->X[0], st->X[1], st->X[2]};
    int org[3];
    for (int q = 0; q < 3; q++) org[q] = (int)floor(X[q] - D.radius) - 2;
    const int Sx = D.S, S3 = Sx * Sx * Sx;
    double *vrho = a.vrho + D.bbox_off * 2;
    uint32_t *pmask = a.pmask + D.bbox_off;
    auto init_rho = [&](int x, int y, int z, int l) {
        uint32_t c0 = (uint32_t)nidx(x, y, z, g), c1 = 0u, c2 = 0u, c3 = 1u;
        philox4x32_10(c0, c1, c2, c3, D.key0, D.key1);
        const uint32_t w = l == 0 ? c0 : c1;
        const bool swap = D.init_split > 0 && z >= D.init_split;  // other phase above the split
        return (swap ? D.rho0[1 - l] : D.rho0[l]) + D.init_amp * (2.0 * (((double)w + 0.5) * 0x1p-32) - 1.0);
    };
    double ns[1] = {0.0};
    for (int b = threadIdx.x; b < S3; b += 256) {
        int p[3];
        const int bb[3] = {b % Sx, (b / Sx) % Sx, b / (Sx * Sx)};
        bool in = true;
        for (int q = 0; q < 3; q++) {
            int v = org[q] + bb[q];
            if (v < 0 || v >= n3[q]) {
                if (w3[q]) in = false;
                else v = ((v % n3[q]) + n3[q]) % n3[q];
            }
            p[q] = v;
        }
        const bool solid = in && pnode(p[0], p[1], p[2], X, D.R2, g);
        pmask[b] = solid ? MASK_SOLID : 0u;  // populations of step 0 sit in own slots
        if (!solid) continue;
        ns[0] += 1.0;
        double s0 = 0.0, s1 = 0.0;
        int cnt = 0;
        for (int i = 1; i < Q; i++) {
            int qx = p[0] + cx(i), qy = p[1] + cy(i), qz = p[2] + cz(i);
            if (!(wrap1(qx, g.nx, g.wx) && wrap1(qy, g.ny, g.wy) && wrap1(qz, g.nz, g.wz))) continue;
            if (pnode(qx, qy, qz, X, D.R2, g)) continue;
            s0 += init_rho(qx, qy, qz, 0);
            s1 += init_rho(qx, qy, qz, 1);
            cnt++;
        }
        vrho[b] = cnt > 0 ? s0 / cnt + D.drho : 0.0;
        vrho[S3 + b] = cnt > 0 ? s1 / cnt - D.drho : 0.0;
    }
    block_sum<256, 1>(ns, red);
    if (threadIdx.x == 0) {
        st->n_fluid = (double)D.N - ns[0];
        for (int q = 0; q < 3; q++) st->org[q] = org[q];
    }
}

// Hydrodynamic velocity v + (F_A + F_B) / (2 rho) per node from the scratch
// written by k_fields_a.
__global__ __launch_bounds__(256) void k_fields_b(FieldArgs a) {
    const RepDesc &D = a.desc[a.rep];
    const Geo g = geo_of(D);
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= g.N) return;
    const int x = (int)(n % g.nx), y = (int)((n / g.nx) % g.ny);
    const int z = (int)(n / ((int64_t)g.nx * g.ny));
    const double *rt = a.scratch, *jt = a.scratch + 2 * g.N, *sol = a.scratch + 8 * g.N;
    double *u = a.scratch + 5 * g.N;
    if (sol[n] != 0.0) {
        for (int q = 0; q < 3; q++) u[q * g.N + n] = 0.0;
        return;
    }
    double grad[2][3] = {{0, 0, 0}, {0, 0, 0}};
    for (int i = 1; i < Q; i++) {
        const int qx = mirror1(x + cx(i), g.nx, g.wx), qy = mirror1(y + cy(i), g.ny, g.wy);
        const int qz = mirror1(z + cz(i), g.nz, g.wz);
        const int64_t m = nidx(qx, qy, qz, g);
        for (int l = 0; l < 2; l++) {
            const double v = wgt(i) * rt[l * g.N + m];
            grad[l][0] += v * cx(i); grad[l][1] += v * cy(i); grad[l][2] += v * cz(i);
        }
    }
    const double rA = rt[n], rB = rt[g.N + n];
    for (int q = 0; q < 3; q++) {
        const double FA = -D.G * rA * grad[1][q] + rA * D.af[q];
        const double FB = -D.G * rB * grad[0][q] + rB * D.af[q];
        u[q * g.N + n] = (jt[q * g.N + n] + 0.5 * (FA + FB)) / (rA + rB);
    }
}

// Column sums over z: mass_A, mass_B, j (3), sum |u|^2, sum u_z, fluid count.
// One thread per column (x, y) and z-chunk of a.cz planes, marching over its
// planes with the 3 x 3 neighbourhoods of three of them in registers, so 9
// densities per component are read per node and not 18, and the velocity (formed
// as k_fields_b forms it, term by term: at rest it is rounding error of the
// gradient) stays in registers.  Partial sums per chunk go where k_fields_b would
// write the velocity; k_columns adds them in the order of the chunks.  Bound by
// memory: 192 x 192 x 1024 takes 0.61 ms with k_columns, where k_fields_b and one
// thread per whole column took 2.24 (60 x 60 x 900, 15 workgroups before: 89 us
// and 730).
__global__ __launch_bounds__(256) void k_column_parts(FieldArgs a) {
    const RepDesc &D = a.desc[a.rep];
    const Geo g = geo_of(D);
    const int64_t plane = (int64_t)g.nx * g.ny, N = g.N;
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= plane) return;
    const int x = (int)(c % g.nx), y = (int)(c / g.nx);
    const int xs[3] = {mirror1(x - 1, g.nx, g.wx), x, mirror1(x + 1, g.nx, g.wx)};
    const int64_t ys[3] = {(int64_t)mirror1(y - 1, g.ny, g.wy) * g.nx, (int64_t)y * g.nx,
                           (int64_t)mirror1(y + 1, g.ny, g.wy) * g.nx};
    const double *rt = a.scratch, *jt = a.scratch + 2 * N, *sol = a.scratch + 8 * N;
    double v[3][2][9];  // planes z - 1, z, z + 1; component; 3 x 3 neighbourhood
    auto load = [&](int zp, double(&to)[2][9]) {
        const double *r = rt + plane * mirror1(zp, g.nz, g.wz);
#pragma unroll
        for (int l = 0; l < 2; l++)
#pragma unroll
            for (int k = 0; k < 9; k++) to[l][k] = r[l * N + ys[k / 3] + xs[k % 3]];
    };
    const int z0 = blockIdx.y * a.cz, z1 = min(z0 + a.cz, g.nz);
    load(z0 - 1, v[0]);
    load(z0, v[1]);
    double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int z = z0; z < z1; z++) {
        load(z + 1, v[2]);
        const int64_t n = c + plane * z;
        const double j[3] = {jt[n], jt[N + n], jt[2 * N + n]};
        if (sol[n] == 0.0) {
            double grad[2][3] = {{0, 0, 0}, {0, 0, 0}};
#pragma unroll
            for (int i = 1; i < Q; i++)
#pragma unroll
                for (int l = 0; l < 2; l++) {
                    const double t = wgt(i) * v[cz(i) + 1][l][3 * (cy(i) + 1) + cx(i) + 1];
                    grad[l][0] += t * cx(i); grad[l][1] += t * cy(i); grad[l][2] += t * cz(i);
                }
            const double rA = v[1][0][4], rB = v[1][1][4];
            double u[3];
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const double FA = -D.G * rA * grad[1][q] + rA * D.af[q];
                const double FB = -D.G * rB * grad[0][q] + rB * D.af[q];
                u[q] = (j[q] + 0.5 * (FA + FB)) / (rA + rB);
                s[2 + q] += j[q];
            }
            s[0] += rA;
            s[1] += rB;
            s[5] += u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
            s[6] += u[2];
            s[7] += 1.0;
        }
#pragma unroll
        for (int l = 0; l < 2; l++)
#pragma unroll
            for (int k = 0; k < 9; k++) {
                v[0][l][k] = v[1][l][k];
                v[1][l][k] = v[2][l][k];
            }
    }
    double *part = gridDim.y == 1 ? a.columns : a.scratch + 5 * N + (int64_t)blockIdx.y * 8 * plane;
    for (int k = 0; k < 8; k++) part[k * plane + c] = s[k];
}

__global__ __launch_bounds__(256) void k_columns(FieldArgs a, int chunks) {
    const Geo g = geo_of(a.desc[a.rep]);
    const int64_t cols = 8 * (int64_t)g.nx * g.ny;
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= cols) return;
    const double *part = a.scratch + 5 * g.N + c;
    double s = 0.0;
#pragma unroll 4
    for (int k = 0; k < chunks; k++) s += part[k * cols];
    a.columns[c] = s;
}

hipError_t launch_main(int prec, const MainArgs &a, int grid, int block, size_t lds, hipStream_t s) {
    if (prec == 0) return launch_main_f64(a, grid, block, lds, s);
    if (prec == 1) return launch_main_f32(a, grid, block, lds, s);
    return launch_main_f16(a, grid, block, lds, s);
}

hipError_t launch_links(int prec, const LinkArgs &a, int grid, hipStream_t s) {
    if (prec == 0) return launch_links_f64(a, grid, s);
    if (prec == 1) return launch_links_f32(a, grid, s);
    return launch_links_f16(a, grid, s);
}

hipError_t launch_particle(int prec, const ParticleArgs &a, int grid, hipStream_t s) {
    if (prec == 0) return launch_particle_f64(a, grid, s);
    if (prec == 1) return launch_particle_f32(a, grid, s);
    return launch_particle_f16(a, grid, s);
}

hipError_t launch_init(int prec, const InitArgs &a, int grid, int nrep, hipStream_t s) {
    hipError_t e = prec == 0 ? launch_init_f64(a, grid, s)
                 : prec == 1 ? launch_init_f32(a, grid, s) : launch_init_f16(a, grid, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_init_layer, dim3(nrep), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_export(int prec, const ExportArgs &a, int64_t count, hipStream_t s) {
    if (prec == 0) return launch_export_f64(a, count, s);
    if (prec == 1) return launch_export_f32(a, count, s);
    return launch_export_f16(a, count, s);
}

hipError_t launch_ck(int prec, bool save, const CkArgs &a, int blocks, int nrep, hipStream_t s) {
    if (prec == 0) return launch_ck_f64(save, a, blocks, nrep, s);
    if (prec == 1) return launch_ck_f32(save, a, blocks, nrep, s);
    return launch_ck_f16(save, a, blocks, nrep, s);
}

hipError_t launch_fields(int prec, const FieldArgs &a, int64_t N, int64_t plane, hipStream_t s) {
    hipError_t e = prec == 0 ? launch_fields_a_f64(a, N, s)
                 : prec == 1 ? launch_fields_a_f32(a, N, s) : launch_fields_a_f16(a, N, s);
    if (e != hipSuccess) return e;
    if (a.columns == nullptr) {
        hipLaunchKernelGGL(k_fields_b, dim3((int)((N + 255) / 256)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    // chunks for about 2048 workgroups (and no more than a grid's y extent); of
    // four planes or more, so that their sums (8 per column) fit the 3 N doubles
    // of the velocity.  A single chunk writes its sums to the columns.
    const int tiles = (int)((plane + 255) / 256), nz = (int)(N / plane);
    FieldArgs f = a;
    f.cz = nz < 8 ? nz : std::max({4, (int)((int64_t)nz * tiles / 2048), nz / 32768 + 1});
    const int chunks = (nz + f.cz - 1) / f.cz;
    hipLaunchKernelGGL(k_column_parts, dim3(tiles, chunks), dim3(256), 0, s, f);
    e = hipGetLastError();
    if (e != hipSuccess || chunks == 1) return e;
    hipLaunchKernelGGL(k_columns, dim3((int)((8 * plane + 255) / 256)), dim3(256), 0, s, f, chunks);
    return hipGetLastError();
}

}  // namespace lbm
