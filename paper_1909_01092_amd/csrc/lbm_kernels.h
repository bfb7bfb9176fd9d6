// Launch interface between the C-ABI host code and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_types.h"

namespace lbm {

struct MainArgs {
    const RepDesc *desc;
    RepState *state;
    const int32_t *wg_begin;   // nrep entries
    int32_t nrep;
    const void *src;           // populations of step n (post-collision of n-1)
    void *dst;                 // post-collision populations of step n
    const uint32_t *pmask;     // node masks of step n (bbox)
    const double *vrho;        // wetting-layer densities of step n (bbox)
    double *rho_n;             // densities of step n near the sphere (bbox), written
    int32_t tau1;              // every relaxation time of every replica is 1
    int32_t groups;            // some fluid holds several spheres
    int32_t noise;             // some replica has kT > 0
    int32_t stream;            // store rows of a multiple of this many bytes (64, 128) past the caches; 0: none
};

struct LinkArgs {
    const RepDesc *desc;
    const RepState *state;
    const int32_t *k3_begin;
    int32_t nrep;
    void *buf;                 // post-collision populations of step n (bounced values written)
    const uint32_t *pmask;     // node masks of step n (bbox)
    const double *vrho;        // wetting-layer densities of step n (bbox)
    const double *rho_n;       // densities of step n (bbox)
    double *raw;               // post-streaming densities and momenta of fluid box nodes, written
    double *part1;             // per-workgroup link partials
};

// Box nodes per workgroup of the bounding-box kernels k_links / k_particle, and
// its threads (four per node).
constexpr int K3_NODES = 64;
constexpr int K3_THREADS = 4 * K3_NODES;

struct ParticleArgs {
    const RepDesc *desc;
    RepState *state;
    const int32_t *k3_begin;
    int32_t nrep;
    void *buf;                 // populations of step n+1 (uncovered-node values written)
    const double *part1;       // link partials
    double *part3;             // cover / uncover partials
    const uint32_t *pmask_old; // node masks of step n
    uint32_t *pmask;           // node masks of step n+1, written
    const double *raw;
    double *vrho;              // wetting-layer densities of step n+1, written
    double *series;
};

struct InitArgs {
    const RepDesc *desc;
    RepState *state;
    const int32_t *init_begin;
    int32_t nrep;
    void *buf;
    double *mass;              // 2 per init workgroup
    double *vrho;
    uint32_t *pmask;
};

struct ExportArgs {
    const RepDesc *desc;
    const RepState *state;
    int32_t rep;
    int32_t z_begin, z_end;
    const void *src;
    const uint32_t *pmask;
    double *out;
};

struct CkArgs {
    const RepDesc *desc;
    int32_t rep0;              // first entry of the launch (grid y)
    void *pop;                 // population buffer
    void *ck;                  // population part of a checkpoint
};

struct FieldArgs {
    const RepDesc *desc;
    const RepState *state;
    int32_t rep;
    const void *src;
    const uint32_t *pmask;
    const double *vrho;
    double *scratch;           // 9 N doubles
    double *columns;           // 8 nx ny doubles, or null
    int32_t cz;                // planes per z-chunk of the column sums
};

// dispatch on the storage precision (0 FP64, 1 FP32, 2 FP16)
hipError_t launch_main(int prec, const MainArgs &a, int grid, int block, size_t lds, hipStream_t s);
hipError_t launch_links(int prec, const LinkArgs &a, int grid, hipStream_t s);
hipError_t launch_particle(int prec, const ParticleArgs &a, int grid, hipStream_t s);
hipError_t launch_init(int prec, const InitArgs &a, int grid, int nrep, hipStream_t s);
hipError_t launch_export(int prec, const ExportArgs &a, int64_t count, hipStream_t s);
hipError_t launch_ck(int prec, bool save, const CkArgs &a, int blocks, int nrep, hipStream_t s);
hipError_t launch_fields(int prec, const FieldArgs &a, int64_t N, int64_t plane, hipStream_t s);

#define LBM_DECLARE(SUFFIX)                                                                        \
    hipError_t launch_main_##SUFFIX(const MainArgs &, int, int, size_t, hipStream_t);              \
    hipError_t launch_links_##SUFFIX(const LinkArgs &, int, hipStream_t);                          \
    hipError_t launch_particle_##SUFFIX(const ParticleArgs &, int, hipStream_t);                   \
    hipError_t launch_init_##SUFFIX(const InitArgs &, int, hipStream_t);                           \
    hipError_t launch_export_##SUFFIX(const ExportArgs &, int64_t, hipStream_t);                   \
    hipError_t launch_ck_##SUFFIX(bool, const CkArgs &, int, int, hipStream_t);                    \
    hipError_t launch_fields_a_##SUFFIX(const FieldArgs &, int64_t, hipStream_t);
LBM_DECLARE(f64)
LBM_DECLARE(f32)
LBM_DECLARE(f16)

}  // namespace lbm
