// lbmbp: lattice-Boltzmann fluid two-way coupled to Brownian point particles
// (Yoshida, Kinjo & Washizu, arXiv:1909.13412), hand-written HIP for gfx950.
//
// One coupled step n (section 2):
//   k_particle        per particle, eight lanes = eight neighbour nodes:
//                     VACF sample C_i(l) += V_i(t0).V_i(n) (section 2.1),
//                     gather u^n at the nodes (Eq. s2-fv), Stokeslet fit
//                     (Eq. s2-slet-v) -> F_H, Philox Brownian force
//                     (Eqs. s2-rf1, s2-rf2), spread -F_H into the node-force
//                     field (first Eq. s2-force), Langevin update (Eqs.
//                     s2-langevin, s2-langevin2)
//   k_stream_collide  every node: pull f^n_a(x) = A_a(x - e_a) (Eq. s2-trans of
//                     the previous step), moments (Eqs. s2-density, s2-fv),
//                     BGK (Eqs. s2-collision, s2-eq) plus forcing (second
//                     Eq. s2-force) where the node is flagged, write B_a(x)
//                     (Eq. s2-coll); A and B swap.
// Two steps n and n + 1 in one sweep, the same bits (twostep.hpp):
//   k_particle        step n, as above
//   k_particle_ahead  step n + 1, on post-collision values of step n that its
//                     blocks compute around the particles
//   k_two_steps       every node: both steps' collisions, A read and B written
//                     once.
//
// Layout and the stream-collide kernel: collide.hpp.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <algorithm>
#include <vector>

#include "lbmbp.h"
#include "adjoint.hpp"
#include "codec.hpp"
#include "collide.hpp"
#include "collide_launch.hpp"
#include "velocities.hpp"
#include "pairs.hpp"
#include "replica.hpp"
#include "particle.hpp"
#include "philox.hpp"
#include "twostep_launch.hpp"

namespace lbmbp {

constexpr int kRedBlocks = 1024;
// Node-force fields of a box: step n spreads into its own field, n mod 2.  A
// two-step sweep reads the fields of both its steps, so neither can be cleared
// before it, and the particle update that follows clears both: where the first
// of them is that update's own field, it takes the third (24 bytes a
// node, in the particle scratch of boxes that can take two-step sweeps with
// particles).  Two sweeps in a
// row so end with the fields in the roles they started with, and an even number of
// steps (the lattices' condition) can be captured into a graph and replayed.
constexpr int kForceFields = 3;
constexpr int kThirdField = 2;

template <class C, int CPT, int BS, bool NTS>
__global__ __launch_bounds__(BS) void k_ens_collide(const typename C::T *__restrict__ A,
                                                    typename C::T *__restrict__ B,
                                                    const Replica *__restrict__ reps,
                                                    const uint16_t *__restrict__ blk_rep,
                                                    int shape, long long *force,
                                                    uint32_t *mask, typename C::R enc_s,
                                                    typename C::R dec_s, EnsClock *clock,
                                                    int vacf_on, uint32_t order) {
    const uint32_t b = sweep_block(order);
    const uint32_t rid = blk_rep[b];
    const Replica &rp = reps[rid];
    const uint32_t lane_cell = (b - rp.first_block[shape]) * BS + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // the step's last reader of the clock has finished (previous kernel)
        clock->step += 1;
        if (vacf_on) clock->vacf_t += 1;
    }
    if (lane_cell >= rp.g.ncell / CPT) return;
    const ForceField ff{force + 3 * rp.cell_off, mask + rp.mask_off};
    double acc[4];
    using R = typename C::R;
    collide_lane<C, true, false, CPT, NTS>(A + rp.pop_off, B + rp.pop_off, rp.g, R(rp.omega),
                                           enc_s, dec_s, ff, R(0), R(0), R(0), lane_cell, acc);
}

// Streaming-only counterpart of k_ens_collide (same block -> box table, block
// order, lanes and store policy): the comparison kernel the ensemble
// stream-collide is measured against.
template <class C, int CPT, int BS, bool NTS>
__global__ __launch_bounds__(BS) void k_ens_stream_only(const typename C::T *__restrict__ A,
                                                        typename C::T *__restrict__ B,
                                                        const Replica *__restrict__ reps,
                                                        const uint16_t *__restrict__ blk_rep, int shape,
                                                        uint32_t order) {
    const uint32_t b = sweep_block(order);
    const Replica &rp = reps[blk_rep[b]];
    const uint32_t lane_cell = (b - rp.first_block[shape]) * BS + threadIdx.x;
    if (lane_cell >= rp.g.ncell / CPT) return;
    stream_only_lane<C, CPT, NTS>(A + rp.pop_off, B + rp.pop_off, rp.g, lane_cell);
}

// ---------------------------------------------------------------------------
// Recorded observables: two fixed-order stages over the per-wavefront partials
// left by the stream-collide (rho~ - 1, u) and the per-block ones of the
// particle kernel (M V).
// ---------------------------------------------------------------------------
constexpr int kSeriesBlocks = 64;

__global__ __launch_bounds__(kBlock) void k_series_stage1(const double *__restrict__ fluid,
                                                          int32_t nfluid,
                                                          const double *__restrict__ part,
                                                          int32_t npart,
                                                          double *__restrict__ stage) {
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    const int32_t stride = kSeriesBlocks * kBlock;
    for (int32_t i = blockIdx.x * kBlock + threadIdx.x; i < nfluid; i += stride)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += fluid[4 * int64_t(i) + k];
    for (int32_t i = blockIdx.x * kBlock + threadIdx.x; i < npart; i += stride)
#pragma unroll
        for (int k = 0; k < 3; ++k) v[4 + k] += part[3 * int64_t(i) + k];
    block_sum<7, kBlock>(v, stage + 7 * blockIdx.x);
}

__global__ void k_series_stage2(const double *__restrict__ stage, double ncell, double step,
                                double *__restrict__ out) {
    if (threadIdx.x < 7) {
        double s = 0.0;
        for (int b = 0; b < kSeriesBlocks; ++b) s += stage[7 * b + threadIdx.x];
        out[1 + threadIdx.x] = threadIdx.x == 0 ? ncell + s : s;
    }
    if (threadIdx.x == 0) out[0] = step;
}

// ---------------------------------------------------------------------------
// Field access kernels (set-up and diagnostics, not on the stepping path).
// ---------------------------------------------------------------------------
template <class C>
__global__ __launch_bounds__(kBlock) void k_get_populations(const typename C::T *__restrict__ A,
                                                            Grid g, typename C::R dec_s,
                                                            double *__restrict__ f) {
    using Vs = typename C::V;
    const uint32_t cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= g.ncell) return;
    const uint32_t x = cell % g.nx, t = cell / g.nx, y = t % g.ny, z = t / g.ny;
    const Neighbours nb(x, y, z, g);
    static_for<0, Vs::Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        f[uint64_t(a) * g.ncell + cell] =
            double(C::dec(A[nb.template pop<Vs, a>(g)], dec_s)) + Vs::template w<double>(a);
    });
}

template <class C>
__global__ __launch_bounds__(kBlock) void k_get_moments(const typename C::T *__restrict__ A,
                                                        Grid g, typename C::R dec_s,
                                                        double *__restrict__ rho,
                                                        double *__restrict__ u) {
    using Vs = typename C::V;
    const uint32_t cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= g.ncell) return;
    const uint32_t x = cell % g.nx, t = cell / g.nx, y = t % g.ny, z = t / g.ny;
    const Neighbours nb(x, y, z, g);
    double dr = 0.0, m[3] = {0.0, 0.0, 0.0};
    static_for<0, Vs::Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        const double gvl = double(C::dec(A[nb.template pop<Vs, a>(g)], dec_s));
        dr += gvl;
        m[0] += Vs::ex[a] * gvl;
        m[1] += Vs::ey[a] * gvl;
        m[2] += Vs::ez[a] * gvl;
    });
    if (rho) rho[cell] = 1.0 + dr;
    if (u) {
        u[cell] = m[0];
        u[uint64_t(g.ncell) + cell] = m[1];
        u[2 * uint64_t(g.ncell) + cell] = m[2];
    }
}

// A_a(y) = enc(f_a(y + e_a) - w_a): the post-streaming population at node x is
// the pulled value A_a(x - e_a).
template <class C>
__global__ __launch_bounds__(kBlock) void k_set_populations(const double *__restrict__ f,
                                                            typename C::T *__restrict__ A, Grid g,
                                                            typename C::R enc_s) {
    using Vs = typename C::V;
    const uint32_t cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= g.ncell) return;
    const uint32_t x = cell % g.nx, t = cell / g.nx, y = t % g.ny, z = t / g.ny;
    const Neighbours nb(x, y, z, g);  // nb.src of the opposite direction is y + e_a
    static_for<0, Vs::Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        constexpr int o = (a == 0) ? 0 : ((a & 1) ? a + 1 : a - 1);
        const double gvl = f[uint64_t(a) * g.ncell + nb.template src<Vs, o>(g)] - Vs::template w<double>(a);
        A[pop_index<Vs>(g, x, y, z, a)] = C::enc(typename C::R(gvl), enc_s);
    });
}

template <class C>
__global__ __launch_bounds__(kBlock) void k_set_equilibrium(const double *__restrict__ rho,
                                                            const double *__restrict__ u,
                                                            typename C::T *__restrict__ A, Grid g,
                                                            typename C::R enc_s) {
    using Vs = typename C::V;
    const uint32_t cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= g.ncell) return;
    const uint32_t x = cell % g.nx, t = cell / g.nx, y = t % g.ny, z = t / g.ny;
    const Neighbours nb(x, y, z, g);
    static_for<0, Vs::Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        constexpr int o = (a == 0) ? 0 : ((a & 1) ? a + 1 : a - 1);
        const uint32_t src = nb.template src<Vs, o>(g);  // node y + e_a
        const double dr = rho ? rho[src] - 1.0 : 0.0;
        double uc[3] = {0.0, 0.0, 0.0};
        if (u) {
            uc[0] = u[src];
            uc[1] = u[uint64_t(g.ncell) + src];
            uc[2] = u[2 * uint64_t(g.ncell) + src];
        }
        const double eu = Vs::ex[a] * uc[0] + Vs::ey[a] * uc[1] + Vs::ez[a] * uc[2];
        const double uu = uc[0] * uc[0] + uc[1] * uc[1] + uc[2] * uc[2];
        const double geq = Vs::template w<double>(a) * (dr + 3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
        A[pop_index<Vs>(g, x, y, z, a)] = C::enc(typename C::R(geq), enc_s);
    });
}

// The same populations in another row-group layout: B[in layout gb] =
// A[in layout ga], element for element (a permutation; no arithmetic).
template <class C>
__global__ __launch_bounds__(kBlock) void k_relayout(const typename C::T *__restrict__ A, Grid ga,
                                                     typename C::T *__restrict__ B, Grid gb) {
    using Vs = typename C::V;
    const uint32_t cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= ga.ncell) return;
    const uint32_t x = cell % ga.nx, t = cell / ga.nx, y = t % ga.ny, z = t / ga.ny;
    static_for<0, Vs::Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        B[pop_index<Vs>(gb, x, y, z, a)] = A[pop_index<Vs>(ga, x, y, z, a)];
    });
}

// FP64 sums of (rho - 1, u) over all nodes: fixed grid, fixed tree order, so the
// result is deterministic.
template <class C>
__global__ __launch_bounds__(kBlock) void k_fluid_partials(const typename C::T *__restrict__ A,
                                                           Grid g, typename C::R dec_s,
                                                           double *__restrict__ partials) {
    using Vs = typename C::V;
    __shared__ double sh[4][kBlock];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint32_t cell = blockIdx.x * kBlock + threadIdx.x; cell < g.ncell;
         cell += gridDim.x * kBlock) {
        const uint32_t x = cell % g.nx, t = cell / g.nx, y = t % g.ny, z = t / g.ny;
        const Neighbours nb(x, y, z, g);
        static_for<0, Vs::Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            const double gvl = double(C::dec(A[nb.template pop<Vs, a>(g)], dec_s));
            acc[0] += gvl;
            acc[1] += Vs::ex[a] * gvl;
            acc[2] += Vs::ey[a] * gvl;
            acc[3] += Vs::ez[a] * gvl;
        });
    }
    for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h)
            for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x < 4) partials[4 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ __launch_bounds__(kBlock) void k_final_sums(const double *__restrict__ partials,
                                                       int32_t nparts, double ncell,
                                                       const double *__restrict__ v, int32_t n,
                                                       double mass, double *__restrict__ out) {
    __shared__ double sh[7][kBlock];
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int32_t b = threadIdx.x; b < nparts; b += kBlock)
        for (int k = 0; k < 4; ++k) acc[k] += partials[4 * b + k];
    for (int32_t i = threadIdx.x; i < n; i += kBlock)
        for (int k = 0; k < 3; ++k) acc[4 + k] += v[3 * i + k];
    for (int k = 0; k < 7; ++k) sh[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (int(threadIdx.x) < h)
            for (int k = 0; k < 7; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = ncell + sh[0][0];
        for (int k = 1; k < 4; ++k) out[k] = sh[k][0];
        for (int k = 0; k < 3; ++k) out[4 + k] = mass * sh[4 + k][0];
    }
}

}  // namespace lbmbp

// ===========================================================================
// Host side: the C ABI.
// ===========================================================================
using namespace lbmbp;

struct lbm_ctx {
    lbm_grid_desc desc;
    Grid g;
    int q;  // velocity set: 19 or 15
    size_t elem;
    void *pop[2];  // pop[cur] holds post-collision values of the last step
    int cur;
    hipStream_t stream;
    double omega;
    double enc_s, dec_s;
    double body[3];  // uniform body force on every node (lbm_set_body_force)
    // grid scratch
    uint32_t *mask[kForceFields];
    long long *force[kForceFields];  // [ncell][3] fixed-point node forces; the third in the particle scratch or null
    uint32_t mask_words;
    double *partials;
    double *result;
    uint32_t *err;
    // particles
    int32_t np;
    lbm_particle_desc pdesc;
    double R;
    double *r, *v;
    uint32_t *cells[2];  // [n][8] nodes spread to in even and odd steps
    int fields_used;     // a particle update has run since the fields were cleared
    int last_field;      // the field that the last step spread into
    int own_held;        // this step's own field still holds the forces of the step before the last
    int older_due;       // the forces of the step before the last may have to be released
    double *fh, *fr;
    const double *fext;  // given force on each particle (lbm_set_particle_force) or null
    uint32_t warnings;   // LBM_WARN_* of the attached particles
    // soft pair repulsion (lbm_set_pair_force)
    int pair_on;
    PairGrid pg;
    PairList plist;       // particle scratch: the cell list
    double *fpair;        // particle scratch: [n][3] pair forces of the last step
    // velocity autocorrelation
    int vacf_on;
    int32_t max_lag, stride, nslot;
    double *acc, *origins;
    int64_t vacf_t;
    int64_t step;
    // per-kernel event timing (host-side event objects)
    int prof_on;
    hipEvent_t *prof_ev;    // pairs: [2k] start, [2k+1] stop
    int32_t *prof_kind;     // per pair: 0 stream-collide, 1 particle phase
    int32_t prof_used, prof_cap;
    int shape;   // index into kShapes
    int order;   // block order of the sweep (kOrderLinear / kOrderXcdSlabs)
    int cap;     // residency cap of the sweep: index into kResidencyCaps
    int lds_cu, lds_block;  // LDS bytes per compute unit and per block (device limits)
    int two;     // two-step sweep: 0 never, else candidate two - 1 of two_step_candidates
    int two_nts; // its populations written with non-temporal stores
    TwoStepTiles two_tiles;
    int device;  // device current at lbm_init (autotune cache key)
    // recorded observables (lbm_series_config)
    int32_t series_every;
    double *series;
    int64_t series_cap, series_count, series_t;
    double *fluid_partials;  // grid scratch: [collide wavefronts][4]
    double *series_stage;    // grid scratch: [kSeriesBlocks][7]
    double *part_partials;   // particle scratch: [particle blocks][3]
    // forward run kept for the adjoint (lbm_record)
    void *rec_tape;
    int64_t rec_n0;
    int32_t rec_nsteps, rec_every, rec_np;
    lbm_particle_desc rec_pdesc;
    double rec_R;
    const double *rec_fext;
    int rec_pair_on;
    PairGrid rec_pg;
    uint32_t rec_rows;  // layout (rows per group) of the recorded lattices
};

namespace {

constexpr size_t kAlign = 256;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

size_t elem_size(int storage) {
    switch (storage) {
        case LBM_STORE_F64: return 8;
        case LBM_STORE_F32: return 4;
        case LBM_STORE_BF16:
        case LBM_STORE_F16: return 2;
        default: return 0;
    }
}

int velocity_count(const lbm_grid_desc *g) { return g->velocities == 15 ? 15 : 19; }

bool grid_ok(const lbm_grid_desc *g) {
    if (!g) return false;
    if (g->nx < 2 || g->ny < 2 || g->nz < 2) return false;
    const uint64_t nc = uint64_t(g->nx) * uint64_t(g->ny) * uint64_t(g->nz);
    if (nc >= (uint64_t(1) << 31)) return false;
    if (!(g->tau > 0.5) || !isfinite(g->tau)) return false;
    if (elem_size(g->storage) == 0) return false;
    if (g->storage == LBM_STORE_F16 && (g->f16_scale_log2 < 0 || g->f16_scale_log2 > 24)) return false;
    if (g->velocities != 0 && g->velocities != 19 && g->velocities != 15) return false;
    if (g->reserved != 0) return false;
    return true;
}

uint64_t ncell_of(const lbm_grid_desc *g) {
    return uint64_t(g->nx) * uint64_t(g->ny) * uint64_t(g->nz);
}

// Elements per population row: nx, unpadded.  (Padding rows to whole
// 128-byte lines left gaps between the rows of a row group and measured 4-14%
// slower at sizes that are not multiples of a line.)
uint32_t row_chunk(const lbm_grid_desc *g) { return uint32_t(g->nx); }

uint32_t mask_words(uint64_t ncell) { return uint32_t(align_up((ncell + 31) / 32, 64)); }

size_t force_field_bytes(const lbm_grid_desc *g) { return align_up(ncell_of(g) * 3 * 8, kAlign); }

// Blocks of the row-aligned stream-collide grid (configurations 8, 9).
uint32_t row_grid_blocks(uint32_t nx, uint32_t ny, uint32_t nz) {
    const uint32_t lpr = row_lanes(nx), nrows = ny * nz;
    if (lpr <= uint32_t(kRowBlock)) {
        const uint32_t rpb = uint32_t(kRowBlock) / lpr;  // rows per block
        return (nrows + rpb - 1) / rpb;
    }
    return nrows * ((lpr + kRowBlock - 1) / kRowBlock);
}

// Per-wavefront moment partials of the largest stream-collide grid: one node
// per lane in whole blocks of up to 512 lanes, or the row-aligned grid,
// whichever has more wavefronts.
size_t fluid_partials_bytes(const lbm_grid_desc *g) {
    const size_t flat = (ncell_of(g) / 512 + 1) * 8;
    const size_t row = row_grid_blocks(uint32_t(g->nx), uint32_t(g->ny), uint32_t(g->nz)) * (kRowBlock / 64);
    return align_up((flat > row ? flat : row) * 4 * 8, kAlign);
}

size_t grid_scratch_size(const lbm_grid_desc *g) {
    const size_t words = mask_words(ncell_of(g));
    size_t s = 0;
    s += kThirdField * align_up(words * 4, kAlign);  // bitmasks
    s += kThirdField * force_field_bytes(g);         // node-force fields
    s += fluid_partials_bytes(g);                    // recorded-moment partials
    s += align_up(size_t(kSeriesBlocks) * 7 * 8, kAlign);
    s += align_up(size_t(kRedBlocks) * 4 * 8, kAlign);  // partials
    s += align_up(8 * 8, kAlign);                    // result
    s += kAlign;                                      // error flags
    return s;
}

size_t particle_blocks(int32_t n) { return (size_t(n) * 8 + kParticleBlock - 1) / kParticleBlock; }

// Lanes of a particle block: a second wavefront takes the VACF sample.
unsigned particle_threads(const ParticleArgs &pa) { return pa.acc ? 2 * kParticleBlock : kParticleBlock; }

// Advisory conditions of a particle set (section 2.2's parameter ranges and
// the sign of the fit's gain); see LBM_WARN_* in the header.
uint32_t coupling_warnings(int32_t friction, double R, int32_t n, double ncell) {
    uint32_t w = 0;
    const double s3 = sqrt(3.0);
    if (friction == LBM_FRICTION_STOKESLET || friction == LBM_FRICTION_STOKESLET_2DX ||
        friction == LBM_FRICTION_STOKESLET_CUBE) {
        const double span = friction == LBM_FRICTION_STOKESLET ? 1.0 : 2.0;  // cube edge
        if (R > s3 * span) w |= LBM_WARN_RADIUS_BOUND;
        if (R > 0.5 * s3 * span) w |= LBM_WARN_NEGATIVE_GAIN;
    }
    if (friction != LBM_FRICTION_BD && double(n) * (4.0 / 3.0) * M_PI * R * R * R > 0.1 * ncell)
        w |= LBM_WARN_VOLUME_FRACTION;
    return w;
}

// Buckets of the pair cell list: a power of two >= 2n.
uint32_t pair_buckets(int32_t n) {
    uint32_t T = 64;
    while (T < 2u * uint32_t(n)) T <<= 1;
    return T;
}

size_t pair_list_bytes(int32_t n) {
    n = std::min(n, kPairMax);  // more have no lists, but their scratch serves fewer
    return 2 * align_up(size_t(n) * sizeof(PairLink), kAlign) + align_up(2 * size_t(pair_buckets(n)) * 4, kAlign);
}

// Carves the cell list out of pair_list_bytes(n) bytes at s.
PairList pair_list_at(char *s, int32_t n) {
    const size_t links = align_up(size_t(n) * sizeof(PairLink), kAlign);
    uint32_t *head = reinterpret_cast<uint32_t *>(s + 2 * links);
    return PairList{reinterpret_cast<PairLink *>(s), reinterpret_cast<PairLink *>(s + links), head, head + pair_buckets(n)};
}

// Nodes per particle from which a two-step sweep pays for its particle update
// one step ahead, which reads the populations around a 4^3 instead of a 2^3
// neighbourhood (us per step in a run, two-step / single: FP32 128^3, 512 nodes
// each 59.8 / 67.2, 304 nodes 73.0 / 73.6, FP64 111 / 127; 16-bit storage saves
// less per sweep: BF16 256^3, 4096 nodes 198 / 222, 2048 nodes 232 / 231; 128^3
// 4096 nodes 30.4 / 31.5, 2048 nodes 32.5 / 32.5, 512 nodes 47.7 / 38.1; 192^3
// 6912 nodes 93.6 / 94.8, 3456 nodes 100 / 95.5), and nodes from which its
// launch does (16 particles: BF16 96^3 18.7 / 18.2, 128^3 27.0 / 29.8; FP32 72^3
// 14.6 / 15.7, but 60 recorded steps and their gradient at 64^3 3.66 / 3.56 ms).
// 16-bit D3Q15 needs more: its single step moves a fifth less, its sweep with
// forces spills as D3Q19's (256^3, 16384 nodes each and more 165-175 / 165-175,
// 4096 nodes 195 / 178; 192^3, 6912 nodes 89 / 83; 128^3, 4096 nodes 28.6 / 27.5).
constexpr double two_step_nodes_per_particle(size_t elem, int q) {
    return elem == 2 ? (q == D3Q15::Q ? 32768.0 : 4000.0) : 300.0;
}
constexpr uint64_t two_step_particle_nodes(size_t elem) { return elem == 2 ? uint64_t(1) << 21 : uint64_t(5) << 16; }

bool two_step_pays(size_t elem, int q, uint64_t nodes, int64_t particles) {
    if (particles == 0) return true;
    if (nodes < two_step_particle_nodes(elem)) return false;
    return double(nodes) >= two_step_nodes_per_particle(elem, q) * double(particles);
}

// The sweep's byte offsets within a plane are of 32 bits.
bool two_step_planes(const lbm_grid_desc *g) {
    return uint64_t(g->nx) * uint64_t(g->ny) * uint64_t(velocity_count(g)) * elem_size(g->storage) < (uint64_t(1) << 32);
}

// Bytes of the third node-force field and its flags (0: this box never has one).
// Room for it does not depend on the number of particles: scratch for many
// serves fewer, too, and it is they that take two-step sweeps.
size_t third_field_bytes(const lbm_grid_desc *g) {
    if (!two_step_planes(g) || !two_step_pays(elem_size(g->storage), velocity_count(g), ncell_of(g), 1)) return 0;
    return align_up(size_t(mask_words(ncell_of(g))) * 4, kAlign) + force_field_bytes(g);
}

size_t particle_scratch_size(const lbm_grid_desc *g, int32_t n) {
    if (n <= 0) return 0;
    size_t s = third_field_bytes(g);
    s += 2 * align_up(size_t(n) * 8 * 4, kAlign);  // nodes spread to, two steps
    s += align_up(particle_blocks(n) * 3 * 8, kAlign);  // momentum partials
    s += 2 * align_up(size_t(n) * 3 * 8, kAlign);  // fh, fr
    s += pair_list_bytes(n);                       // pair cell list
    s += align_up(size_t(n) * 3 * 8, kAlign);      // pair forces
    return s;
}

bool aligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) % kAlign) == 0; }

lbm_status launch_status() {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LBM_OK : LBM_E_DEVICE;
}

unsigned blocks_for(uint64_t n) { return unsigned((n + kBlock - 1) / kBlock); }
// The row-aligned mapping places lanes exactly as configurations 1 and 5 do
// when every 256-lane block holds whole rows that fill it (64 | nx and nx
// divides 256) or every row fills whole blocks (256 | nx).
bool row_mapping_is_flat(uint32_t nx) { return nx % 64 == 0 && (256 % nx == 0 || nx % 256 == 0); }

bool shape_ok(const lbm_ctx *c, int k) {
    return config_row(k) || c->g.ny % uint32_t(kShapes[k & 3].cpt) == 0;
}

uint32_t collide_grid(const lbm_ctx *c, int shape) {
    if (config_row(shape)) return row_grid_blocks(c->g.nx, c->g.ny, c->g.nz);
    const CollideShape &sh = kShapes[shape & 3];
    const uint64_t band = c->g.ncell / uint32_t(sh.cpt);
    return uint32_t((band + sh.bs - 1) / sh.bs);
}

// Dynamic LDS that caps the sweep at kResidencyCaps[cap] waves per SIMD for
// blocks of bs lanes (0: no cap); -1 if the device cannot impose that cap.
// The kernels never touch it: it only keeps further blocks off the unit.
// Up to 1 KiB of the unit is left for the kernels' own LDS.
long residency_lds(int lds_cu, int lds_block, int cap, int bs) {
    const int waves = kResidencyCaps[cap];
    if (waves == 0) return 0;
    // bs / 64 waves per block over the unit's four SIMDs: `blocks` resident
    // blocks give blocks * bs / 256 waves per SIMD
    const int blocks = waves * 256 / bs;
    if (blocks < 1 || lds_cu <= 0) return -1;
    const long per = (long(lds_cu) / blocks - 1024) / 512 * 512;
    if (per <= 0 || per + 1024 > lds_block) return -1;
    if (long(blocks + 1) * per <= lds_cu) return -1;  // would not cap
    return per;
}

long sweep_lds(const lbm_ctx *c, int cap, int bs) { return residency_lds(c->lds_cu, c->lds_block, cap, bs); }

// One stream-collide launch A -> B.  mom != nullptr: also leave the
// per-wavefront FP64 moment sums there.  order, cap: block order and residency
// cap (-1: the context's).
template <class C, bool FORCED>
void launch_collide(lbm_ctx *c, const typename C::T *A, typename C::T *B, ForceField ff, int shape,
                    double *mom = nullptr, int order = -1, int cap = -1) {
    CollideArgs a;
    a.A = A;
    a.B = B;
    a.g = c->g;
    a.omega = c->omega;
    a.enc_s = c->enc_s;
    a.dec_s = c->dec_s;
    for (int k = 0; k < 3; ++k) a.body[k] = c->body[k];
    a.ff = ff;
    a.mom = mom;
    a.shape = shape;
    a.grid = collide_grid(c, shape);
    a.order = order < 0 ? c->order : order;
    const long lds = sweep_lds(c, cap < 0 ? c->cap : cap, config_block(shape));
    a.dyn = lds > 0 ? size_t(lds) : 0;
    a.stream = c->stream;
    launch_stream_collide<C, FORCED>(a);
}

ForceField field(const lbm_ctx *c, int k) { return ForceField{c->force[k], c->mask[k]}; }
// The field that the step at hand spreads into.
int step_field(const lbm_ctx *c) { return c->own_held ? kThirdField : int(c->step & 1); }

// Blocks for the neighbour sums: kPairLanes lanes per particle.
dim3 pair_group_blocks(int32_t n) {
    return dim3(unsigned((size_t(n) * kPairLanes + kPairBlock - 1) / kPairBlock));
}

// Pair forces of the positions r: link the cell list, order long ones, then the
// neighbour sums.  The list heads are none before; the particle update that follows sets them
// back (its pair_head), or pair_list_clear does.
void launch_pairs(hipStream_t st, const double *r, int32_t n, const PairGrid &pg, const PairList &pl,
                  double *F) {
    const dim3 pblocks(unsigned((n + kPairBlock - 1) / kPairBlock));
    hipLaunchKernelGGL(k_pair_link, pblocks, dim3(kPairBlock), 0, st, r, n, pg, pl);
    if (pg.ordered) {
        hipLaunchKernelGGL(k_pair_order, pblocks, dim3(kPairBlock), 0, st, n, pg, pl);
        hipLaunchKernelGGL(k_pair_force<true>, pair_group_blocks(n), dim3(kPairBlock), 0, st, r, n, pg, pl, F);
    } else {
        hipLaunchKernelGGL(k_pair_force<false>, pair_group_blocks(n), dim3(kPairBlock), 0, st, r, n, pg, pl, F);
    }
}

hipError_t pair_list_clear(hipStream_t st, const PairList &pl, uint32_t T) {
    return hipMemsetAsync(pl.head, 0xFF, size_t(T) * 4, st);
}

// Returns the start event of a new timing pair (or nullptr when profiling is
// off); the caller records it before the launch and prof_stop after.
bool prof_grow(lbm_ctx *c) {
    const int32_t cap = c->prof_cap ? 2 * c->prof_cap : 256;
    hipEvent_t *ev = static_cast<hipEvent_t *>(realloc(c->prof_ev, sizeof(hipEvent_t) * 2 * cap));
    if (!ev) return false;
    c->prof_ev = ev;
    int32_t *kind = static_cast<int32_t *>(realloc(c->prof_kind, sizeof(int32_t) * cap));
    if (!kind) return false;
    c->prof_kind = kind;
    for (int32_t k = 2 * c->prof_cap; k < 2 * cap; ++k)
        if (hipEventCreate(&c->prof_ev[k]) != hipSuccess) return false;
    c->prof_cap = cap;
    return true;
}

int32_t prof_start(lbm_ctx *c, int32_t kind) {
    if (!c->prof_on) return -1;
    if (c->prof_used == c->prof_cap && !prof_grow(c)) return -1;
    const int32_t k = c->prof_used++;
    c->prof_kind[k] = kind;
    (void)hipEventRecord(c->prof_ev[2 * k], c->stream);
    return k;
}

void prof_stop(lbm_ctx *c, int32_t k) {
    if (k >= 0) (void)hipEventRecord(c->prof_ev[2 * k + 1], c->stream);
}

// Whether the state at the start of the step `ahead` steps from now is to be
// recorded (no recording in between).
bool sample_at(const lbm_ctx *c, int64_t ahead) {
    return c->series_every > 0 && (c->series_t + ahead) % c->series_every == 0 && c->series_count < c->series_cap;
}

// Arguments of this step's particle update; advances the VACF clock.
ParticleArgs step_particle_args(lbm_ctx *c) {
    ParticleArgs pa;
    pa.pmom = nullptr;
    pa.acc = nullptr;
    pa.origins = nullptr;
    pa.t = pa.k_lo = 0;
    pa.k_hi = -1;
    pa.nslot = pa.stride = 1;
    pa.max_lag = 0;
    pa.slot_lo = 0;
    if (c->vacf_on) {
        // active origins k*stride with t - max_lag <= k*stride <= t
        const int64_t t = c->vacf_t;
        pa.acc = c->acc;
        pa.origins = c->origins;
        pa.t = t;
        pa.k_hi = t / c->stride;
        pa.k_lo = t > c->max_lag ? (t - c->max_lag + c->stride - 1) / c->stride : 0;
        pa.nslot = c->nslot;
        pa.slot_lo = int32_t(pa.k_lo % c->nslot);
        pa.stride = c->stride;
        pa.max_lag = c->max_lag;
        c->vacf_t += 1;
    }
    pa.r = pa.r_out = c->r;
    pa.v = pa.v_out = c->v;
    pa.fh = c->fh;
    pa.fr = c->fr;
    // this step's nodes, and those still to be released: the last step's, and
    // after a two-step sweep the one's before it (kept where this step's go)
    pa.cells = c->cells[c->step & 1];
    pa.last_cells = c->cells[(c->step & 1) ^ 1];
    pa.older_cells = c->older_due ? pa.cells : nullptr;
    pa.err = c->err;
    pa.n = c->np;
    pa.friction = c->pdesc.friction;
    pa.mass = c->pdesc.mass;
    pa.gamma = c->pdesc.gamma;
    pa.sig = c->pdesc.kT > 0.0 ? sqrt(2.0 * c->pdesc.gamma * c->pdesc.kT) : 0.0;
    pa.R = c->R;
    pa.seed = c->pdesc.seed;
    pa.replica = c->pdesc.replica;
    pa.step = uint32_t(c->step);
    pa.fext = c->fext;
    pa.fpair = nullptr;
    pa.pair_link = nullptr;
    pa.pair_head = nullptr;
    if (c->pair_on) {
        launch_pairs(c->stream, c->r, c->np, c->pg, c->plist, c->fpair);
        pa.fpair = c->fpair;
        pa.pair_link = c->plist.link;
        pa.pair_head = c->plist.head;
    }
    return pa;
}

// The particle update of the step at hand; earlier fields are released with it.
template <class C>
void launch_particle(lbm_ctx *c, const typename C::T *A, const ParticleArgs &pa) {
    const int cur = step_field(c);
    hipLaunchKernelGGL(k_particle<C>, dim3(unsigned(particle_blocks(c->np))), dim3(particle_threads(pa)), 0, c->stream, A,
                       c->g, typename C::R(c->dec_s), pa, field(c, cur), field(c, c->last_field),
                       field(c, c->own_held ? int(c->step & 1) : kThirdField));
    c->fields_used = 1;
    c->last_field = cur;
    c->own_held = 0;
    c->older_due = 0;
}

// Releases the nodes of the last step and of the one before, lists of n entries.
__global__ __launch_bounds__(kBlock) void k_release(int32_t n, const uint32_t *last_cells, ForceField last,
                                                    const uint32_t *older_cells, ForceField older) {
    const int32_t i = int32_t(blockIdx.x * kBlock + threadIdx.x);
    if (i >= n) return;
    release_node(last, last_cells[i]);
    release_node(older, older_cells[i]);
}

// Leaves the fields as every call finds them: the last step's forces in its own
// field, those of the step before it in the third or released.  Only steps
// recorded between two-step sweeps can end otherwise.
void settle_fields(lbm_ctx *c) {
    const int last = int(c->step & 1) ^ 1;
    if (c->np == 0 || (!c->own_held && c->last_field == last)) return;
    hipLaunchKernelGGL(k_release, dim3(blocks_for(uint64_t(c->np) * 8)), dim3(kBlock), 0, c->stream, c->np * 8,
                       c->cells[last], field(c, c->last_field), c->cells[last ^ 1],
                       field(c, c->own_held ? last ^ 1 : kThirdField));
    c->last_field = last;
    c->own_held = 0;
}

template <class C>
void launch_step(lbm_ctx *c) {
    using T = typename C::T;
    const T *A = static_cast<const T *>(c->pop[c->cur]);
    T *B = static_cast<T *>(c->pop[c->cur ^ 1]);
    // Record the observables of the state at the start of this step?
    const bool sample = sample_at(c, 0);
    if (c->series_every > 0) c->series_t += 1;
    double *mom = sample ? c->fluid_partials : nullptr;
    if (c->np > 0) {
        const int32_t pk = prof_start(c, 1);
        ParticleArgs pa = step_particle_args(c);
        pa.pmom = sample ? c->part_partials : nullptr;
        launch_particle<C>(c, A, pa);
        prof_stop(c, pk);
        const int32_t ck = prof_start(c, 0);
        launch_collide<C, true>(c, A, B, field(c, c->last_field), c->shape, mom);
        prof_stop(c, ck);
    } else {
        const int32_t ck = prof_start(c, 0);
        launch_collide<C, false>(c, A, B, field(c, 0), c->shape, mom);
        prof_stop(c, ck);
    }
    if (sample) {
        const int32_t np_blocks = c->np > 0 ? int32_t(particle_blocks(c->np)) : 0;
        hipLaunchKernelGGL(k_series_stage1, dim3(kSeriesBlocks), dim3(kBlock), 0, c->stream,
                           c->fluid_partials,
                           int32_t(collide_grid(c, c->shape) * (config_block(c->shape) / 64)),
                           c->part_partials,
                           np_blocks, c->series_stage);
        hipLaunchKernelGGL(k_series_stage2, dim3(1), dim3(64), 0, c->stream, c->series_stage,
                           double(c->g.ncell), double(c->step), c->series + 8 * c->series_count);
        c->series_count += 1;
    }
    c->cur ^= 1;
    c->step += 1;
}

TwoStepArgs two_step_args(lbm_ctx *c, const TwoStepTiles &tl, bool nts, ForceField f0, ForceField f1) {
    TwoStepArgs a;
    a.A = c->pop[c->cur];
    a.B = c->pop[c->cur ^ 1];
    a.g = c->g;
    a.omega = c->omega;
    a.enc_s = c->enc_s;
    a.dec_s = c->dec_s;
    for (int k = 0; k < 3; ++k) a.body[k] = c->body[k];
    a.f0 = f0;
    a.f1 = f1;
    a.tl = tl;
    a.forced = c->np > 0;
    a.nts = nts;
    a.stream = c->stream;
    return a;
}

// Steps n and n + 1 in one sweep, neither of them recorded: both particle
// updates first (the second on the fluid around the particles one step ahead),
// then the two-step sweep.
template <class C>
void launch_two_step(lbm_ctx *c) {
    const int f0 = step_field(c), f1 = int(c->step & 1) ^ 1;
    const TwoStepArgs a = two_step_args(c, c->two_tiles, c->two_nts != 0, field(c, f0), field(c, f1));
    if (c->series_every > 0) c->series_t += 2;
    if (c->np > 0) {
        const typename C::T *A = static_cast<const typename C::T *>(a.A);
        int32_t pk = prof_start(c, 1);
        launch_particle<C>(c, A, step_particle_args(c));
        prof_stop(c, pk);
        c->step += 1;
        pk = prof_start(c, 1);
        ParticleArgs pa = step_particle_args(c);
        pa.last_cells = nullptr;  // the field of step n is still to be read
        if (c->pdesc.friction == LBM_FRICTION_BD)
            launch_particle<C>(c, A, pa);  // reads no fluid
        else
            launch_particle_ahead<C>(a, pa);
        prof_stop(c, pk);
        c->last_field = f1;
        c->own_held = f0 != kThirdField && c->pdesc.friction != LBM_FRICTION_BD;
        c->older_due = c->pdesc.friction != LBM_FRICTION_BD;
    } else {
        c->step += 1;
    }
    const int32_t ck = prof_start(c, 0);
    launch_two_steps<C>(a);
    prof_stop(c, ck);
    c->cur ^= 1;
    c->step += 1;
}

// Times stream-collide launches on A -> B without swapping (the simulation
// state in A is untouched; B is the next step's output anyway): ms[j] for
// the launch (ks[j], orders[j], caps[j]), -1 where it does not apply.  With
// particles attached the forced variant is timed, reading the node forces of
// the last step (still in place until the next particle kernel).
template <class C>
void time_launches(lbm_ctx *c, int32_t iters, int n, const int *ks, const int *orders,
                   const int *caps, double *ms, hipError_t *err) {
    using T = typename C::T;
    const T *A = static_cast<const T *>(c->pop[c->cur]);
    T *B = static_cast<T *>(c->pop[c->cur ^ 1]);
    hipEvent_t e0, e1;
    *err = hipEventCreate(&e0);
    if (*err == hipSuccess) *err = hipEventCreate(&e1);
    if (*err != hipSuccess) return;
    const bool forced = c->np > 0;
    const ForceField last = field(c, c->last_field);
    for (int j = 0; j < n && *err == hipSuccess; ++j) {
        const int k = ks[j], order = orders[j], cap = caps[j];
        ms[j] = -1.0;
        if (!shape_ok(c, k) || (config_row(k) && row_mapping_is_flat(c->g.nx))) continue;
        if (sweep_lds(c, cap, config_block(k)) < 0) continue;
        auto launch = [&]() {
            if (forced)
                launch_collide<C, true>(c, A, B, last, k, nullptr, order, cap);
            else
                launch_collide<C, false>(c, A, B, last, k, nullptr, order, cap);
        };
        for (int w = 0; w < 2; ++w) launch();
        (void)hipEventRecord(e0, c->stream);
        for (int it = 0; it < iters; ++it) launch();
        (void)hipEventRecord(e1, c->stream);
        *err = hipEventSynchronize(e1);
        float t = 0.0f;
        if (*err == hipSuccess) *err = hipEventElapsedTime(&t, e0, e1);
        ms[j] = double(t) / iters;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
}

// Mean time per launch of the streaming-only kernel in configuration k with
// the context's block order and residency cap, over iters launches (A -> B,
// as the autotuner's trial launches).
template <class C, int CPT, int BS, bool NTS, bool ROW>
void stream_only_shape(lbm_ctx *c, const typename C::T *A, typename C::T *B, unsigned grid,
                       uint32_t order, size_t dyn) {
    const int addr = sweep_addr<C>(c->g, ROW);
    if constexpr (ROW) {
        hipLaunchKernelGGL((k_stream_only<C, CPT, BS, NTS, ROW, kAddrRow>), dim3(grid), dim3(BS), dyn,
                           c->stream, A, B, c->g, order);
    } else {
        if constexpr (sizeof(typename C::T) == 2)
            if (addr == kAddrRow) {
                hipLaunchKernelGGL((k_stream_only<C, CPT, BS, NTS, ROW, kAddrRow>), dim3(grid), dim3(BS), dyn,
                                   c->stream, A, B, c->g, order);
                return;
            }
        if (addr == kAddrLane64)
            hipLaunchKernelGGL((k_stream_only<C, CPT, BS, NTS, ROW, kAddrLane64>), dim3(grid), dim3(BS),
                               dyn, c->stream, A, B, c->g, order);
        else
            hipLaunchKernelGGL((k_stream_only<C, CPT, BS, NTS, ROW, kAddrLane32>), dim3(grid), dim3(BS),
                               dyn, c->stream, A, B, c->g, order);
    }
}

template <class C>
void time_stream_only(lbm_ctx *c, int k, int32_t iters, double *ms, hipError_t *err) {
    using T = typename C::T;
    const T *A = static_cast<const T *>(c->pop[c->cur]);
    T *B = static_cast<T *>(c->pop[c->cur ^ 1]);
    const unsigned grid = collide_grid(c, k);
    const long lds = sweep_lds(c, c->cap, config_block(k));
    const size_t dyn = lds > 0 ? size_t(lds) : 0;
    const uint32_t order = uint32_t(c->order);
    auto launch = [&]() {
#define LBM_STREAM_ONLY(CPT, BS, NTS, ROW) stream_only_shape<C, CPT, BS, NTS, ROW>(c, A, B, grid, order, dyn)
        LBM_CONFIG_SWITCH(k, LBM_STREAM_ONLY)
#undef LBM_STREAM_ONLY
    };
    hipEvent_t e0, e1;
    *err = hipEventCreate(&e0);
    if (*err == hipSuccess) *err = hipEventCreate(&e1);
    if (*err != hipSuccess) return;
    for (int w = 0; w < 2; ++w) launch();
    (void)hipEventRecord(e0, c->stream);
    for (int it = 0; it < iters; ++it) launch();
    (void)hipEventRecord(e1, c->stream);
    *err = hipEventSynchronize(e1);
    float t = 0.0f;
    if (*err == hipSuccess) *err = hipEventElapsedTime(&t, e0, e1);
    *ms = double(t) / iters;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
}

// Leaves lattice A (unchanged) and the other lattice in the last-level cache as a
// step's sweep does that wrote A and read the other: 16-byte words, n of each.
__global__ __launch_bounds__(kBlock) void k_as_in_a_run(void *A, const void *other, size_t n, int nts) {
    typedef uint32_t word __attribute__((ext_vector_type(4)));
    for (size_t i = size_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += size_t(gridDim.x) * kBlock) {
        word a = static_cast<word *>(A)[i];
        const word b = static_cast<const word *>(other)[i];
        asm volatile("" : "+v"(a) : "v"(b));  // both are loaded
        if (nts)
            __builtin_nontemporal_store(a, static_cast<word *>(A) + i);
        else
            static_cast<word *>(A)[i] = a;
    }
}

// Mean ms of a sweep A -> B launched by `launch`, each after the lattices (bytes
// each) have been left as in a run.  Trials that launch the same sweep over and
// over read from the last-level cache what a run has written past it: by those
// 16-bit 192^3 (256 MiB) took single steps, 0.129 against 0.143 ms, which a run
// does in 0.187 and 0.142.  Lattices beyond one and a half times that cache are
// launched over and over, within 1% of a run (FP32 320 x 200 x 150, 700 MiB, two
// single steps 0.468 ms in a run, 0.468 so, 0.554 after the kernel above).
template <typename Launch>
double time_as_in_a_run(hipStream_t st, void *A, const void *B, size_t bytes, bool nts, int32_t iters, Launch &&launch,
                        hipError_t *err) {
    hipEvent_t e0, e1;
    *err = hipEventCreate(&e0);
    if (*err != hipSuccess) return -1.0;
    *err = hipEventCreate(&e1);
    if (*err != hipSuccess) {
        (void)hipEventDestroy(e0);
        return -1.0;
    }
    const bool cached = bytes < kStreamStoreBytes + kStreamStoreBytes / 2;
    double sum = 0.0;
    float t = 0.0f;
    for (int32_t it = -2; it < iters && *err == hipSuccess; ++it) {
        if (cached) hipLaunchKernelGGL(k_as_in_a_run, dim3(2048), dim3(kBlock), 0, st, A, B, bytes / 16, int(nts));
        if (cached || it == 0) (void)hipEventRecord(e0, st);
        launch();
        if (!cached && it + 1 < iters) continue;
        (void)hipEventRecord(e1, st);
        *err = hipEventSynchronize(e1);
        if (*err == hipSuccess) *err = hipEventElapsedTime(&t, e0, e1);
        if (it >= 0) sum += double(t);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return sum / iters;
}

// Mean ms of two single steps of the context's configuration (tl null), or of one
// two-step sweep with these tiles, as in a run.
template <class C>
void time_two_steps(lbm_ctx *c, const TwoStepTiles *tl, int32_t iters, double *ms, hipError_t *err) {
    size_t bytes = 0;
    lbm_lattice_bytes(&c->desc, &bytes);
    const ForceField last = field(c, c->last_field);
    void *A = c->pop[c->cur], *B = c->pop[c->cur ^ 1];
    if (tl) {
        const TwoStepArgs a = two_step_args(c, *tl, c->two_nts != 0, last, last);
        *ms = time_as_in_a_run(c->stream, A, B, bytes, c->two_nts != 0, iters, [&] { launch_two_steps<C>(a); }, err);
    } else {
        using T = typename C::T;
        *ms = 2.0 * time_as_in_a_run(c->stream, A, B, bytes, config_nts(c->shape), iters, [&] {
            if (c->np > 0)
                launch_collide<C, true>(c, static_cast<const T *>(A), static_cast<T *>(B), last, c->shape);
            else
                launch_collide<C, false>(c, static_cast<const T *>(A), static_cast<T *>(B), last, c->shape);
        }, err);
    }
}

template <class C>
void launch_get_populations(lbm_ctx *c, double *f) {
    hipLaunchKernelGGL(k_get_populations<C>, dim3(blocks_for(c->g.ncell)), dim3(kBlock), 0,
                       c->stream, static_cast<const typename C::T *>(c->pop[c->cur]), c->g,
                       typename C::R(c->dec_s), f);
}

template <class C>
void launch_get_moments(lbm_ctx *c, double *rho, double *u) {
    hipLaunchKernelGGL(k_get_moments<C>, dim3(blocks_for(c->g.ncell)), dim3(kBlock), 0,
                       c->stream, static_cast<const typename C::T *>(c->pop[c->cur]), c->g,
                       typename C::R(c->dec_s), rho, u);
}

template <class C>
void launch_set_populations(lbm_ctx *c, const double *f) {
    hipLaunchKernelGGL(k_set_populations<C>, dim3(blocks_for(c->g.ncell)), dim3(kBlock), 0,
                       c->stream, f, static_cast<typename C::T *>(c->pop[c->cur]), c->g,
                       typename C::R(c->enc_s));
}

template <class C>
void launch_set_equilibrium(lbm_ctx *c, const double *rho, const double *u) {
    hipLaunchKernelGGL(k_set_equilibrium<C>, dim3(blocks_for(c->g.ncell)), dim3(kBlock), 0,
                       c->stream, rho, u, static_cast<typename C::T *>(c->pop[c->cur]), c->g,
                       typename C::R(c->enc_s));
}

template <class C>
void launch_partials(lbm_ctx *c, double *partials) {
    hipLaunchKernelGGL(k_fluid_partials<C>, dim3(kRedBlocks), dim3(kBlock), 0, c->stream,
                       static_cast<const typename C::T *>(c->pop[c->cur]), c->g,
                       typename C::R(c->dec_s), partials);
}

// Moves the state into the layout with Y rows per group: the current lattice
// is permuted into the spare one and copied back, so the current populations
// stay in the same buffer.
template <class C>
void launch_relayout(lbm_ctx *c, uint32_t Y, hipError_t *err) {
    const Grid gn = with_rows_per_group(c->g, Y);
    hipLaunchKernelGGL(k_relayout<C>, dim3(blocks_for(c->g.ncell)), dim3(kBlock), 0, c->stream,
                       static_cast<const typename C::T *>(c->pop[c->cur]), c->g,
                       static_cast<typename C::T *>(c->pop[c->cur ^ 1]), gn);
    size_t lat = 0;
    lbm_lattice_bytes(&c->desc, &lat);
    *err = hipMemcpyAsync(c->pop[c->cur], c->pop[c->cur ^ 1], lat, hipMemcpyDeviceToDevice,
                          c->stream);
    c->g = gn;
}

// The storage codec x velocity set combinations the library instantiates.
using F64Q19 = Cfg<CodecF64, D3Q19>;
using F32Q19 = Cfg<CodecF32, D3Q19>;
using BF16Q19 = Cfg<CodecBF16, D3Q19>;
using F16Q19 = Cfg<CodecF16, D3Q19>;
using F64Q15 = Cfg<CodecF64, D3Q15>;
using F32Q15 = Cfg<CodecF32, D3Q15>;
using BF16Q15 = Cfg<CodecBF16, D3Q15>;
using F16Q15 = Cfg<CodecF16, D3Q15>;

#define LBM_DISPATCH(ctx, FN, ...)                                                      \
    do {                                                                                \
        if ((ctx)->q == 15) {                                                           \
            switch ((ctx)->desc.storage) {                                              \
                case LBM_STORE_F64: FN<F64Q15>(ctx, ##__VA_ARGS__); break;              \
                case LBM_STORE_F32: FN<F32Q15>(ctx, ##__VA_ARGS__); break;              \
                case LBM_STORE_BF16: FN<BF16Q15>(ctx, ##__VA_ARGS__); break;            \
                case LBM_STORE_F16: FN<F16Q15>(ctx, ##__VA_ARGS__); break;              \
            }                                                                           \
        } else {                                                                        \
            switch ((ctx)->desc.storage) {                                              \
                case LBM_STORE_F64: FN<F64Q19>(ctx, ##__VA_ARGS__); break;              \
                case LBM_STORE_F32: FN<F32Q19>(ctx, ##__VA_ARGS__); break;              \
                case LBM_STORE_BF16: FN<BF16Q19>(ctx, ##__VA_ARGS__); break;            \
                case LBM_STORE_F16: FN<F16Q19>(ctx, ##__VA_ARGS__); break;              \
            }                                                                           \
        }                                                                               \
    } while (0)

}  // namespace

extern "C" {

lbm_status lbm_lattice_bytes(const lbm_grid_desc *grid, size_t *bytes) {
    if (!grid_ok(grid) || !bytes) return LBM_E_INVAL;
    *bytes = align_up(size_t(row_chunk(grid)) * size_t(velocity_count(grid)) * size_t(grid->ny) *
                          size_t(grid->nz) *
                          elem_size(grid->storage),
                      kAlign);
    return LBM_OK;
}

lbm_status lbm_grid_scratch_bytes(const lbm_grid_desc *grid, size_t *bytes) {
    if (!grid_ok(grid) || !bytes) return LBM_E_INVAL;
    *bytes = grid_scratch_size(grid);
    return LBM_OK;
}

lbm_status lbm_particle_scratch_bytes(const lbm_grid_desc *grid, int32_t n, size_t *bytes) {
    if (!grid_ok(grid) || !bytes || n < 0 || n > (1 << 24)) return LBM_E_INVAL;
    *bytes = particle_scratch_size(grid, n);
    return LBM_OK;
}

lbm_status lbm_vacf_origin_bytes(int32_t n, int32_t max_lag, int32_t stride, size_t *bytes) {
    if (!bytes || n < 0 || max_lag < 0 || stride < 1) return LBM_E_INVAL;
    *bytes = size_t(max_lag / stride + 1) * size_t(n) * 3 * sizeof(double);
    return LBM_OK;
}

}  // extern "C"

// Device memory of lbm_observables_noalloc: the FP64 reduction partials
// ([kRedBlocks][4]) followed by the seven sums.  Every device the library runs
// on holds one copy until the process ends.  Host code never passes this name
// to a kernel or a copy (on the host it is only a stand-in for the symbol):
// it uses the device address that hipGetSymbolAddress returned for that
// device, kept in g_noalloc below.
constexpr size_t kNoAllocDoubles = size_t(kRedBlocks) * 4 + 8;
static __device__ __align__(256) double scratch[kNoAllocDoubles];

namespace {

// Device address of `scratch` per device, looked up once per device by
// lbm_init (with that device current).
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
bool g_noalloc_done[kMaxDevices];
double *g_noalloc[kMaxDevices];

void noalloc_setup(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return;
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (g_noalloc_done[dev]) return;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_noalloc[dev] = (e == hipSuccess) ? static_cast<double *>(p) : nullptr;
    g_noalloc_done[dev] = true;
}

double *noalloc_scratch(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    return g_noalloc[dev];
}

}  // namespace

namespace {

// Launch configurations the autotuners chose, kept for the life of the
// process and keyed by device, storage, velocity set and the sizes of every
// box: a context or ensemble created later with the same key starts from that
// choice instead of the size-based default.
struct TuneKey {
    int kind;  // 0 single box (its code holds configuration, order and cap), 1 ensemble
    int device, storage, q;
    std::vector<int32_t> dims;  // nx, ny, nz of each box
    bool operator<(const TuneKey &o) const {
        return std::tie(kind, device, storage, q, dims) <
               std::tie(o.kind, o.device, o.storage, o.q, o.dims);
    }
};

std::mutex g_tune_mu;
std::map<TuneKey, int> g_tune;

int current_device() {
    int d = 0;
    return hipGetDevice(&d) == hipSuccess ? d : -1;
}

int tune_lookup(const TuneKey &k, int fallback) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    const auto it = g_tune.find(k);
    return it == g_tune.end() ? fallback : it->second;
}

void tune_store(const TuneKey &k, int shape) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tune[k] = shape;
}

// A single-box choice is kept as one code: configuration, block order,
// residency cap and layout (log2 of the rows per group); an ensemble's code
// holds the same four, its layout being the rows per group requested of
// every box.
int tune_code(int shape, int order, int cap, int rows_log2) {
    return shape + kNumShapes * (order + int(kNumOrders) * (cap + kNumCaps * rows_log2));
}

int rows_log2(const Grid &g) {
    int k = 0;
    while ((1u << k) < g.ymask + 1u) ++k;
    return k;
}

// Layouts of the lattice: 1, 2, 4, ..., 64 rows per group, those that divide ny.
constexpr int kMaxRowsLog2 = 6;

int layout_candidates(const lbm_ctx *c, uint32_t *ys) {
    int n = 0;
    for (int k = 0; k <= kMaxRowsLog2; ++k)
        if (c->g.ny % (1u << k) == 0) ys[n++] = 1u << k;
    return n;
}

// Puts the state into the layout with Y rows per group (no change of value).
lbm_status set_layout(lbm_ctx *c, uint32_t Y) {
    if (Y == c->g.ymask + 1u) return LBM_OK;
    hipError_t err = hipSuccess;
    LBM_DISPATCH(c, launch_relayout, Y, &err);
    const lbm_status st = launch_status();
    return err != hipSuccess ? LBM_E_DEVICE : st;
}

// ---- two-step sweep: tiles and when it is used ----

// Tiles of the two-step sweep for a box, best first by a cost model: a block
// takes lz planes and a start of two more; a plane costs the wavefronts of its
// two steps on the busiest of the compute unit's four SIMDs, plus the 128-byte
// lines that its row pieces touch; blocks run one per compute unit (the LDS and
// registers of a block this size allow no second one), so whole rounds of 256
// count.  In runs of 55 boxes of every storage, 40 to 320 nodes long, the model's
// first choice takes 2.5% more than the fastest of its first six on average, and
// 14% at most (FP32 56^3 11.7 and 10.3 us a sweep; of the boxes that take such
// sweeps untuned BF16 130 x 129 x 130 50.8 and 45.3, F16 D3Q15 250 x 130 x 77 47.9
// and 43.3).  lbm_autotune times those six.
constexpr int kTwoStepCandidates = 6;

double two_step_plane_cost(uint32_t tx, uint32_t ty, size_t elem) {
    const double lines = (ty + 2) * ((tx + 2) * double(elem) / 128.0 + 1.5);
    const uint32_t first = ((tx + 2) * (ty + 2) + 63) / 64, second = (tx * ty + 63) / 64;  // wavefronts
    return double((first + 3) / 4 + (second + 3) / 4) + 0.4 * lines;
}

constexpr uint32_t kTwoStepUnits = 256;
constexpr double kTwoStepStart = 2.0;

// Whether population rows are whole 128-byte lines.
bool rows_are_lines(uint32_t nx, size_t elem) { return nx * elem % 128 == 0; }

// Calls fn(tx, ty, ntx, nty) for every even split of an nx x ny plane into tiles
// that fit a block (rows of 16 nodes at least, unless nx is shorter).  Where
// rows are whole lines, so are the tiles' pieces of them: a line written by two
// blocks costs far more than an uneven last tile (256^3 FP32, tiles of 52 x 11
// and 43 x 13 nodes 0.907 and 1.294 ms, 64 x 8 0.486).
template <typename Fn>
void two_step_each_tile(uint32_t nx, uint32_t ny, size_t elem, Fn &&fn) {
    const uint32_t most = two_step_nodes(elem);
    const uint32_t line = rows_are_lines(nx, elem) ? uint32_t(128 / elem) : 1;
    uint32_t last_tx = 0;
    for (uint32_t split = 1; split <= nx; ++split) {
        const uint32_t tx = ((nx + split - 1) / split + line - 1) / line * line, ntx = (nx + tx - 1) / tx;
        if (tx < 16 && split > 1) break;
        if ((tx + 2) * 3 > most || tx == last_tx) continue;
        last_tx = tx;
        uint32_t last = 0;
        for (uint32_t top = std::min(ny, most / (tx + 2) - 2); top >= 1; --top) {
            const uint32_t nty = (ny + top - 1) / top, ty = (ny + nty - 1) / nty;
            if (ty != last) fn(tx, ty, ntx, nty);
            last = ty;
        }
    }
}

int two_step_candidates(const lbm_grid_desc *g, TwoStepTiles *out) {
    const uint32_t nx = uint32_t(g->nx), ny = uint32_t(g->ny), nz = uint32_t(g->nz);
    const size_t elem = elem_size(g->storage);
    if (!two_step_planes(g)) return 0;
    struct Cand {
        TwoStepTiles tl;
        double cost;
    };
    std::vector<Cand> all;
    two_step_each_tile(nx, ny, elem, [&](uint32_t tx, uint32_t ty, uint32_t ntx, uint32_t nty) {
        const double plane = two_step_plane_cost(tx, ty, elem);
        const uint64_t tiles = uint64_t(ntx) * nty;
        const uint64_t r0 = (tiles + kTwoStepUnits - 1) / kTwoStepUnits;
        Cand best{{}, -1.0};
        for (uint64_t r = r0; r < r0 + 8; ++r) {  // rounds of blocks
            const uint32_t ns = uint32_t(std::min<uint64_t>(nz, r * kTwoStepUnits / tiles));
            const uint32_t lz = (nz + ns - 1) / ns;
            const double cost = double(r) * (lz + kTwoStepStart) * plane;
            if (best.cost < 0.0 || cost < best.cost) best = Cand{{tx, ty, lz, ntx, nty, (nz + lz - 1) / lz}, cost};
        }
        all.push_back(best);
    });
    std::sort(all.begin(), all.end(), [](const Cand &x, const Cand &y) { return x.cost < y.cost; });
    const int n = int(std::min<size_t>(kTwoStepCandidates, all.size()));
    for (int k = 0; k < n; ++k) out[k] = all[k].tl;
    return n;
}

// Store policy of the two-step sweep: non-temporal once the two lattices
// outgrow the 256 MB last-level cache, where rows are whole lines (two sweeps
// in turn, ms plain / non-temporal: BF16 128^3, 80 MB a lattice, 0.0437 /
// 0.0488; FP32 128^3, 159 MB, 0.0717 / 0.0673; FP32 256^3 0.502 / 0.486).
// Other rows leave lines that two tiles write, which a cache has to join (FP32
// 250^3, 1.19 GB, 0.522 / 0.565; BF16 300 x 200 x 150, 342 MB, 0.214 / 0.220).
constexpr size_t kTwoStepStreamBytes = size_t(128) << 20;

// Boxes of fewer nodes than this take single steps until tuned: a block's two
// planes of start are too large a part of its slab (us per step in a run, two-
// step / single: FP32 64^3 5.8 / 7.0, 80^3 8.8 / 12.0; FP64 64^3 10.9 / 12.3; BF16
// 72^3 7.5 / 6.6, 96^3 11.3 / 12.5).
constexpr uint64_t two_step_min_nodes(size_t elem) { return uint64_t(1) << (elem == 2 ? 19 : 18); }

bool two_step_by_size(const lbm_grid_desc *g) { return ncell_of(g) >= two_step_min_nodes(elem_size(g->storage)); }

// Boxes in which lbm_autotune tries the two-step sweep.  In smaller ones a launch
// is a few us of latency, which trials do not tell apart (two steps in a run /
// by trial, us, single and two-step: BF16 64^3 10.0 and 12.1 / 19.7 and 14.6, 72^3
// 13.1 and 14.5 / 25.2 and 17.1; but FP32 48^3 11.3 and 9.4 / 18.6 and 13.5, FP64
// 48^3 16.3 and 12.9 / 19.1 and 15.4).  In 44 of 45 larger ones the trials' choice was
// the run's fastest or within 5% of it (F16 201 x 150 x 117, a tie by trial, went to
// the slower side by 21% in one of three sets).
bool two_step_trial(const lbm_grid_desc *g) {
    return ncell_of(g) >= (elem_size(g->storage) == 2 ? two_step_min_nodes(2) : uint64_t(1) << 16);
}

// The tiles of choice `two` (1: the model's first); 0 where the box has none.
TwoStepTiles two_step_tiles(const lbm_grid_desc *g, int &two) {
    TwoStepTiles tl[kTwoStepCandidates] = {};
    if (two > 0 && two > two_step_candidates(g, tl)) two = 0;
    return tl[two > 0 ? two - 1 : 0];
}

bool two_step_pays(const lbm_ctx *c) {
    // (BD friction reads no fluid and spreads nothing: no update ahead, no fields)
    return c->np == 0 || c->pdesc.friction == LBM_FRICTION_BD || c->force[kThirdField];
}

// The remembered code of a box holds, above the single-step launch, the
// two-step choice plus one.
constexpr int kTuneTwo = kNumShapes * int(kNumOrders) * kNumCaps * (kMaxRowsLog2 + 1);

TuneKey ctx_tune_key(const lbm_ctx *c) {
    return TuneKey{0, c->device, c->desc.storage, c->q, {c->desc.nx, c->desc.ny, c->desc.nz}};
}

}  // namespace

extern "C" {

lbm_status lbm_init(const lbm_grid_desc *grid, void *pop_a, void *pop_b, void *grid_scratch,
                    void *stream, lbm_ctx **out) {
    if (!grid_ok(grid) || !pop_a || !pop_b || !grid_scratch || !out) return LBM_E_INVAL;
    if (!aligned(pop_a) || !aligned(pop_b) || !aligned(grid_scratch) || pop_a == pop_b)
        return LBM_E_INVAL;
    lbm_ctx *c = static_cast<lbm_ctx *>(calloc(1, sizeof(lbm_ctx)));
    if (!c) return LBM_E_DEVICE;
    uint32_t init_rows = 1;
    c->desc = *grid;
    c->g.nx = uint32_t(grid->nx);
    c->g.ny = uint32_t(grid->ny);
    c->g.nz = uint32_t(grid->nz);
    c->g.ncell = uint32_t(ncell_of(grid));
    c->g.chunk = row_chunk(grid);
    c->g = with_rows_per_group(c->g, 1);
    c->q = velocity_count(grid);
    c->device = current_device();
    noalloc_setup(c->device);
    {
        size_t lat = 0;
        lbm_lattice_bytes(grid, &lat);
        // until lbm_autotune: the last choice for this key, else the row-aligned
        // mapping for rows that are not whole wavefronts (and long enough that
        // idle lanes are few), else by lattice size
        const int fallback = (grid->nx % 64 != 0 && grid->nx >= 96) ? kNumFlatShapes
                             : lat >= kStreamStoreBytes              ? kNumGeomShapes
                                                                     : 0;
        const int code = tune_lookup(ctx_tune_key(c), fallback);
        c->shape = code % kNumShapes;
        c->order = (code / kNumShapes) % int(kNumOrders);
        c->cap = (code / (kNumShapes * int(kNumOrders))) % kNumCaps;
        // the remembered layout, applied once the lattices are at rest below
        init_rows = uint32_t(1) << ((code / (kNumShapes * int(kNumOrders) * kNumCaps)) % (kMaxRowsLog2 + 1));
        const int two = code / kTuneTwo;  // remembered two-step choice + 1, 0: none
        c->two = two > 0 ? two - 1 : two_step_by_size(grid);
        c->two_nts = lat >= kTwoStepStreamBytes && rows_are_lines(c->g.nx, elem_size(grid->storage));
        c->two_tiles = two_step_tiles(grid, c->two);
        if (grid->ny % int32_t(init_rows) != 0) init_rows = 1;
        // LDS limits of the device, for the residency caps (none if unknown)
        int v = 0;
        c->lds_cu = (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                                           c->device) == hipSuccess) ? v : 0;
        c->lds_block = (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock,
                                              c->device) == hipSuccess) ? v : 0;
        if (sweep_lds(c, c->cap, config_block(c->shape)) < 0) c->cap = 0;
    }
    c->elem = elem_size(grid->storage);
    c->pop[0] = pop_a;
    c->pop[1] = pop_b;
    c->cur = 0;
    c->stream = static_cast<hipStream_t>(stream);
    c->omega = 1.0 / grid->tau;
    if (grid->storage == LBM_STORE_F16) {
        c->enc_s = ldexp(1.0, grid->f16_scale_log2);
        c->dec_s = ldexp(1.0, -grid->f16_scale_log2);
    } else {
        c->enc_s = c->dec_s = 1.0;
    }
    char *s = static_cast<char *>(grid_scratch);
    c->mask_words = mask_words(c->g.ncell);
    for (int k = 0; k < kThirdField; ++k) {
        c->mask[k] = reinterpret_cast<uint32_t *>(s);
        s += align_up(size_t(c->mask_words) * 4, kAlign);
    }
    for (int k = 0; k < kThirdField; ++k) {
        c->force[k] = reinterpret_cast<long long *>(s);
        s += force_field_bytes(grid);
    }
    c->fluid_partials = reinterpret_cast<double *>(s);
    s += fluid_partials_bytes(grid);
    // every configuration's grid must fit the per-wavefront partials
    for (int k = 0; k < kNumShapes; ++k)
        if (shape_ok(c, k) &&
            size_t(collide_grid(c, k)) * (config_block(k) / 64) * 4 * 8 > fluid_partials_bytes(grid)) {
            free(c);
            return LBM_E_UNSUPPORTED;
        }
    c->series_stage = reinterpret_cast<double *>(s);
    s += align_up(size_t(kSeriesBlocks) * 7 * 8, kAlign);
    c->partials = reinterpret_cast<double *>(s);
    s += align_up(size_t(kRedBlocks) * 4 * 8, kAlign);
    c->result = reinterpret_cast<double *>(s);
    s += align_up(8 * 8, kAlign);
    c->err = reinterpret_cast<uint32_t *>(s);
    c->R = -1.0;

    size_t lat;
    lbm_lattice_bytes(grid, &lat);
    hipError_t e = hipMemsetAsync(pop_a, 0, lat, c->stream);  // g = 0 is the rest state
    if (e == hipSuccess) e = hipMemsetAsync(pop_b, 0, lat, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(grid_scratch, 0, grid_scratch_size(grid), c->stream);
    if (e != hipSuccess) {
        free(c);
        return LBM_E_DEVICE;
    }
    // the rest state is all zeros in every layout
    c->g = with_rows_per_group(c->g, init_rows);
    *out = c;
    return LBM_OK;
}

lbm_status lbm_set_equilibrium(lbm_ctx *ctx, const double *rho, const double *u) {
    if (!ctx) return LBM_E_INVAL;
    LBM_DISPATCH(ctx, launch_set_equilibrium, rho, u);
    return launch_status();
}

lbm_status lbm_set_populations(lbm_ctx *ctx, const double *f) {
    if (!ctx || !f) return LBM_E_INVAL;
    LBM_DISPATCH(ctx, launch_set_populations, f);
    return launch_status();
}

lbm_status lbm_set_body_force(lbm_ctx *ctx, const double *g) {
    if (!ctx) return LBM_E_INVAL;
    double v[3] = {0.0, 0.0, 0.0};
    if (g) {
        for (int k = 0; k < 3; ++k) {
            if (!isfinite(g[k])) return LBM_E_INVAL;
            v[k] = g[k];
        }
    }
    for (int k = 0; k < 3; ++k) ctx->body[k] = v[k];
    return LBM_OK;
}

lbm_status lbm_get_populations(lbm_ctx *ctx, double *f) {
    if (!ctx || !f) return LBM_E_INVAL;
    LBM_DISPATCH(ctx, launch_get_populations, f);
    return launch_status();
}

lbm_status lbm_get_moments(lbm_ctx *ctx, double *rho, double *u) {
    if (!ctx || (!rho && !u)) return LBM_E_INVAL;
    LBM_DISPATCH(ctx, launch_get_moments, rho, u);
    return launch_status();
}

lbm_status particles_couple(lbm_ctx *ctx, const lbm_particle_desc *d, double *r, double *v,
                            void *particle_scratch) {
    if (!ctx || !d) return LBM_E_INVAL;
    if (d->n < 0 || d->n > (1 << 24) || d->reserved != 0) return LBM_E_INVAL;
    if (d->n > 0) {
        if (!r || !v || !particle_scratch || !aligned(particle_scratch)) return LBM_E_INVAL;
        if (!(d->mass > 0.0) || !isfinite(d->mass)) return LBM_E_INVAL;
        if (!(d->gamma >= 0.0) || !isfinite(d->gamma)) return LBM_E_INVAL;
        if (!(d->kT >= 0.0) || !isfinite(d->kT)) return LBM_E_INVAL;
        if (!isfinite(d->radius)) return LBM_E_INVAL;
        if (d->friction < LBM_FRICTION_STOKESLET || d->friction > LBM_FRICTION_STOKESLET_CUBE)
            return LBM_E_INVAL;
    }
    // Node forces left by any previous particle set are cleared (the fields lie
    // back to back: the masks, then the forces; lbm_init cleared them first).
    hipError_t e = hipSuccess;
    if (ctx->fields_used) {
        e = hipMemsetAsync(ctx->mask[0], 0, kThirdField * align_up(size_t(ctx->mask_words) * 4, kAlign), ctx->stream);
        if (e == hipSuccess)
            e = hipMemsetAsync(ctx->force[0], 0, kThirdField * force_field_bytes(&ctx->desc), ctx->stream);
        if (e != hipSuccess) return LBM_E_DEVICE;
    }
    ctx->fields_used = 0;
    ctx->last_field = int(ctx->step & 1) ^ 1;
    ctx->own_held = 0;
    ctx->mask[kThirdField] = nullptr;
    ctx->force[kThirdField] = nullptr;
    ctx->vacf_on = 0;
    ctx->fext = nullptr;
    ctx->pair_on = 0;
    ctx->np = d->n;
    ctx->pdesc = *d;
    ctx->warnings = 0;
    if (d->n == 0) {
        ctx->R = -1.0;
        return LBM_OK;
    }
    // Stokes' law gamma = 6 pi eta R, eta = rho0 nu, nu = (tau - 1/2)/3.
    const double nu = (ctx->desc.tau - 0.5) / 3.0;
    ctx->R = d->radius > 0.0 ? d->radius : d->gamma / (6.0 * M_PI * nu);
    ctx->warnings = coupling_warnings(d->friction, ctx->R, d->n, double(ctx->g.ncell));
    ctx->r = r;
    ctx->v = v;
    char *s = static_cast<char *>(particle_scratch);
    for (int k = 0; k < 2; ++k) {
        ctx->cells[k] = reinterpret_cast<uint32_t *>(s);
        s += align_up(size_t(d->n) * 8 * 4, kAlign);
    }
    ctx->part_partials = reinterpret_cast<double *>(s);
    s += align_up(particle_blocks(d->n) * 3 * 8, kAlign);
    ctx->fh = reinterpret_cast<double *>(s);
    s += align_up(size_t(d->n) * 3 * 8, kAlign);
    ctx->fr = reinterpret_cast<double *>(s);
    s += align_up(size_t(d->n) * 3 * 8, kAlign);
    ctx->plist = pair_list_at(s, d->n);
    s += pair_list_bytes(d->n);
    ctx->fpair = reinterpret_cast<double *>(s);
    s += align_up(size_t(d->n) * 3 * 8, kAlign);
    const size_t third = third_field_bytes(&ctx->desc);
    if (third && two_step_pays(ctx->elem, ctx->q, ctx->g.ncell, d->n)) {
        ctx->mask[kThirdField] = reinterpret_cast<uint32_t *>(s);
        ctx->force[kThirdField] = reinterpret_cast<long long *>(s + align_up(size_t(ctx->mask_words) * 4, kAlign));
        e = hipMemsetAsync(s, 0, third, ctx->stream);
        if (e != hipSuccess) return LBM_E_DEVICE;
    }
    // nodes spread to -> kNoNode (all ones), list heads -> none; forces zero.
    e = hipMemsetAsync(ctx->cells[0], 0xFF, 2 * align_up(size_t(d->n) * 8 * 4, kAlign), ctx->stream);
    if (e == hipSuccess && d->n <= kPairMax)
        e = pair_list_clear(ctx->stream, ctx->plist, pair_buckets(d->n));
    if (e == hipSuccess) e = hipMemsetAsync(ctx->fh, 0, size_t(d->n) * 3 * 8, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->fr, 0, size_t(d->n) * 3 * 8, ctx->stream);
    return e == hipSuccess ? LBM_OK : LBM_E_DEVICE;
}

lbm_status lbm_set_pair_force(lbm_ctx *ctx, double a_f, double r_c) {
    if (!ctx || !isfinite(a_f) || !isfinite(r_c)) return LBM_E_INVAL;
    if (a_f == 0.0) {
        ctx->pair_on = 0;
        return LBM_OK;
    }
    if (ctx->np == 0) return LBM_E_STATE;
    const uint32_t Ln[3] = {ctx->g.nx, ctx->g.ny, ctx->g.nz};
    const uint32_t lmin = Ln[0] < Ln[1] ? (Ln[0] < Ln[2] ? Ln[0] : Ln[2]) : (Ln[1] < Ln[2] ? Ln[1] : Ln[2]);
    if (!(r_c > 0.0) || r_c > 0.5 * double(lmin)) return LBM_E_INVAL;
    if (ctx->np > kPairMax) return LBM_E_UNSUPPORTED;
    PairGrid pg;
    for (int k = 0; k < 3; ++k) {
        const double cells = floor(double(Ln[k]) / r_c);
        pg.nc[k] = cells < 1.0 ? 1u : uint32_t(cells);
        pg.L[k] = double(Ln[k]);
    }
    pg.T = pair_buckets(ctx->np);
    pg.n = uint32_t(ctx->np);
    pg.a = a_f;
    pg.rc = r_c;
    pg.ordered = pair_list_ordered(pg.n, uint64_t(pg.nc[0]) * pg.nc[1] * pg.nc[2]);
    ctx->pg = pg;
    ctx->pair_on = 1;
    return LBM_OK;
}

lbm_status lbm_pair_forces(lbm_ctx *ctx, double *fc) {
    if (!ctx || !fc) return LBM_E_INVAL;
    if (ctx->np == 0) return LBM_E_STATE;
    const size_t bytes = size_t(ctx->np) * 3 * 8;
    const hipError_t e = ctx->pair_on
                             ? hipMemcpyAsync(fc, ctx->fpair, bytes, hipMemcpyDeviceToDevice, ctx->stream)
                             : hipMemsetAsync(fc, 0, bytes, ctx->stream);
    return e == hipSuccess ? LBM_OK : LBM_E_DEVICE;
}

lbm_status lbm_set_particle_force(lbm_ctx *ctx, const double *f) {
    if (!ctx) return LBM_E_INVAL;
    if (f && ctx->np == 0) return LBM_E_STATE;
    ctx->fext = f;
    return LBM_OK;
}

double lbm_particle_radius(const lbm_ctx *ctx) { return (ctx && ctx->np > 0) ? ctx->R : -1.0; }

lbm_status lbm_particle_forces(lbm_ctx *ctx, double *fh, double *fr) {
    if (!ctx) return LBM_E_INVAL;
    if (ctx->np == 0) return LBM_E_STATE;
    const size_t bytes = size_t(ctx->np) * 3 * 8;
    hipError_t e = hipSuccess;
    if (fh) e = hipMemcpyAsync(fh, ctx->fh, bytes, hipMemcpyDeviceToDevice, ctx->stream);
    if (e == hipSuccess && fr)
        e = hipMemcpyAsync(fr, ctx->fr, bytes, hipMemcpyDeviceToDevice, ctx->stream);
    return e == hipSuccess ? LBM_OK : LBM_E_DEVICE;
}

lbm_status lbm_vacf_config(lbm_ctx *ctx, int32_t max_lag, int32_t stride, double *acc,
                           double *origins) {
    if (!ctx) return LBM_E_INVAL;
    if (max_lag == -1) {
        ctx->vacf_on = 0;
        return LBM_OK;
    }
    if (max_lag < 0 || stride < 1 || !acc || !origins) return LBM_E_INVAL;
    if (ctx->np == 0) return LBM_E_STATE;
    ctx->max_lag = max_lag;
    ctx->stride = stride;
    ctx->nslot = max_lag / stride + 1;
    ctx->acc = acc;
    ctx->origins = origins;
    ctx->vacf_t = 0;
    const hipError_t e = hipMemsetAsync(acc, 0, size_t(ctx->np) * size_t(max_lag + 1) * 8,
                                        ctx->stream);
    if (e != hipSuccess) return LBM_E_DEVICE;
    ctx->vacf_on = 1;
    return LBM_OK;
}

lbm_status lbm_vacf_counts(const lbm_ctx *ctx, int64_t *cnt) {
    if (!ctx || !cnt) return LBM_E_INVAL;
    if (!ctx->vacf_on) return LBM_E_STATE;
    // Samples t = 0 .. T-1; origins t0 = k * stride; lag l counts the origins
    // with t0 + l <= T - 1.
    const int64_t T = ctx->vacf_t;
    for (int32_t l = 0; l <= ctx->max_lag; ++l)
        cnt[l] = (T - 1 - l >= 0) ? (T - 1 - l) / ctx->stride + 1 : 0;
    return LBM_OK;
}

}  // extern "C"

namespace {

// Takes n steps, two at a time where the box has a two-step sweep, its
// particles are few enough (two_step_pays) and neither step is recorded.  An
// even number of two-step sweeps per call keeps the rule that n steps leave
// the state in the lattice n swaps away.
void advance(lbm_ctx *c, int32_t n) {
    // A captured call is replayed after any other of an even number of steps:
    // its first step always releases the third field (nodes that have been
    // released are cleared again).
    c->older_due = c->force[kThirdField] != nullptr;
    int32_t twos = 0;
    if (c->two > 0 && two_step_pays(c)) {
        int64_t count = c->series_count;
        auto sampled = [&](int32_t s) {
            return c->series_every > 0 && (c->series_t + s) % c->series_every == 0 && count < c->series_cap;
        };
        for (int32_t s = 0; s + 1 < n;) {
            const bool now = sampled(s), two = !now && !sampled(s + 1);
            count += now;
            twos += two;
            s += two ? 2 : 1;
        }
        twos &= ~1;
    }
    for (int32_t left = n; left > 0;) {
        if (twos > 0 && left >= 2 && !sample_at(c, 0) && !sample_at(c, 1)) {
            LBM_DISPATCH(c, launch_two_step);
            --twos;
            left -= 2;
        } else {
            LBM_DISPATCH(c, launch_step);
            --left;
        }
    }
    settle_fields(c);
}

}  // namespace

extern "C" {

lbm_status lbm_step(lbm_ctx *ctx, int32_t nsteps) {
    if (!ctx || nsteps < 0) return LBM_E_INVAL;
    advance(ctx, nsteps);
    return launch_status();
}

}  // extern "C"

namespace {

// The sums of lbm_observables with the reduction partials ([kRedBlocks][4])
// and the result (7 doubles) in the given device buffers.
lbm_status observables_into(lbm_ctx *ctx, double *partials, double *result, double out[7]) {
    LBM_DISPATCH(ctx, launch_partials, partials);
    hipLaunchKernelGGL(k_final_sums, dim3(1), dim3(kBlock), 0, ctx->stream, partials,
                       kRedBlocks, double(ctx->g.ncell), ctx->np > 0 ? ctx->v : nullptr, ctx->np,
                       ctx->np > 0 ? ctx->pdesc.mass : 0.0, result);
    if (launch_status() != LBM_OK) return LBM_E_DEVICE;
    double host[7];
    uint32_t err = 0;
    hipError_t e = hipMemcpyAsync(host, result, sizeof(host), hipMemcpyDeviceToHost,
                                  ctx->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(&err, ctx->err, sizeof(err), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->err, 0, sizeof(uint32_t), ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return LBM_E_DEVICE;
    bool finite = true;
    for (int k = 0; k < 7; ++k) {
        out[k] = host[k];
        finite = finite && isfinite(host[k]);
    }
    return (finite && err == 0) ? LBM_OK : LBM_E_NONFINITE;
}

}  // namespace

extern "C" {

lbm_status lbm_observables(lbm_ctx *ctx, double out[7]) {
    if (!ctx || !out) return LBM_E_INVAL;
    return observables_into(ctx, ctx->partials, ctx->result, out);
}

lbm_status lbm_observables_noalloc(lbm_ctx *ctx, double out[7]) {
    if (!ctx || !out) return LBM_E_INVAL;
    // the reduction runs over a fixed grid whatever the box or particle count,
    // so every context fits the array
    static_assert(kNoAllocDoubles >= size_t(kRedBlocks) * 4 + 7, "scratch too small");
    // the kernels run on the context's device, with that device's copy
    if (current_device() != ctx->device) return LBM_E_STATE;
    double *s = noalloc_scratch(ctx->device);
    if (!s) return LBM_E_DEVICE;
    return observables_into(ctx, s, s + size_t(kRedBlocks) * 4, out);
}

lbm_status lbm_profile_enable(lbm_ctx *ctx, int32_t enable) {
    if (!ctx || (enable != 0 && enable != 1)) return LBM_E_INVAL;
    ctx->prof_on = enable;
    return LBM_OK;
}

lbm_status lbm_profile_read(lbm_ctx *ctx, double out[4]) {
    if (!ctx || !out) return LBM_E_INVAL;
    if (hipStreamSynchronize(ctx->stream) != hipSuccess) return LBM_E_DEVICE;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int32_t k = 0; k < ctx->prof_used; ++k) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, ctx->prof_ev[2 * k], ctx->prof_ev[2 * k + 1]) != hipSuccess)
            return LBM_E_DEVICE;
        const int kind = ctx->prof_kind[k];
        acc[2 * kind] += ms;
        acc[2 * kind + 1] += 1.0;
    }
    ctx->prof_used = 0;
    for (int k = 0; k < 4; ++k) out[k] = acc[k];
    return LBM_OK;
}

lbm_status lbm_autotune(lbm_ctx *ctx, int32_t iters, double *ms, int32_t *chosen) {
    if (!ctx || iters < 1 || iters > 10000) return LBM_E_INVAL;
    uint32_t ys[kMaxRowsLog2 + 1];
    const int nl = layout_candidates(ctx, ys);
    size_t lat = 0;
    lbm_lattice_bytes(&ctx->desc, &lat);
    constexpr int kMaxTrials = kNumShapes * kNumOrders * kNumCaps;
    int ks[kMaxTrials], os[kMaxTrials], cs[kMaxTrials];
    double t[kMaxTrials];
    hipError_t err = hipSuccess;
    double best_k[kNumShapes];
    for (int k = 0; k < kNumShapes; ++k) best_k[k] = -1.0;
    // every launch timed: configuration, order, cap, layout index, ms
    struct Trial {
        int k, o, c, l;
        double t;
    };
    std::vector<Trial> trials;
    auto note = [&](int k, int o, int c, int l, double v) {
        if (v <= 0.0) return;
        if (best_k[k] <= 0.0 || v < best_k[k]) best_k[k] = v;
        if (config_tunable(k, lat)) trials.push_back(Trial{k, o, c, l, v});
    };
    auto time_one_layout = [&](int l, int n) -> bool {
        if (set_layout(ctx, ys[l]) != LBM_OK) return false;
        LBM_DISPATCH(ctx, time_launches, iters, n, ks, os, cs, t, &err);
        return err == hipSuccess && launch_status() == LBM_OK;
    };
    // Stage 1: every configuration in linear order without a residency cap,
    // in every layout; keep the layout of the fastest launch.
    double t1[kMaxRowsLog2 + 1][kNumShapes];
    int bl = -1, first = -1;
    for (int l = 0; l < nl; ++l) {
        for (int k = 0; k < kNumShapes; ++k) ks[k] = k, os[k] = int(kOrderLinear), cs[k] = 0;
        if (!time_one_layout(l, kNumShapes)) return LBM_E_DEVICE;
        for (int k = 0; k < kNumShapes; ++k) {
            t1[l][k] = config_tunable(k, lat) ? t[k] : -1.0;
            note(k, int(kOrderLinear), 0, l, t[k]);
            if (t1[l][k] > 0.0 && (bl < 0 || t[k] < t1[bl][first])) bl = l, first = k;
        }
    }
    if (bl < 0) return LBM_E_DEVICE;
    // Stage 2: in that layout, its two fastest configurations with every block
    // order and cap.
    int second = -1;
    for (int k = 0; k < kNumShapes; ++k)
        if (k != first && t1[bl][k] > 0.0 && (second < 0 || t1[bl][k] < t1[bl][second])) second = k;
    int n = 0;
    for (int k : {first, second}) {
        if (k < 0) continue;
        for (int o = 0; o < int(kNumOrders); ++o)
            for (int cap = 0; cap < kNumCaps; ++cap) {
                if (o == int(kOrderLinear) && cap == 0) continue;  // timed in stage 1
                ks[n] = k, os[n] = o, cs[n] = cap;
                ++n;
            }
    }
    if (!time_one_layout(bl, n)) return LBM_E_DEVICE;
    Trial best{first, int(kOrderLinear), 0, bl, t1[bl][first]};
    for (int j = 0; j < n; ++j) {
        note(ks[j], os[j], cs[j], bl, t[j]);
        if (t[j] > 0.0 && t[j] < best.t) best = Trial{ks[j], os[j], cs[j], bl, t[j]};
    }
    // Stage 3: that launch in every other layout (a cap or order can change
    // which layout streams best).
    if (best.o != int(kOrderLinear) || best.c != 0) {
        const Trial b0 = best;
        for (int l = 0; l < nl; ++l) {
            if (l == b0.l) continue;
            ks[0] = b0.k, os[0] = b0.o, cs[0] = b0.c;
            if (!time_one_layout(l, 1)) return LBM_E_DEVICE;
            note(b0.k, b0.o, b0.c, l, t[0]);
        }
    }
    // Stage 4: single timings differ by a percent or two from run to run, so
    // the three fastest launches are timed again, in turn, twice each with
    // twice the iterations, and the lowest total wins.
    std::sort(trials.begin(), trials.end(), [](const Trial &x, const Trial &y) { return x.t < y.t; });
    const int m = int(std::min<size_t>(3, trials.size()));
    double total[3] = {0.0, 0.0, 0.0};
    for (int round = 0; round < 2; ++round)
        for (int j = 0; j < m; ++j) {
            ks[0] = trials[j].k, os[0] = trials[j].o, cs[0] = trials[j].c;
            if (set_layout(ctx, ys[trials[j].l]) != LBM_OK) return LBM_E_DEVICE;
            LBM_DISPATCH(ctx, time_launches, 2 * iters, 1, ks, os, cs, t, &err);
            if (err != hipSuccess || launch_status() != LBM_OK) return LBM_E_DEVICE;
            total[j] += t[0] > 0.0 ? t[0] : 1e30;
        }
    int jb = 0;
    for (int j = 1; j < m; ++j)
        if (total[j] < total[jb]) jb = j;
    best = trials[jb];
    if (set_layout(ctx, ys[best.l]) != LBM_OK) return LBM_E_DEVICE;
    ctx->shape = best.k;
    ctx->order = best.o;
    ctx->cap = best.c;
    // Two-step sweep: the fastest of its tiles, if two steps in it are faster
    // than two launches of the choice above.
    {
        TwoStepTiles tl[kTwoStepCandidates];
        const int nt = two_step_trial(&ctx->desc) ? two_step_candidates(&ctx->desc, tl) : 0;
        double two_best = 0.0;
        ctx->two = 0;
        for (int j = 0; j <= nt; ++j) {
            double v = 0.0;
            if (nt > 0) LBM_DISPATCH(ctx, time_two_steps, j > 0 ? &tl[j - 1] : nullptr, iters, &v, &err);
            if (err != hipSuccess || launch_status() != LBM_OK) return LBM_E_DEVICE;
            if (j == 0 || (v > 0.0 && v < two_best)) {
                two_best = v;
                ctx->two = j;
                if (j > 0) ctx->two_tiles = tl[j - 1];
            }
        }
    }
    tune_store(ctx_tune_key(ctx),
               tune_code(best.k, best.o, best.c, rows_log2(ctx->g)) + kTuneTwo * (ctx->two + 1));
    if (ms)
        for (int k = 0; k < kNumShapes; ++k) ms[k] = best_k[k];
    if (chosen) *chosen = best.k;
    return LBM_OK;
}

lbm_status lbm_set_layout(lbm_ctx *ctx, int32_t rows_per_group) {
    if (!ctx || rows_per_group < 1 || rows_per_group > (1 << kMaxRowsLog2) ||
        (rows_per_group & (rows_per_group - 1)) != 0 || ctx->desc.ny % rows_per_group != 0)
        return LBM_E_INVAL;
    return set_layout(ctx, uint32_t(rows_per_group));
}

lbm_status lbm_get_layout(const lbm_ctx *ctx, int32_t *rows_per_group) {
    if (!ctx || !rows_per_group) return LBM_E_INVAL;
    *rows_per_group = int32_t(ctx->g.ymask + 1);
    return LBM_OK;
}

lbm_status lbm_set_sweep_launch(lbm_ctx *ctx, int32_t order, int32_t waves_per_simd) {
    if (!ctx || order < 0 || order >= int32_t(kNumOrders)) return LBM_E_INVAL;
    int cap = -1;
    for (int j = 0; j < kNumCaps; ++j)
        if (kResidencyCaps[j] == waves_per_simd) cap = j;
    if (cap < 0 || sweep_lds(ctx, cap, config_block(ctx->shape)) < 0) return LBM_E_INVAL;
    ctx->order = order;
    ctx->cap = cap;
    return LBM_OK;
}

lbm_status lbm_get_sweep_launch(const lbm_ctx *ctx, int32_t *order, int32_t *waves_per_simd) {
    if (!ctx || !order || !waves_per_simd) return LBM_E_INVAL;
    *order = ctx->order;
    *waves_per_simd = kResidencyCaps[ctx->cap];
    return LBM_OK;
}

lbm_status lbm_stream_ceiling(lbm_ctx *ctx, int32_t k, int32_t iters, double *ms) {
    if (!ctx || !ms || iters < 1 || iters > 10000) return LBM_E_INVAL;
    if (k < 0) k = ctx->shape;
    if (k >= kNumShapes || !shape_ok(ctx, k)) return LBM_E_INVAL;
    hipError_t err = hipSuccess;
    double t = 0.0;
    LBM_DISPATCH(ctx, time_stream_only, k, iters, &t, &err);
    if (err != hipSuccess || launch_status() != LBM_OK) return LBM_E_DEVICE;
    *ms = t;
    return LBM_OK;
}

lbm_status lbm_set_shape(lbm_ctx *ctx, int32_t k) {
    if (!ctx || k < 0 || k >= kNumShapes || !shape_ok(ctx, k)) return LBM_E_INVAL;
    ctx->shape = k;
    if (sweep_lds(ctx, ctx->cap, config_block(k)) < 0) ctx->cap = 0;  // cap not possible here
    return LBM_OK;
}

lbm_status lbm_warnings(const lbm_ctx *ctx, uint32_t *flags) {
    if (!ctx || !flags) return LBM_E_INVAL;
    *flags = ctx->warnings;
    return LBM_OK;
}

lbm_status lbm_get_shape(const lbm_ctx *ctx, int32_t *k) {
    if (!ctx || !k) return LBM_E_INVAL;
    *k = ctx->shape;
    return LBM_OK;
}

lbm_status lbm_series_config(lbm_ctx *ctx, int32_t every, double *series, int64_t capacity) {
    if (!ctx || every < 0) return LBM_E_INVAL;
    if (every > 0 && (!series || capacity < 1)) return LBM_E_INVAL;
    ctx->series_every = every;
    ctx->series = every > 0 ? series : nullptr;
    ctx->series_cap = every > 0 ? capacity : 0;
    ctx->series_count = 0;
    ctx->series_t = 0;
    return LBM_OK;
}

lbm_status lbm_series_count(const lbm_ctx *ctx, int64_t *count) {
    if (!ctx || !count) return LBM_E_INVAL;
    *count = ctx->series_count;
    return LBM_OK;
}

lbm_status lbm_get_step(const lbm_ctx *ctx, int64_t *step) {
    if (!ctx || !step) return LBM_E_INVAL;
    *step = ctx->step;
    return LBM_OK;
}

lbm_status lbm_destroy(lbm_ctx *ctx) {
    if (!ctx) return LBM_E_INVAL;
    for (int32_t k = 0; k < 2 * ctx->prof_cap; ++k) (void)hipEventDestroy(ctx->prof_ev[k]);
    free(ctx->prof_ev);
    free(ctx->prof_kind);
    free(ctx);
    return LBM_OK;
}

const char *lbm_status_string(lbm_status status) {
    switch (status) {
        case LBM_OK: return "ok";
        case LBM_E_INVAL: return "invalid argument";
        case LBM_E_DEVICE: return "device error";
        case LBM_E_STATE: return "invalid state";
        case LBM_E_NONFINITE: return "non-finite value or node force out of range";
        case LBM_E_UNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

}  // extern "C"

// ===========================================================================
// Host side: ensembles of independent boxes.
// ===========================================================================
struct lbm_ens {
    lbm_ensemble_desc desc;
    int32_t nrep;
    lbm_replica_desc *host_reps;  // copy of the caller's descriptors
    Replica *host_table;          // device-side table, host copy
    size_t elem;
    void *pop[2];
    int cur;
    hipStream_t stream;
    double enc_s, dec_s;
    uint64_t total_cells, total_pop;
    uint32_t total_blocks[kNumGeomShapes];
    int32_t n;  // particles in all replicas
    // scratch
    Replica *reps;
    uint16_t *blk_rep[kNumGeomShapes];
    uint16_t *part_rep;
    uint32_t *mask[kForceFields];
    long long *force[kForceFields];
    uint64_t total_mask_words;
    uint32_t *cells[2];  // [n][8] nodes spread to in even and odd steps
    double *fh, *fr;
    EnsClock *clock;
    uint32_t *err;
    double *partials, *result;
    double *r, *v;
    // velocity autocorrelation
    int vacf_on;
    int32_t max_lag, stride, nslot;
    double *acc, *origins;
    int64_t vacf_t;
    int64_t step;
    int shape;
    int order, cap;         // block order and residency cap of the stream-collide
    int lds_cu, lds_block;  // LDS bytes per compute unit and per block (device limits)
    int two, two_nts;       // two-step sweeps, and their store policy
    int two_possible;
    uint32_t two_blocks, two_threads;
    uint16_t *two_rep;      // block -> box of the two-step sweep
    int rows;    // requested rows per group: each box takes the largest power of two <= rows dividing its ny
    int device;  // device current at lbm_ens_init (autotune cache key)
    // graph of LBM_ENS_GRAPH_STEPS steps, captured on a private stream and
    // replayed on `stream`
    int use_graph;
    hipGraphExec_t graph;
    int graph_valid;
    hipStream_t cap_stream;
    int graph_replays;  // number of graph launches so far
};

namespace {

TuneKey ens_tune_key(const lbm_ens *e) {
    TuneKey k{1, e->device, e->desc.storage, int(D3Q19::Q), {}};
    k.dims.reserve(3 * size_t(e->nrep));
    for (int32_t q = 0; q < e->nrep; ++q) {
        k.dims.push_back(e->host_reps[q].nx);
        k.dims.push_back(e->host_reps[q].ny);
        k.dims.push_back(e->host_reps[q].nz);
    }
    return k;
}

uint32_t ens_chunk(int32_t nx) { return uint32_t(nx); }  // unpadded, as row_chunk

// Two-step tiles of one box of an ensemble of total_cells nodes: the boxes'
// blocks share the units, so the tile is the one of least total cost, and slabs
// are of 24 planes (two planes and a start more per slab, against some thousand
// blocks to even the units out), or as many as give each unit a block where
// that is fewer, but 4 at least (13 BF16 boxes of 32 to 48 nodes, five steps:
// 194 us in slabs of 24 planes, 128 in single steps).
TwoStepTiles ens_two_tiles(const lbm_replica_desc &r, size_t elem, uint64_t total_cells) {
    const uint32_t nx = uint32_t(r.nx), ny = uint32_t(r.ny), nz = uint32_t(r.nz);
    TwoStepTiles best{};
    double cost = -1.0;
    // 32-bit byte offsets within a plane
    if (uint64_t(nx) * ny * D3Q19::Q * elem >= (uint64_t(1) << 32)) return best;
    two_step_each_tile(nx, ny, elem, [&](uint32_t tx, uint32_t ty, uint32_t ntx, uint32_t nty) {
        const double c = two_step_plane_cost(tx, ty, elem) * ntx * nty;
        if (cost > 0.0 && c >= cost) return;
        const uint64_t share = total_cells / (uint64_t(kTwoStepUnits) * tx * ty);  // planes per unit
        const uint32_t most = uint32_t(std::min<uint64_t>(24, std::max<uint64_t>(4, share)));
        const uint32_t ns = (nz + most - 1) / most, lz = (nz + ns - 1) / ns;
        best = TwoStepTiles{tx, ty, lz, ntx, nty, (nz + lz - 1) / lz};
        cost = c;
    });
    return best;
}

// Ensembles of fewer nodes than 2^21 (16-bit 2^22) take single steps: their
// blocks' slabs are a few planes (16 steps, us, two-step / single: 13 boxes of 32
// to 48 nodes FP32 601 / 596, FP64 1221 / 1144, BF16 565 / 413; 40 such boxes
// FP32 1236 / 1469, 64 BF16 1516 / 1525; 40 of 48 to 96 BF16 3520 / 4048).
bool ens_two_step_pays(size_t elem, uint64_t nodes, int64_t particles) {
    return nodes >= uint64_t(1) << (elem == 2 ? 22 : 21) && two_step_pays(elem, D3Q19::Q, nodes, particles);
}

struct EnsLayout {
    uint64_t total_cells = 0, total_pop = 0, total_mask_words = 0;
    uint32_t total_blocks[kNumGeomShapes] = {0, 0, 0, 0};
    uint32_t two_blocks = 0, two_threads = 0;  // two-step sweep
    bool two_ok = true;                        // every box has tiles for it, and it pays
    std::vector<TwoStepTiles> two;             // per box
    int fields = 0;                            // node-force fields
    // Rows of whole 32-byte sectors in boxes of half the nodes and more: the sweep
    // stores non-temporally (ms per 16 steps, plain / non-temporal: 64 FP32 boxes
    // of 48 to 96 8.79 / 8.41, 100 of 48 3.62 / 3.54, BF16 2.93 / 2.85; but 40 FP32
    // boxes of 66 3.87 / 4.49, 80 of 50 3.34 / 3.47, 64 of 33, 50, 64 and 70 4.03 / 4.16;
    // 80 FP64 boxes of 50 6.34 / 6.58).  A tile of a small box is whole rows, so
    // that rows need not be whole lines.
    bool two_stream = false;
    int32_t n = 0;
    size_t lattice_bytes = 0, scratch_bytes = 0;
    // scratch offsets
    size_t o_reps, o_blk[kNumGeomShapes], o_two, o_part, o_mask[kForceFields], o_force[kForceFields],
        o_cells[2], o_fh, o_fr, o_clock, o_err, o_partials, o_result;
};

bool ens_desc_ok(const lbm_ensemble_desc *d, const lbm_replica_desc *reps) {
    if (!d || !reps || d->nrep < 1 || d->nrep > 65535 || d->reserved != 0) return false;
    if (elem_size(d->storage) == 0) return false;
    if (d->storage == LBM_STORE_F16 && (d->f16_scale_log2 < 0 || d->f16_scale_log2 > 24)) return false;
    if (!(d->mass > 0.0) || !isfinite(d->mass) || !(d->gamma >= 0.0) || !isfinite(d->gamma)) return false;
    if (!(d->kT >= 0.0) || !isfinite(d->kT) || !isfinite(d->radius)) return false;
    if (d->friction < LBM_FRICTION_STOKESLET || d->friction > LBM_FRICTION_STOKESLET_CUBE) return false;
    uint64_t cells = 0, n = 0;
    for (int32_t k = 0; k < d->nrep; ++k) {
        const lbm_replica_desc &r = reps[k];
        if (r.nx < 2 || r.ny < 2 || r.nz < 2 || r.n < 1 || !(r.tau > 0.5) || !isfinite(r.tau))
            return false;
        if (r.reserved != 0) return false;
        // a box's sweep indexes within the box in 32 bits
        if (uint64_t(r.nx) * uint64_t(r.ny) * uint64_t(r.nz) * 19 >= (uint64_t(1) << 32)) return false;
        cells += uint64_t(r.nx) * uint64_t(r.ny) * uint64_t(r.nz);
        n += uint64_t(r.n);
    }
    return cells < (uint64_t(1) << 31) && n < (uint64_t(1) << 24);
}

EnsLayout ens_layout(const lbm_ensemble_desc *d, const lbm_replica_desc *reps) {
    EnsLayout L;
    const size_t elem = elem_size(d->storage);
    for (int32_t k = 0; k < d->nrep; ++k) {
        const lbm_replica_desc &r = reps[k];
        const uint64_t cells = uint64_t(r.nx) * r.ny * r.nz;
        L.total_cells += cells;
        L.total_pop += uint64_t(ens_chunk(r.nx)) * D3Q19::Q * r.ny * r.nz;
        L.total_mask_words += mask_words(cells);
        for (int s = 0; s < kNumGeomShapes; ++s) {
            const uint64_t band = (r.ny % kShapes[s].cpt == 0) ? cells / kShapes[s].cpt : 0;
            L.total_blocks[s] += uint32_t((band + kShapes[s].bs - 1) / kShapes[s].bs);
        }
        L.n += r.n;
    }
    uint64_t sector_cells = 0;
    std::map<std::tuple<int32_t, int32_t, int32_t>, TwoStepTiles> tiles;
    L.two.reserve(size_t(d->nrep));
    for (int32_t k = 0; k < d->nrep; ++k) {
        const lbm_replica_desc &r = reps[k];
        const auto at = tiles.try_emplace(std::make_tuple(r.nx, r.ny, r.nz));
        if (at.second) at.first->second = ens_two_tiles(r, elem, L.total_cells);
        const TwoStepTiles &tl = at.first->second;
        L.two.push_back(tl);
        L.two_ok = L.two_ok && tl.lz > 0;
        L.two_blocks += tl.ntx * tl.nty * tl.nslab;
        if (size_t(r.nx) * elem % 32 == 0) sector_cells += uint64_t(r.nx) * uint64_t(r.ny) * uint64_t(r.nz);
        L.two_threads = std::max(L.two_threads, two_step_threads(tl));
    }
    L.two_stream = 2 * sector_cells >= L.total_cells;
    L.two_ok = L.two_ok && ens_two_step_pays(elem, L.total_cells, L.n);
    L.lattice_bytes = align_up(L.total_pop * elem, kAlign);
    size_t o = 0;
    L.o_reps = o;
    o += align_up(sizeof(Replica) * size_t(d->nrep), kAlign);
    for (int s = 0; s < kNumGeomShapes; ++s) {
        L.o_blk[s] = o;
        o += align_up(size_t(L.total_blocks[s]) * 2 + 2, kAlign);
    }
    L.o_two = o;
    o += align_up(size_t(L.two_blocks) * 2, kAlign);
    L.o_part = o;
    o += align_up(size_t(L.n) * 2, kAlign);
    L.fields = L.two_ok ? kForceFields : kThirdField;
    for (int k = 0; k < L.fields; ++k) {
        L.o_mask[k] = o;
        o += align_up(L.total_mask_words * 4, kAlign);
    }
    for (int k = 0; k < L.fields; ++k) {
        L.o_force[k] = o;
        o += align_up(L.total_cells * 3 * 8, kAlign);
    }
    for (int k = 0; k < 2; ++k) {
        L.o_cells[k] = o;
        o += align_up(size_t(L.n) * 8 * 4, kAlign);
    }
    L.o_fh = o;
    o += align_up(size_t(L.n) * 3 * 8, kAlign);
    L.o_fr = o;
    o += align_up(size_t(L.n) * 3 * 8, kAlign);
    L.o_clock = o;
    o += kAlign;
    L.o_err = o;
    o += kAlign;
    L.o_partials = o;
    o += align_up(size_t(kRedBlocks) * 4 * 8, kAlign);
    L.o_result = o;
    o += kAlign;
    L.scratch_bytes = o;
    return L;
}

ParticleArgs ens_particle_args(lbm_ens *e) {
    ParticleArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.r = pa.r_out = e->r;
    pa.v = pa.v_out = e->v;
    pa.fh = e->fh;
    pa.fr = e->fr;
    pa.err = e->err;
    pa.n = e->n;
    pa.friction = e->desc.friction;
    pa.mass = e->desc.mass;
    pa.gamma = e->desc.gamma;
    pa.sig = e->desc.kT > 0.0 ? sqrt(2.0 * e->desc.gamma * e->desc.kT) : 0.0;
    pa.acc = nullptr;
    pa.origins = nullptr;
    pa.k_hi = -1;
    pa.nslot = pa.stride = 1;
    pa.pmom = nullptr;
    if (e->vacf_on) {
        pa.acc = e->acc;
        pa.origins = e->origins;
        pa.nslot = e->nslot;
        pa.stride = e->stride;
        pa.max_lag = e->max_lag;
    }
    return pa;
}

// Dynamic LDS that caps the ensemble sweep at kResidencyCaps[cap] waves per
// SIMD for blocks of bs lanes (0: no cap; -1: not possible on this device).
long ens_sweep_lds(const lbm_ens *e, int cap, int bs) { return residency_lds(e->lds_cu, e->lds_block, cap, bs); }

ForceField ens_field(const lbm_ens *e, int64_t k) { return ForceField{e->force[k], e->mask[k]}; }

template <class C, int CPT, int BS, bool NTS>
void ens_collide_shape(lbm_ens *e, const typename C::T *A, typename C::T *B, const ForceField &ff) {
    using R = typename C::R;
    const int sh = e->shape & 3;
    const long lds = ens_sweep_lds(e, e->cap, BS);
    hipLaunchKernelGGL((k_ens_collide<C, CPT, BS, NTS>), dim3(e->total_blocks[sh]), dim3(BS),
                       lds > 0 ? size_t(lds) : 0, e->stream, A, B, e->reps, e->blk_rep[sh], sh,
                       ff.f, ff.mask, R(e->enc_s), R(e->dec_s), e->clock, e->vacf_on,
                       uint32_t(e->order));
}

// The particle update of step n (`ahead` steps after the device clock), and the
// nodes it has to release: those of the last two steps (where the step two back
// was released already its nodes are cleared again in the third field, which is
// idle).  held: the step's own field is one of them, it spreads into the third.
template <class C>
void ens_launch_particle(lbm_ens *e, const typename C::T *A, int64_t n, int ahead, bool held) {
    const int own = int(n & 1);
    ParticleArgs pa = ens_particle_args(e);
    pa.cells = e->cells[own];
    if (!ahead) {
        pa.last_cells = e->cells[own ^ 1];
        pa.older_cells = e->two_possible ? pa.cells : nullptr;
    }
    hipLaunchKernelGGL(k_ens_particle<C>, dim3(unsigned(particle_blocks(e->n))), dim3(particle_threads(pa)), 0, e->stream, A,
                       e->reps, e->part_rep, typename C::R(e->dec_s), pa, e->clock, ahead,
                       ens_field(e, held ? kThirdField : own), ens_field(e, own ^ 1), ens_field(e, held ? own : kThirdField));
}

// Step n of every replica, from lattice cur.
template <class C>
void ens_launch_step(lbm_ens *e, int cur, int64_t n) {
    using T = typename C::T;
    const T *A = static_cast<const T *>(e->pop[cur]);
    T *B = static_cast<T *>(e->pop[cur ^ 1]);
    ens_launch_particle<C>(e, A, n, 0, false);
#define LBM_ENS_CALL(CPT, BS, NTS, ROW) ens_collide_shape<C, CPT, BS, NTS>(e, A, B, ens_field(e, n & 1))
    LBM_CONFIG_SWITCH(e->shape, LBM_ENS_CALL)
#undef LBM_ENS_CALL
}

EnsTwoStepArgs ens_two_step_args(lbm_ens *e, int cur, const ForceField &f0, const ForceField &f1) {
    EnsTwoStepArgs a;
    a.A = e->pop[cur];
    a.B = e->pop[cur ^ 1];
    a.reps = e->reps;
    a.blk_rep = e->two_rep;
    a.part_rep = e->part_rep;
    a.blocks = e->two_blocks;
    a.threads = e->two_threads;
    a.enc_s = e->enc_s;
    a.dec_s = e->dec_s;
    a.f0 = f0;
    a.f1 = f1;
    a.clock = e->clock;
    a.vacf_on = e->vacf_on;
    a.nts = e->two_nts != 0;
    a.stream = e->stream;
    return a;
}

// Steps n and n + 1 of every replica in one sweep (see launch_two_step).
// held: steps n - 2 and n - 1 were the first such sweep of a pair.
template <class C>
void ens_launch_two_step(lbm_ens *e, int cur, int64_t n, bool held) {
    const EnsTwoStepArgs a =
        ens_two_step_args(e, cur, ens_field(e, held ? kThirdField : n & 1), ens_field(e, (n + 1) & 1));
    const typename C::T *A = static_cast<const typename C::T *>(a.A);
    ens_launch_particle<C>(e, A, n, 0, held);
    if (e->desc.friction == LBM_FRICTION_BD) {
        ens_launch_particle<C>(e, A, n + 1, 1, false);  // reads no fluid
    } else {
        ParticleArgs pa = ens_particle_args(e);
        pa.cells = e->cells[(n + 1) & 1];
        launch_ens_particle_ahead<C>(a, pa);
    }
    launch_ens_two_steps<C>(a);
}

template <class C>
void ens_launch_any(lbm_ens *e, int cur, int64_t n, int sweep) {
    if (sweep)
        ens_launch_two_step<C>(e, cur, n, sweep == 2);
    else
        ens_launch_step<C>(e, cur, n);
}

// Step n (sweep 0), or steps n and n + 1 in the first or the second of a pair of
// two-step sweeps (1, 2), from lattice cur.
void ens_dispatch_step(lbm_ens *e, int cur, int64_t n, int sweep) {
    switch (e->desc.storage) {
        case LBM_STORE_F64: ens_launch_any<F64Q19>(e, cur, n, sweep); break;
        case LBM_STORE_F32: ens_launch_any<F32Q19>(e, cur, n, sweep); break;
        case LBM_STORE_BF16: ens_launch_any<BF16Q19>(e, cur, n, sweep); break;
        case LBM_STORE_F16: ens_launch_any<F16Q19>(e, cur, n, sweep); break;
    }
}

// Rows per group of a box with ny rows per plane when `rows` is requested: the
// largest power of two not above it that divides ny.
uint32_t ens_box_rows(int rows, int32_t ny) {
    uint32_t y = uint32_t(rows);
    while (y > 1 && ny % int32_t(y) != 0) y >>= 1;
    return y;
}

// Moves every box into the layout ens_box_rows(rows, ny): each box is permuted
// into the spare lattice, and the whole spare lattice is copied back, so the
// state stays in the current buffer; then the device table is updated.
template <class C>
void ens_relayout(lbm_ens *e, int rows, hipError_t *err) {
    using T = typename C::T;
    const T *A = static_cast<const T *>(e->pop[e->cur]);
    T *B = static_cast<T *>(e->pop[e->cur ^ 1]);
    for (int32_t k = 0; k < e->nrep; ++k) {
        Replica &t = e->host_table[k];
        const Grid gn = with_rows_per_group(t.g, ens_box_rows(rows, int32_t(t.g.ny)));
        hipLaunchKernelGGL(k_relayout<C>, dim3(blocks_for(t.g.ncell)), dim3(kBlock), 0, e->stream,
                           A + t.pop_off, t.g, B + t.pop_off, gn);
        t.g = gn;
    }
    *err = hipGetLastError();
    if (*err == hipSuccess)
        *err = hipMemcpyAsync(e->pop[e->cur], e->pop[e->cur ^ 1], e->total_pop * sizeof(T),
                              hipMemcpyDeviceToDevice, e->stream);
    if (*err == hipSuccess)
        *err = hipMemcpyAsync(e->reps, e->host_table, sizeof(Replica) * e->nrep,
                              hipMemcpyHostToDevice, e->stream);
    if (*err == hipSuccess) *err = hipStreamSynchronize(e->stream);  // host_table is reused
    e->rows = rows;
}

void ens_drop_graph(lbm_ens *e);

lbm_status ens_set_layout(lbm_ens *e, int rows) {
    if (rows == e->rows) return LBM_OK;
    ens_drop_graph(e);
    hipError_t err = hipSuccess;
    switch (e->desc.storage) {
        case LBM_STORE_F64: ens_relayout<F64Q19>(e, rows, &err); break;
        case LBM_STORE_F32: ens_relayout<F32Q19>(e, rows, &err); break;
        case LBM_STORE_BF16: ens_relayout<BF16Q19>(e, rows, &err); break;
        case LBM_STORE_F16: ens_relayout<F16Q19>(e, rows, &err); break;
    }
    return err == hipSuccess ? LBM_OK : LBM_E_DEVICE;
}

void ens_drop_graph(lbm_ens *e) {
    if (e->graph_valid) (void)hipGraphExecDestroy(e->graph);
    e->graph_valid = 0;
}

// Two steps per graph cost about 1.5% over plain launches on the 64-box
// workload; sixteen amortise the graph launch.
static_assert(LBM_ENS_GRAPH_STEPS % 4 == 0, "pairs of two-step sweeps, so that lattices and fields return to their start");

// Capture LBM_ENS_GRAPH_STEPS steps from an even step number, starting from
// lattice e->cur, into a graph.
// Capture runs on a private non-blocking stream (the caller's stream may be
// the null stream, which cannot be captured); the graph is then launched on
// the caller's stream.  Returns false when no graph could be made.
bool ens_capture(lbm_ens *e) {
    ens_drop_graph(e);
    if (!e->cap_stream && hipStreamCreateWithFlags(&e->cap_stream, hipStreamNonBlocking) != hipSuccess) {
        e->cap_stream = nullptr;
        return false;
    }
    hipStream_t user = e->stream;
    if (hipStreamBeginCapture(e->cap_stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
        return false;
    e->stream = e->cap_stream;
    int cur = e->cur;
    for (int k = 0; k < LBM_ENS_GRAPH_STEPS; k += e->two ? 2 : 1) {
        ens_dispatch_step(e, cur, k, e->two ? 1 + (k / 2) % 2 : 0);
        cur ^= 1;
    }
    e->stream = user;
    hipGraph_t g = nullptr;
    const hipError_t end = hipStreamEndCapture(e->cap_stream, &g);
    if (end != hipSuccess || !g) {
        (void)hipGetLastError();
        return false;
    }
    const hipError_t err = hipGraphInstantiate(&e->graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (err != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    e->graph_valid = 1;
    return true;
}

template <class C, int CPT, int BS, bool NTS>
void ens_time_shape(lbm_ens *e, int k, int o, int c) {
    // A -> B without swapping (the state in A is untouched); the caller
    // restores the device clock the launches advance.
    const int saved[3] = {e->shape, e->order, e->cap};
    e->shape = k;
    e->order = o;
    e->cap = c;
    ens_collide_shape<C, CPT, BS, NTS>(e, static_cast<const typename C::T *>(e->pop[e->cur]),
                                       static_cast<typename C::T *>(e->pop[e->cur ^ 1]),
                                       ens_field(e, (e->step + 1) & 1));  // last step's node forces
    e->shape = saved[0];
    e->order = saved[1];
    e->cap = saved[2];
}

template <class C>
void ens_time_dispatch(lbm_ens *e, int k, int o, int c) {
#define LBM_ENS_TIME(CPT, BS, NTS, ROW) ens_time_shape<C, CPT, BS, NTS>(e, k, o, c)
    LBM_CONFIG_SWITCH(k, LBM_ENS_TIME)
#undef LBM_ENS_TIME
}

template <class C>
void ens_stream_only(lbm_ens *e, int k) {
    using T = typename C::T;
    const int sh = k & 3;
    const T *A = static_cast<const T *>(e->pop[e->cur]);
    T *B = static_cast<T *>(e->pop[e->cur ^ 1]);
#define LBM_ENS_STREAM_ONLY(CPT, BS, NTS, ROW)                                                   \
    do {                                                                                          \
        const long lds = ens_sweep_lds(e, e->cap, BS);                                            \
        hipLaunchKernelGGL((k_ens_stream_only<C, CPT, BS, NTS>), dim3(e->total_blocks[sh]),       \
                           dim3(BS), lds > 0 ? size_t(lds) : 0, e->stream, A, B, e->reps,         \
                           e->blk_rep[sh], sh, uint32_t(e->order));                               \
    } while (0)
    LBM_CONFIG_SWITCH(k, LBM_ENS_STREAM_ONLY)
#undef LBM_ENS_STREAM_ONLY
}

void ens_stream_only_any(lbm_ens *e, int k) {
    switch (e->desc.storage) {
        case LBM_STORE_F64: ens_stream_only<F64Q19>(e, k); break;
        case LBM_STORE_F32: ens_stream_only<F32Q19>(e, k); break;
        case LBM_STORE_BF16: ens_stream_only<BF16Q19>(e, k); break;
        case LBM_STORE_F16: ens_stream_only<F16Q19>(e, k); break;
    }
}

void ens_time_any(lbm_ens *e, int k, int o, int c) {
    switch (e->desc.storage) {
        case LBM_STORE_F64: ens_time_dispatch<F64Q19>(e, k, o, c); break;
        case LBM_STORE_F32: ens_time_dispatch<F32Q19>(e, k, o, c); break;
        case LBM_STORE_BF16: ens_time_dispatch<BF16Q19>(e, k, o, c); break;
        case LBM_STORE_F16: ens_time_dispatch<F16Q19>(e, k, o, c); break;
    }
}

// Configuration k applies to every box (two-node shapes need an even ny) and
// cap c can be imposed on its blocks.
bool ens_launch_ok(const lbm_ens *e, int k, int c) {
    if (k < 0 || k >= kNumShapes || config_row(k) || e->total_blocks[k & 3] == 0) return false;
    for (int32_t q = 0; q < e->nrep; ++q)
        if (e->host_reps[q].ny % kShapes[k & 3].cpt != 0) return false;
    return ens_sweep_lds(e, c, config_block(k)) >= 0;
}

void ens_two_steps_any(lbm_ens *e, const EnsTwoStepArgs &a) {
    switch (e->desc.storage) {
        case LBM_STORE_F64: launch_ens_two_steps<F64Q19>(a); break;
        case LBM_STORE_F32: launch_ens_two_steps<F32Q19>(a); break;
        case LBM_STORE_BF16: launch_ens_two_steps<BF16Q19>(a); break;
        case LBM_STORE_F16: launch_ens_two_steps<F16Q19>(a); break;
    }
}

// Mean ms per launch of configuration k with block order o and cap c over
// iters launches (after two unrecorded ones); < 0 on a device error.
double ens_time_launch(lbm_ens *e, int k, int o, int c, int32_t iters, hipEvent_t e0, hipEvent_t e1) {
    for (int w = 0; w < 2; ++w) ens_time_any(e, k, o, c);
    (void)hipEventRecord(e0, e->stream);
    for (int32_t it = 0; it < iters; ++it) ens_time_any(e, k, o, c);
    (void)hipEventRecord(e1, e->stream);
    float f = 0.0f;
    if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&f, e0, e1) != hipSuccess ||
        launch_status() != LBM_OK)
        return -1.0;
    return double(f) / iters;
}

}  // namespace

extern "C" {

lbm_status lbm_ens_bytes(const lbm_ensemble_desc *desc, const lbm_replica_desc *reps,
                         size_t *lattice_bytes, size_t *scratch_bytes) {
    if (!ens_desc_ok(desc, reps) || !lattice_bytes || !scratch_bytes) return LBM_E_INVAL;
    const EnsLayout L = ens_layout(desc, reps);
    *lattice_bytes = L.lattice_bytes;
    *scratch_bytes = L.scratch_bytes;
    return LBM_OK;
}

lbm_status lbm_ens_init(const lbm_ensemble_desc *desc, const lbm_replica_desc *reps, void *pop_a,
                        void *pop_b, void *scratch, double *r, double *v, void *stream,
                        lbm_ens **out) {
    if (!ens_desc_ok(desc, reps) || !pop_a || !pop_b || !scratch || !r || !v || !out)
        return LBM_E_INVAL;
    if (!aligned(pop_a) || !aligned(pop_b) || !aligned(scratch) || pop_a == pop_b) return LBM_E_INVAL;
    const EnsLayout L = ens_layout(desc, reps);
    lbm_ens *e = static_cast<lbm_ens *>(calloc(1, sizeof(lbm_ens)));
    if (!e) return LBM_E_DEVICE;
    e->desc = *desc;
    e->nrep = desc->nrep;
    e->host_reps = static_cast<lbm_replica_desc *>(malloc(sizeof(lbm_replica_desc) * e->nrep));
    e->host_table = static_cast<Replica *>(calloc(e->nrep, sizeof(Replica)));
    uint16_t *blk[kNumGeomShapes];
    for (int s = 0; s < kNumGeomShapes; ++s)
        blk[s] = static_cast<uint16_t *>(malloc(size_t(L.total_blocks[s]) * 2 + 2));
    uint16_t *prep = static_cast<uint16_t *>(malloc(size_t(L.n) * 2));
    uint16_t *two = static_cast<uint16_t *>(malloc(size_t(L.two_blocks) * 2 + 2));
    bool ok = e->host_reps && e->host_table && prep && two;
    for (int s = 0; s < kNumGeomShapes; ++s) ok = ok && blk[s];
    if (!ok) {
        for (int s = 0; s < kNumGeomShapes; ++s) free(blk[s]);
        free(prep);
        free(two);
        free(e->host_reps);
        free(e->host_table);
        free(e);
        return LBM_E_DEVICE;
    }
    memcpy(e->host_reps, reps, sizeof(lbm_replica_desc) * e->nrep);
    e->elem = elem_size(desc->storage);
    e->pop[0] = pop_a;
    e->pop[1] = pop_b;
    e->stream = static_cast<hipStream_t>(stream);
    if (desc->storage == LBM_STORE_F16) {
        e->enc_s = ldexp(1.0, desc->f16_scale_log2);
        e->dec_s = ldexp(1.0, -desc->f16_scale_log2);
    } else {
        e->enc_s = e->dec_s = 1.0;
    }
    e->total_cells = L.total_cells;
    e->total_pop = L.total_pop;
    e->total_mask_words = L.total_mask_words;
    e->device = current_device();
    // until lbm_ens_autotune: the last choice for this key, else by lattice size
    {
        const int code = tune_lookup(ens_tune_key(e), L.lattice_bytes >= kStreamStoreBytes ? kNumGeomShapes : 0);
        e->shape = code % kNumShapes;
        e->order = (code / kNumShapes) % int(kNumOrders);
        e->cap = (code / (kNumShapes * int(kNumOrders))) % kNumCaps;
        // applied to every box below (the rest state is all zeros)
        e->rows = 1 << ((code / (kNumShapes * int(kNumOrders) * kNumCaps)) % (kMaxRowsLog2 + 1));
        const int two = code / kTuneTwo;  // remembered two-step choice + 1, 0: none
        e->two_possible = L.two_ok;
        e->two = e->two_possible && (two == 0 || two - 1 > 0);
        e->two_nts = L.lattice_bytes >= kTwoStepStreamBytes && L.two_stream;
        int v = 0;
        e->lds_cu = (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                                           e->device) == hipSuccess) ? v : 0;
        e->lds_block = (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock,
                                              e->device) == hipSuccess) ? v : 0;
        if (ens_sweep_lds(e, e->cap, config_block(e->shape)) < 0) e->cap = 0;
    }
    for (int s = 0; s < kNumGeomShapes; ++s) e->total_blocks[s] = L.total_blocks[s];
    e->n = L.n;
    char *base = static_cast<char *>(scratch);
    e->reps = reinterpret_cast<Replica *>(base + L.o_reps);
    for (int s = 0; s < kNumGeomShapes; ++s) e->blk_rep[s] = reinterpret_cast<uint16_t *>(base + L.o_blk[s]);
    e->part_rep = reinterpret_cast<uint16_t *>(base + L.o_part);
    e->two_rep = reinterpret_cast<uint16_t *>(base + L.o_two);
    e->two_blocks = L.two_blocks;
    e->two_threads = L.two_threads;
    for (int k = 0; k < L.fields; ++k) {
        e->mask[k] = reinterpret_cast<uint32_t *>(base + L.o_mask[k]);
        e->force[k] = reinterpret_cast<long long *>(base + L.o_force[k]);
    }
    for (int k = 0; k < 2; ++k) e->cells[k] = reinterpret_cast<uint32_t *>(base + L.o_cells[k]);
    e->fh = reinterpret_cast<double *>(base + L.o_fh);
    e->fr = reinterpret_cast<double *>(base + L.o_fr);
    e->clock = reinterpret_cast<EnsClock *>(base + L.o_clock);
    e->err = reinterpret_cast<uint32_t *>(base + L.o_err);
    e->partials = reinterpret_cast<double *>(base + L.o_partials);
    e->result = reinterpret_cast<double *>(base + L.o_result);
    e->r = r;
    e->v = v;
    e->use_graph = 1;
    // replica table, block and particle maps
    uint64_t pop_off = 0, cell_off = 0, mask_off = 0;
    uint32_t first[kNumGeomShapes] = {0, 0, 0, 0};
    uint32_t part_off = 0, first_two = 0;
    for (int32_t k = 0; k < e->nrep; ++k) {
        const lbm_replica_desc &rd = reps[k];
        Replica &t = e->host_table[k];
        t.g.nx = uint32_t(rd.nx);
        t.g.ny = uint32_t(rd.ny);
        t.g.nz = uint32_t(rd.nz);
        t.g.ncell = uint32_t(uint64_t(rd.nx) * rd.ny * rd.nz);
        t.g.chunk = ens_chunk(rd.nx);
        t.g = with_rows_per_group(t.g, ens_box_rows(e->rows, rd.ny));
        t.pop_off = pop_off;
        t.cell_off = cell_off;
        t.mask_off = uint32_t(mask_off);
        t.part_off = part_off;
        t.npart = uint32_t(rd.n);
        t.replica_id = rd.replica;
        t.seed = rd.seed;
        t.omega = 1.0 / rd.tau;
        const double nu = (rd.tau - 0.5) / 3.0;
        t.R = desc->radius > 0.0 ? desc->radius : desc->gamma / (6.0 * M_PI * nu);
        for (int s = 0; s < kNumGeomShapes; ++s) {
            t.first_block[s] = first[s];
            const uint64_t band = (rd.ny % kShapes[s].cpt == 0) ? t.g.ncell / kShapes[s].cpt : 0;
            const uint32_t nb = uint32_t((band + kShapes[s].bs - 1) / kShapes[s].bs);
            for (uint32_t b = 0; b < nb; ++b) blk[s][first[s] + b] = uint16_t(k);
            first[s] += nb;
        }
        t.two = L.two[size_t(k)];
        t.first_two = first_two;
        for (uint32_t b = 0; b < t.two.ntx * t.two.nty * t.two.nslab; ++b) two[first_two++] = uint16_t(k);
        for (int32_t q = 0; q < rd.n; ++q) prep[part_off + q] = uint16_t(k);
        pop_off += uint64_t(t.g.chunk) * D3Q19::Q * rd.ny * rd.nz;
        cell_off += t.g.ncell;
        mask_off += mask_words(t.g.ncell);
        part_off += uint32_t(rd.n);
    }
    hipError_t err = hipMemsetAsync(pop_a, 0, L.lattice_bytes, e->stream);
    if (err == hipSuccess) err = hipMemsetAsync(pop_b, 0, L.lattice_bytes, e->stream);
    if (err == hipSuccess) err = hipMemsetAsync(scratch, 0, L.scratch_bytes, e->stream);
    if (err == hipSuccess)
        err = hipMemsetAsync(e->cells[0], 0xFF, 2 * align_up(size_t(L.n) * 8 * 4, kAlign), e->stream);
    if (err == hipSuccess)
        err = hipMemcpyAsync(e->reps, e->host_table, sizeof(Replica) * e->nrep,
                             hipMemcpyHostToDevice, e->stream);
    for (int s = 0; s < kNumGeomShapes && err == hipSuccess; ++s)
        if (L.total_blocks[s] > 0)
            err = hipMemcpyAsync(e->blk_rep[s], blk[s], size_t(L.total_blocks[s]) * 2,
                                 hipMemcpyHostToDevice, e->stream);
    if (err == hipSuccess)
        err = hipMemcpyAsync(e->part_rep, prep, size_t(L.n) * 2, hipMemcpyHostToDevice, e->stream);
    if (err == hipSuccess && L.two_blocks > 0)
        err = hipMemcpyAsync(e->two_rep, two, size_t(L.two_blocks) * 2, hipMemcpyHostToDevice, e->stream);
    if (err == hipSuccess) err = hipStreamSynchronize(e->stream);  // host staging is freed below
    for (int s = 0; s < kNumGeomShapes; ++s) free(blk[s]);
    free(prep);
    free(two);
    if (err != hipSuccess) {
        free(e->host_reps);
        free(e->host_table);
        free(e);
        return LBM_E_DEVICE;
    }
    *out = e;
    return LBM_OK;
}

lbm_status lbm_ens_use_graph(lbm_ens *e, int32_t use) {
    if (!e || (use != 0 && use != 1)) return LBM_E_INVAL;
    e->use_graph = use;
    if (!use) ens_drop_graph(e);
    return LBM_OK;
}

lbm_status lbm_ens_vacf_config(lbm_ens *e, int32_t max_lag, int32_t stride, double *acc,
                               double *origins) {
    if (!e) return LBM_E_INVAL;
    ens_drop_graph(e);
    if (max_lag == -1) {
        e->vacf_on = 0;
        return LBM_OK;
    }
    if (max_lag < 0 || stride < 1 || !acc || !origins) return LBM_E_INVAL;
    e->max_lag = max_lag;
    e->stride = stride;
    e->nslot = max_lag / stride + 1;
    e->acc = acc;
    e->origins = origins;
    e->vacf_t = 0;
    const EnsClock clk{e->step, 0};
    hipError_t err = hipMemsetAsync(acc, 0, size_t(e->n) * size_t(max_lag + 1) * 8, e->stream);
    if (err == hipSuccess)
        err = hipMemcpyAsync(e->clock, &clk, sizeof(clk), hipMemcpyHostToDevice, e->stream);
    if (err == hipSuccess) err = hipStreamSynchronize(e->stream);
    if (err != hipSuccess) return LBM_E_DEVICE;
    e->vacf_on = 1;
    return LBM_OK;
}

lbm_status lbm_ens_vacf_counts(const lbm_ens *e, int64_t *cnt) {
    if (!e || !cnt) return LBM_E_INVAL;
    if (!e->vacf_on) return LBM_E_STATE;
    const int64_t T = e->vacf_t;
    for (int32_t l = 0; l <= e->max_lag; ++l)
        cnt[l] = (T - 1 - l >= 0) ? (T - 1 - l) / e->stride + 1 : 0;
    return LBM_OK;
}

lbm_status lbm_ens_step(lbm_ens *e, int32_t nsteps) {
    if (!e || nsteps < 0) return LBM_E_INVAL;
    int32_t left = nsteps;
    auto eager = [&](int sweep) {
        const int32_t k = sweep ? 2 : 1;
        ens_dispatch_step(e, e->cur, e->step, sweep);
        e->cur ^= 1;
        e->step += k;
        if (e->vacf_on) e->vacf_t += k;
        left -= k;
    };
    if (e->use_graph) {
        if (left > 0 && (e->step & 1)) eager(0);
        constexpr int32_t per = LBM_ENS_GRAPH_STEPS;
        if (left >= per && !e->graph_valid && !ens_capture(e)) e->use_graph = 0;  // plain launches
        if (left >= per && e->graph_valid) {
            // the graph was captured from lattice parity cur at an even step;
            // cur and the step parity change together, so they still match
            while (left >= per) {
                if (hipGraphLaunch(e->graph, e->stream) != hipSuccess) return LBM_E_DEVICE;
                e->graph_replays += 1;
                e->step += per;
                if (e->vacf_on) e->vacf_t += per;
                left -= per;
            }
        }
    }
    // an even number of two-step sweeps, so that n steps leave the state in the
    // lattice n swaps away
    while (e->two && left >= 4) {
        eager(1);
        eager(2);
    }
    while (left > 0) eager(0);
    return launch_status();
}

lbm_status lbm_ens_autotune(lbm_ens *e, int32_t iters, double *ms, int32_t *chosen) {
    if (!e || iters < 1 || iters > 10000) return LBM_E_INVAL;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return LBM_E_DEVICE;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return LBM_E_DEVICE;
    }
    // the timing launches advance the device clock; restore it afterwards
    EnsClock saved;
    hipError_t err = hipMemcpyAsync(&saved, e->clock, sizeof(saved), hipMemcpyDeviceToHost, e->stream);
    if (err == hipSuccess) err = hipStreamSynchronize(e->stream);
    double best_k[kNumShapes];
    for (int k = 0; k < kNumShapes; ++k) best_k[k] = -1.0;
    // every launch timed: configuration, order, cap, layout (log2 of the rows
    // per group requested of all boxes), ms
    struct Trial {
        int k, o, c, l;
        double t;
    };
    std::vector<Trial> trials;
    const size_t lat = size_t(e->total_cells) * D3Q19::Q * e->elem;
    bool ok = err == hipSuccess;
    auto time_in = [&](int l, int k, int o, int c, int32_t n) -> double {
        if (!ok) return -1.0;
        if (ens_set_layout(e, 1 << l) != LBM_OK) {
            ok = false;
            return -1.0;
        }
        const double v = ens_time_launch(e, k, o, c, n, e0, e1);
        if (v < 0.0) ok = false;
        return v;
    };
    auto note = [&](int k, int o, int c, int l, double v) {
        if (v <= 0.0) return;
        if (best_k[k] <= 0.0 || v < best_k[k]) best_k[k] = v;
        if (config_tunable(k, lat)) trials.push_back(Trial{k, o, c, l, v});
    };
    // Stage 1: every configuration in linear order without a residency cap,
    // in every layout; keep the layout of the fastest launch.
    double t1[kMaxRowsLog2 + 1][kNumShapes];
    int bl = -1, first = -1;
    for (int l = 0; l <= kMaxRowsLog2 && ok; ++l)
        for (int k = 0; k < kNumShapes && ok; ++k) {
            t1[l][k] = ens_launch_ok(e, k, 0) ? time_in(l, k, int(kOrderLinear), 0, iters) : -1.0;
            note(k, int(kOrderLinear), 0, l, t1[l][k]);
            if (!config_tunable(k, lat)) t1[l][k] = -1.0;
            if (t1[l][k] > 0.0 && (bl < 0 || t1[l][k] < t1[bl][first])) bl = l, first = k;
        }
    if (bl < 0) ok = false;
    // Stage 2: in that layout, its two fastest configurations with every block
    // order and cap.
    Trial best{first, int(kOrderLinear), 0, bl, ok ? t1[bl][first] : 0.0};
    if (ok) {
        int second = -1;
        for (int k = 0; k < kNumShapes; ++k)
            if (k != first && t1[bl][k] > 0.0 && (second < 0 || t1[bl][k] < t1[bl][second])) second = k;
        for (int k : {first, second}) {
            if (k < 0) continue;
            for (int o = 0; o < int(kNumOrders) && ok; ++o)
                for (int c = 0; c < kNumCaps && ok; ++c) {
                    if ((o == int(kOrderLinear) && c == 0) || !ens_launch_ok(e, k, c)) continue;
                    const double v = time_in(bl, k, o, c, iters);
                    note(k, o, c, bl, v);
                    if (v > 0.0 && v < best.t) best = Trial{k, o, c, bl, v};
                }
        }
    }
    // Stage 3: that launch in every other layout (a cap or order can change
    // which layout streams best).
    if (ok && (best.o != int(kOrderLinear) || best.c != 0)) {
        const Trial b0 = best;
        for (int l = 0; l <= kMaxRowsLog2 && ok; ++l)
            if (l != b0.l) note(b0.k, b0.o, b0.c, l, time_in(l, b0.k, b0.o, b0.c, iters));
    }
    // Stage 4: the three fastest launches timed again, in turn, twice each
    // with twice the iterations; the lowest total wins.
    if (ok) {
        std::sort(trials.begin(), trials.end(), [](const Trial &x, const Trial &y) { return x.t < y.t; });
        const int m = int(std::min<size_t>(3, trials.size()));
        double total[3] = {0.0, 0.0, 0.0};
        for (int round = 0; round < 2 && ok; ++round)
            for (int j = 0; j < m && ok; ++j) {
                const double v = time_in(trials[j].l, trials[j].k, trials[j].o, trials[j].c, 2 * iters);
                total[j] += v > 0.0 ? v : 1e30;
            }
        int jb = 0;
        for (int j = 1; j < m; ++j)
            if (total[j] < total[jb]) jb = j;
        if (m > 0) best = trials[jb];
    }
    if (ok && ens_set_layout(e, 1 << best.l) != LBM_OK) ok = false;
    // Two-step sweeps, if two steps in one are faster than two of that launch.
    int two = 0;
    if (ok && e->two_possible) {
        void *A = e->pop[e->cur], *B = e->pop[e->cur ^ 1];
        const ForceField last = ens_field(e, (e->step + 1) & 1);
        const EnsTwoStepArgs a = ens_two_step_args(e, e->cur, last, last);
        hipError_t st = hipSuccess;
        const double one = time_as_in_a_run(e->stream, A, B, lat, config_nts(best.k), 2 * iters,
                                            [&] { ens_time_any(e, best.k, best.o, best.c); }, &st);
        ok = st == hipSuccess;
        double both = -1.0;
        if (ok) both = time_as_in_a_run(e->stream, A, B, lat, a.nts, 2 * iters, [&] { ens_two_steps_any(e, a); }, &st);
        ok = st == hipSuccess && launch_status() == LBM_OK && one > 0.0 && both > 0.0;
        two = ok && both < 2.0 * one;
    }
    if (ok) {
        err = hipMemcpyAsync(e->clock, &saved, sizeof(saved), hipMemcpyHostToDevice, e->stream);
        if (err == hipSuccess) err = hipStreamSynchronize(e->stream);
        ok = err == hipSuccess;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!ok) return LBM_E_DEVICE;
    if (best.k != e->shape || best.o != e->order || best.c != e->cap || two != e->two) ens_drop_graph(e);
    e->shape = best.k;
    e->order = best.o;
    e->cap = best.c;
    e->two = two;
    // the trial's outcome; nothing of it where these particles leave no choice
    tune_store(ens_tune_key(e),
               tune_code(best.k, best.o, best.c, best.l) + (e->two_possible ? kTuneTwo * (two + 1) : 0));
    if (ms)
        for (int k = 0; k < kNumShapes; ++k) ms[k] = best_k[k];
    if (chosen) *chosen = best.k;
    return LBM_OK;
}

lbm_status lbm_ens_get_two_step(const lbm_ens *e, int32_t *two) {
    if (!e || !two) return LBM_E_INVAL;
    *two = e->two;
    return LBM_OK;
}

lbm_status lbm_ens_set_sweep_launch(lbm_ens *e, int32_t order, int32_t waves_per_simd) {
    if (!e || order < 0 || order >= int32_t(kNumOrders)) return LBM_E_INVAL;
    int cap = -1;
    for (int j = 0; j < kNumCaps; ++j)
        if (kResidencyCaps[j] == waves_per_simd) cap = j;
    if (cap < 0 || ens_sweep_lds(e, cap, config_block(e->shape)) < 0) return LBM_E_INVAL;
    if (order != e->order || cap != e->cap) ens_drop_graph(e);
    e->order = order;
    e->cap = cap;
    return LBM_OK;
}

lbm_status lbm_ens_get_sweep_launch(const lbm_ens *e, int32_t *order, int32_t *waves_per_simd) {
    if (!e || !order || !waves_per_simd) return LBM_E_INVAL;
    *order = e->order;
    *waves_per_simd = kResidencyCaps[e->cap];
    return LBM_OK;
}

lbm_status lbm_ens_set_layout(lbm_ens *e, int32_t rows_per_group) {
    if (!e || rows_per_group < 1 || rows_per_group > (1 << kMaxRowsLog2) ||
        (rows_per_group & (rows_per_group - 1)) != 0)
        return LBM_E_INVAL;
    return ens_set_layout(e, rows_per_group);
}

lbm_status lbm_ens_get_layout(const lbm_ens *e, int32_t replica, int32_t *rows_per_group) {
    if (!e || !rows_per_group || replica < 0 || replica >= e->nrep) return LBM_E_INVAL;
    *rows_per_group = int32_t(e->host_table[replica].g.ymask + 1);
    return LBM_OK;
}

lbm_status lbm_ens_stream_ceiling(lbm_ens *e, int32_t k, int32_t iters, double *ms) {
    if (!e || !ms || iters < 1 || iters > 10000) return LBM_E_INVAL;
    if (k < 0) k = e->shape;
    if (k >= kNumShapes || config_row(k) || e->total_blocks[k & 3] == 0) return LBM_E_INVAL;
    for (int32_t q = 0; q < e->nrep; ++q)
        if (e->host_reps[q].ny % kShapes[k & 3].cpt != 0) return LBM_E_INVAL;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return LBM_E_DEVICE;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return LBM_E_DEVICE;
    }
    for (int w = 0; w < 2; ++w) ens_stream_only_any(e, k);
    (void)hipEventRecord(e0, e->stream);
    for (int32_t it = 0; it < iters; ++it) ens_stream_only_any(e, k);
    (void)hipEventRecord(e1, e->stream);
    hipError_t err = hipEventSynchronize(e1);
    float f = 0.0f;
    if (err == hipSuccess) err = hipEventElapsedTime(&f, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (err != hipSuccess || launch_status() != LBM_OK) return LBM_E_DEVICE;
    *ms = double(f) / iters;
    return LBM_OK;
}

lbm_status lbm_ens_observables(lbm_ens *e, int32_t replica, double out[7]) {
    if (!e || !out || replica < 0 || replica >= e->nrep) return LBM_E_INVAL;
    const Replica &t = e->host_table[replica];
    const char *A = static_cast<const char *>(e->pop[e->cur]) + t.pop_off * e->elem;
    switch (e->desc.storage) {
#define LBM_ENS_PARTIALS(CODEC)                                                                 \
    hipLaunchKernelGGL(k_fluid_partials<CODEC>, dim3(kRedBlocks), dim3(kBlock), 0, e->stream, \
                       reinterpret_cast<const CODEC::T *>(A), t.g, CODEC::R(e->dec_s),          \
                       e->partials)
        case LBM_STORE_F64: LBM_ENS_PARTIALS(F64Q19); break;
        case LBM_STORE_F32: LBM_ENS_PARTIALS(F32Q19); break;
        case LBM_STORE_BF16: LBM_ENS_PARTIALS(BF16Q19); break;
        case LBM_STORE_F16: LBM_ENS_PARTIALS(F16Q19); break;
#undef LBM_ENS_PARTIALS
    }
    hipLaunchKernelGGL(k_final_sums, dim3(1), dim3(kBlock), 0, e->stream, e->partials, kRedBlocks,
                       double(t.g.ncell), e->v + 3 * uint64_t(t.part_off), int32_t(t.npart),
                       e->desc.mass, e->result);
    if (launch_status() != LBM_OK) return LBM_E_DEVICE;
    double host[7];
    uint32_t flag = 0;
    hipError_t err = hipMemcpyAsync(host, e->result, sizeof(host), hipMemcpyDeviceToHost, e->stream);
    if (err == hipSuccess)
        err = hipMemcpyAsync(&flag, e->err, sizeof(flag), hipMemcpyDeviceToHost, e->stream);
    if (err == hipSuccess) err = hipStreamSynchronize(e->stream);
    if (err != hipSuccess) return LBM_E_DEVICE;
    bool finite = true;
    for (int k = 0; k < 7; ++k) {
        out[k] = host[k];
        finite = finite && isfinite(host[k]);
    }
    return (finite && flag == 0) ? LBM_OK : LBM_E_NONFINITE;
}

lbm_status lbm_ens_get_populations(lbm_ens *e, int32_t replica, double *f) {
    if (!e || !f || replica < 0 || replica >= e->nrep) return LBM_E_INVAL;
    const Replica &t = e->host_table[replica];
    const char *A = static_cast<const char *>(e->pop[e->cur]) + t.pop_off * e->elem;
    switch (e->desc.storage) {
#define LBM_ENS_POPS(CODEC)                                                                      \
    hipLaunchKernelGGL(k_get_populations<CODEC>, dim3(blocks_for(t.g.ncell)), dim3(kBlock), 0, \
                       e->stream, reinterpret_cast<const CODEC::T *>(A), t.g, CODEC::R(e->dec_s), f)
        case LBM_STORE_F64: LBM_ENS_POPS(F64Q19); break;
        case LBM_STORE_F32: LBM_ENS_POPS(F32Q19); break;
        case LBM_STORE_BF16: LBM_ENS_POPS(BF16Q19); break;
        case LBM_STORE_F16: LBM_ENS_POPS(F16Q19); break;
#undef LBM_ENS_POPS
    }
    return launch_status();
}

lbm_status lbm_ens_set_shape(lbm_ens *e, int32_t k) {
    if (!e || !ens_launch_ok(e, k, 0)) return LBM_E_INVAL;
    const int cap = ens_sweep_lds(e, e->cap, config_block(k)) < 0 ? 0 : e->cap;  // cap not possible here
    if (k != e->shape || cap != e->cap) ens_drop_graph(e);
    e->shape = k;
    e->cap = cap;
    return LBM_OK;
}

lbm_status lbm_ens_get_shape(const lbm_ens *e, int32_t *k) {
    if (!e || !k) return LBM_E_INVAL;
    *k = e->shape;
    return LBM_OK;
}

lbm_status lbm_ens_get_step(const lbm_ens *e, int64_t *step) {
    if (!e || !step) return LBM_E_INVAL;
    *step = e->step;
    return LBM_OK;
}

lbm_status lbm_ens_graph_replays(const lbm_ens *e, int64_t *replays) {
    if (!e || !replays) return LBM_E_INVAL;
    *replays = e->graph_replays;
    return LBM_OK;
}

lbm_status lbm_ens_destroy(lbm_ens *e) {
    if (!e) return LBM_E_INVAL;
    ens_drop_graph(e);
    if (e->cap_stream) (void)hipStreamDestroy(e->cap_stream);
    free(e->host_reps);
    free(e->host_table);
    free(e);
    return LBM_OK;
}

}  // extern "C"

// ===========================================================================
// Reverse mode: recorded forward runs and their adjoint.
// ===========================================================================
namespace {

// One checkpoint: the lattice as stored (post-collision values at their
// source node) and the particle state r[n][3], v[n][3].
struct TapeLayout {
    size_t lat, part, slot;
};

TapeLayout tape_layout(const lbm_ctx *c, int32_t np) {
    TapeLayout t;
    lbm_lattice_bytes(&c->desc, &t.lat);
    t.part = align_up(size_t(np) * 6 * 8, kAlign);
    t.slot = t.lat + t.part;
    return t;
}

// The FP64 adjoint lattice: interleaved rows of 128-byte-aligned doubles, one
// row per group whatever the forward lattice's layout.
Grid adj_grid(const lbm_ctx *c) {
    Grid gd = c->g;
    gd.chunk = uint32_t(align_up(c->g.nx, 16));
    return with_rows_per_group(gd, 1);
}

size_t adj_lattice_bytes(const lbm_ctx *c) {
    const Grid gd = adj_grid(c);
    return align_up(size_t(gd.chunk) * size_t(c->q) * gd.ny * gd.nz * 8, kAlign);
}

struct AdjLayout {
    size_t seg_lat, seg_part;  // `every` lattice / particle states of one segment
    size_t abar[2];            // adjoint lattices
    size_t uf[2], um[2];       // adjoint node fields and their flags
    size_t ff[2], fm[2];       // node-force fields of the forward recompute
    size_t prev_fwd, prev_adj, fh, fr, pgrad, wacc;
    size_t plist, fpair, fcbar;  // pair forces (when recorded with them)
    size_t total;
};

AdjLayout adj_layout(const lbm_ctx *c, int32_t np, int32_t every) {
    AdjLayout L;
    const TapeLayout t = tape_layout(c, np);
    const size_t field = force_field_bytes(&c->desc);
    const size_t mask = align_up(size_t(c->mask_words) * 4, kAlign);
    const size_t pcell = align_up(size_t(np) * 8 * 4, kAlign);
    size_t o = 0;
    L.seg_lat = o;
    o += size_t(every) * t.lat;
    L.seg_part = o;
    o += size_t(every) * t.part;
    for (int k = 0; k < 2; ++k) {
        L.abar[k] = o;
        o += adj_lattice_bytes(c);
    }
    for (int k = 0; k < 2; ++k) {
        L.uf[k] = o;
        o += field;
        L.um[k] = o;
        o += mask;
    }
    for (int k = 0; k < 2; ++k) {
        L.ff[k] = o;
        o += field;
        L.fm[k] = o;
        o += mask;
    }
    L.prev_fwd = o;
    o += pcell;
    L.prev_adj = o;
    o += pcell;
    L.fh = o;
    o += align_up(size_t(np) * 3 * 8, kAlign);
    L.fr = o;
    o += align_up(size_t(np) * 3 * 8, kAlign);
    L.pgrad = o;
    o += align_up(size_t(np) * 4 * 8, kAlign);
    L.wacc = o;
    o += align_up(size_t(blocks_for(c->g.ncell)) * 8, kAlign);
    L.plist = o;
    o += pair_list_bytes(np);
    L.fpair = o;
    o += align_up(size_t(np) * 3 * 8, kAlign);
    L.fcbar = o;
    o += align_up(size_t(np) * 3 * 8, kAlign);
    L.total = o;
    return L;
}

bool adjoint_storage(const lbm_ctx *c) {
    return c->desc.storage == LBM_STORE_F64 || c->desc.storage == LBM_STORE_F32;
}

// The adjoint stream-collide, addressing by wavefront rows where every
// wavefront lies in one lattice row (64 | nx), by per-lane 64-bit indices
// otherwise.
template <class C, bool FORCED, bool NTS>
void launch_adj_collide(hipStream_t st, unsigned cgrid, const typename C::T *A, const Grid &g,
                        typename C::R dec_s, const double *Abar, double *Bbar, const Grid &gd,
                        double omega, AdjField uf, double *wacc) {
    if (g.nx % 64 == 0)
        hipLaunchKernelGGL((k_adj_collide<C, FORCED, NTS, true>), dim3(cgrid), dim3(kBlock), 0, st, A, g,
                           dec_s, Abar, Bbar, gd, omega, uf, wacc);
    else
        hipLaunchKernelGGL((k_adj_collide<C, FORCED, NTS, false>), dim3(cgrid), dim3(kBlock), 0, st, A, g,
                           dec_s, Abar, Bbar, gd, omega, uf, wacc);
}

template <class C>
hipError_t adjoint_run(lbm_ctx *c, char *tape, char *work, double *adj_pop, double *adj_r,
                       double *adj_v, double *adj_param) {
    using T = typename C::T;
    using R = typename C::R;
    const int32_t np = c->rec_np, N = c->rec_nsteps, K = c->rec_every;
    const lbm_particle_desc &pd = c->rec_pdesc;
    const TapeLayout t = tape_layout(c, np);
    const AdjLayout L = adj_layout(c, np, K);
    const Grid gd = adj_grid(c);
    hipStream_t st = c->stream;
    const size_t field = force_field_bytes(&c->desc);
    const size_t mask = size_t(c->mask_words) * 4;
    const size_t pbytes = size_t(np) * 3 * 8;
    auto at = [&](size_t off) { return work + off; };
    auto seg = [&](int32_t k) { return reinterpret_cast<T *>(at(L.seg_lat + size_t(k) * t.lat)); };
    auto seg_r = [&](int32_t k) { return reinterpret_cast<double *>(at(L.seg_part + size_t(k) * t.part)); };
    auto seg_v = [&](int32_t k) { return seg_r(k) + 3 * size_t(np); };
    double *abar[2] = {reinterpret_cast<double *>(at(L.abar[0])),
                       reinterpret_cast<double *>(at(L.abar[1]))};
    AdjField uf[2], ff_unused{nullptr, nullptr};
    ForceField ff[2];
    for (int k = 0; k < 2; ++k) {
        uf[k] = AdjField{reinterpret_cast<double *>(at(L.uf[k])), reinterpret_cast<uint32_t *>(at(L.um[k]))};
        ff[k] = ForceField{reinterpret_cast<long long *>(at(L.ff[k])), reinterpret_cast<uint32_t *>(at(L.fm[k]))};
    }
    double *pgrad = reinterpret_cast<double *>(at(L.pgrad));
    double *wacc = reinterpret_cast<double *>(at(L.wacc));
    const PairList plist = pair_list_at(at(L.plist), np);
    double *fpair = reinterpret_cast<double *>(at(L.fpair));
    double *fcbar = reinterpret_cast<double *>(at(L.fcbar));
    const bool pairs = c->rec_pair_on && np > 0;
    uint32_t *prev_fwd = reinterpret_cast<uint32_t *>(at(L.prev_fwd));
    uint32_t *prev_adj = reinterpret_cast<uint32_t *>(at(L.prev_adj));

    hipError_t e = hipSuccess;
    auto memset_ = [&](void *p, int v, size_t n) {
        if (e == hipSuccess && n) e = hipMemsetAsync(p, v, n, st);
    };
    auto copy_ = [&](void *dst, const void *src, size_t n) {
        if (e == hipSuccess && n) e = hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToDevice, st);
    };
    for (int k = 0; k < 2; ++k) {
        memset_(uf[k].u, 0, field);
        memset_(uf[k].mask, 0, mask);
    }
    memset_(prev_adj, 0xFF, size_t(np) * 8 * 4);
    memset_(pgrad, 0, size_t(np) * 4 * 8);
    memset_(wacc, 0, size_t(blocks_for(c->g.ncell)) * 8);
    if (pairs && e == hipSuccess) e = pair_list_clear(st, plist, c->rec_pg.T);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_adj_import<typename C::V>, dim3(blocks_for(c->g.ncell)), dim3(kBlock), 0, st, adj_pop,
                       abar[0], gd);

    // Forward recompute: the particle kernel without VACF or sums.
    ParticleArgs pa{};
    pa.fh = reinterpret_cast<double *>(at(L.fh));
    pa.fr = reinterpret_cast<double *>(at(L.fr));
    pa.cells = prev_fwd;
    pa.last_cells = prev_fwd;
    pa.older_cells = nullptr;
    pa.err = c->err;
    pa.n = np;
    pa.friction = pd.friction;
    pa.mass = pd.mass;
    pa.gamma = pd.gamma;
    pa.sig = pd.kT > 0.0 ? sqrt(2.0 * pd.gamma * pd.kT) : 0.0;
    pa.R = c->rec_R;
    pa.seed = pd.seed;
    pa.replica = pd.replica;
    pa.acc = nullptr;
    pa.origins = nullptr;
    pa.pmom = nullptr;
    pa.fext = c->rec_fext;
    pa.k_hi = -1;
    pa.nslot = pa.stride = 1;
    pa.slot_lo = 0;

    AdjParticleArgs ap{};
    ap.rbar = adj_r;
    ap.vbar = adj_v;
    ap.pgrad = pgrad;
    ap.fext = c->rec_fext;
    ap.prev_cell = prev_adj;
    ap.n = np;
    ap.friction = pd.friction;
    ap.mass = pd.mass;
    ap.gamma = pd.gamma;
    ap.kT = pd.kT;
    ap.sig = pa.sig;
    ap.R = c->rec_R;
    if (pd.radius > 0.0) {
        ap.dR_dgamma = ap.dR_dtau = 0.0;
    } else {
        const double nu = (c->desc.tau - 0.5) / 3.0;
        ap.dR_dgamma = 1.0 / (6.0 * M_PI * nu);
        ap.dR_dtau = -c->rec_R / (3.0 * nu);
    }
    ap.seed = pd.seed;
    ap.replica = pd.replica;
    const unsigned pgrid = np > 0 ? unsigned(particle_blocks(np)) : 0;
    const unsigned cgrid = blocks_for(c->g.ncell);
    // the adjoint lattice is FP64: stream its stores once it outgrows the cache
    const bool stream_stores = adj_lattice_bytes(c) >= kStreamStoreBytes;

    int cur = 0;
    const int32_t nseg = (N + K - 1) / K;
    for (int32_t j = nseg - 1; j >= 0 && e == hipSuccess; --j) {
        const int32_t len = (N - j * K) < K ? (N - j * K) : K;
        const char *slot = tape + size_t(j) * t.slot;
        copy_(seg(0), slot, t.lat);
        copy_(seg_r(0), slot + t.lat, 2 * pbytes);
        if (np > 0 && len > 1) {
            for (int k = 0; k < 2; ++k) {
                memset_(ff[k].f, 0, field);
                memset_(ff[k].mask, 0, mask);
            }
            memset_(prev_fwd, 0xFF, size_t(np) * 8 * 4);
        }
        for (int32_t k = 0; k + 1 < len && e == hipSuccess; ++k) {
            const int64_t n = c->rec_n0 + int64_t(j) * K + k;
            const int par = int(n & 1);
            if (np > 0) {
                pa.r = seg_r(k);
                pa.v = seg_v(k);
                pa.r_out = seg_r(k + 1);
                pa.v_out = seg_v(k + 1);
                pa.step = uint32_t(n);
                pa.fpair = nullptr;
                if (pairs) {
                    launch_pairs(st, seg_r(k), np, c->rec_pg, plist, fpair);
                    pa.fpair = fpair;
                    pa.pair_link = plist.link;
                    pa.pair_head = plist.head;
                }
                hipLaunchKernelGGL(k_particle<C>, dim3(pgrid), dim3(kParticleBlock), 0, st, seg(k),
                                   c->g, R(c->dec_s), pa, ff[par], ff[par ^ 1], ff[par]);
                launch_collide<C, true>(c, seg(k), seg(k + 1), ff[par], c->shape);
            } else {
                launch_collide<C, false>(c, seg(k), seg(k + 1), ff[0], c->shape);
            }
        }
        for (int32_t k = len - 1; k >= 0 && e == hipSuccess; --k) {
            const int64_t n = c->rec_n0 + int64_t(j) * K + k;
            const int par = int(n & 1);
            if (np > 0) {
                ap.r = seg_r(k);
                ap.v = seg_v(k);
                ap.step = uint32_t(n);
                ap.fpair = ap.fcbar = nullptr;
                if (pairs) {
                    launch_pairs(st, seg_r(k), np, c->rec_pg, plist, fpair);
                    ap.fpair = fpair;
                    ap.fcbar = fcbar;
                }
                hipLaunchKernelGGL(k_adj_particle<C>, dim3(pgrid), dim3(kParticleBlock), 0, st,
                                   seg(k), c->g, R(c->dec_s), abar[cur], gd, ap, uf[par],
                                   uf[par ^ 1]);
                if (pairs) {
                    hipLaunchKernelGGL(c->rec_pg.ordered ? k_adj_pair<true> : k_adj_pair<false>, pair_group_blocks(np),
                                       dim3(kPairBlock), 0, st, seg_r(k), np, c->rec_pg, plist, fcbar, adj_r);
                    if (e == hipSuccess) e = pair_list_clear(st, plist, c->rec_pg.T);
                }
                if (stream_stores)
                    launch_adj_collide<C, true, true>(st, cgrid, seg(k), c->g, R(c->dec_s), abar[cur], abar[cur ^ 1], gd,
                                       1.0 / c->desc.tau, uf[par], wacc);
                else
                    launch_adj_collide<C, true, false>(st, cgrid, seg(k), c->g, R(c->dec_s), abar[cur], abar[cur ^ 1], gd,
                                       1.0 / c->desc.tau, uf[par], wacc);
            } else if (stream_stores) {
                launch_adj_collide<C, false, true>(st, cgrid,
                                   seg(k), c->g, R(c->dec_s), abar[cur], abar[cur ^ 1], gd,
                                   1.0 / c->desc.tau, ff_unused, wacc);
            } else {
                launch_adj_collide<C, false, false>(st, cgrid,
                                   seg(k), c->g, R(c->dec_s), abar[cur], abar[cur ^ 1], gd,
                                   1.0 / c->desc.tau, ff_unused, wacc);
            }
            cur ^= 1;
            const hipError_t le = hipGetLastError();
            if (le != hipSuccess) e = le;
        }
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_adj_export<typename C::V>, dim3(cgrid), dim3(kBlock), 0, st, abar[cur], adj_pop, gd);
    hipLaunchKernelGGL(k_adj_params, dim3(1), dim3(kBlock), 0, st, pgrad, np, wacc,
                       int32_t(cgrid), c->desc.tau, adj_param);
    return hipGetLastError();
}

template <class C>
void adjoint_dispatch(lbm_ctx *c, char *tape, char *work, double *adj_pop, double *adj_r,
                      double *adj_v, double *adj_param, hipError_t *e) {
    *e = adjoint_run<C>(c, tape, work, adj_pop, adj_r, adj_v, adj_param);
}

}  // namespace

extern "C" {

lbm_status lbm_tape_bytes(const lbm_ctx *ctx, int32_t nsteps, int32_t every, size_t *bytes) {
    if (!ctx || !bytes || nsteps < 1 || every < 1) return LBM_E_INVAL;
    const TapeLayout t = tape_layout(ctx, ctx->np);
    *bytes = size_t((nsteps + every - 1) / every) * t.slot;
    return LBM_OK;
}

lbm_status lbm_record(lbm_ctx *ctx, int32_t nsteps, int32_t every, void *tape) {
    if (!ctx || nsteps < 1 || every < 1 || !tape || !aligned(tape)) return LBM_E_INVAL;
    if (!adjoint_storage(ctx)) return LBM_E_UNSUPPORTED;
    // the reverse sweep spreads on the unit cell (the cube spreading has no adjoint here)
    if (ctx->np > 0 && ctx->pdesc.friction == LBM_FRICTION_STOKESLET_CUBE) return LBM_E_UNSUPPORTED;
    const TapeLayout t = tape_layout(ctx, ctx->np);
    ctx->rec_tape = tape;
    ctx->rec_n0 = ctx->step;
    ctx->rec_nsteps = nsteps;
    ctx->rec_every = every;
    ctx->rec_np = ctx->np;
    ctx->rec_pdesc = ctx->pdesc;
    ctx->rec_R = ctx->R;
    ctx->rec_fext = ctx->fext;
    ctx->rec_pair_on = ctx->pair_on;
    ctx->rec_pg = ctx->pg;
    ctx->rec_rows = ctx->g.ymask + 1;
    const size_t pbytes = size_t(ctx->np) * 3 * 8;
    char *tp = static_cast<char *>(tape);
    for (int64_t s = 0; s < nsteps; s += every) {
        char *slot = tp + size_t(s / every) * t.slot;
        hipError_t e = hipMemcpyAsync(slot, ctx->pop[ctx->cur], t.lat, hipMemcpyDeviceToDevice, ctx->stream);
        if (e == hipSuccess && pbytes)
            e = hipMemcpyAsync(slot + t.lat, ctx->r, pbytes, hipMemcpyDeviceToDevice, ctx->stream);
        if (e == hipSuccess && pbytes)
            e = hipMemcpyAsync(slot + t.lat + pbytes, ctx->v, pbytes, hipMemcpyDeviceToDevice, ctx->stream);
        if (e != hipSuccess) {
            ctx->rec_tape = nullptr;
            return LBM_E_DEVICE;
        }
        advance(ctx, int32_t(std::min<int64_t>(every, nsteps - s)));
    }
    return launch_status();
}

lbm_status lbm_adjoint_work_bytes(const lbm_ctx *ctx, size_t *bytes) {
    if (!ctx || !bytes) return LBM_E_INVAL;
    if (!ctx->rec_tape) return LBM_E_STATE;
    *bytes = adj_layout(ctx, ctx->rec_np, ctx->rec_every).total;
    return LBM_OK;
}

lbm_status lbm_adjoint(lbm_ctx *ctx, const void *tape, void *work, double *adj_pop,
                       double *adj_r, double *adj_v, double *adj_param) {
    if (!ctx || !tape || !work || !aligned(work) || !adj_pop || !adj_param) return LBM_E_INVAL;
    if (!adjoint_storage(ctx)) return LBM_E_UNSUPPORTED;
    if (ctx->rec_np > 0 && ctx->rec_pdesc.friction == LBM_FRICTION_STOKESLET_CUBE)
        return LBM_E_UNSUPPORTED;
    if (!ctx->rec_tape || tape != ctx->rec_tape) return LBM_E_STATE;
    // the checkpoints hold lattices in the layout they were recorded in
    if (ctx->g.ymask + 1 != ctx->rec_rows) return LBM_E_STATE;
    if (ctx->rec_np > 0 && (!adj_r || !adj_v)) return LBM_E_INVAL;
    hipError_t e = hipSuccess;
    LBM_DISPATCH(ctx, adjoint_dispatch, static_cast<char *>(const_cast<void *>(tape)),
                 static_cast<char *>(work), adj_pop, adj_r, adj_v, adj_param, &e);
    return e == hipSuccess ? LBM_OK : LBM_E_DEVICE;
}

}  // extern "C"
