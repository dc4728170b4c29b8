// Soft repulsion between particles: the conservative force F_C of Eq.
// s2-langevin with the potential of Eq. s2-softpot, read as the conservative
// force of dissipative particle dynamics: a pair closer than the cutoff r_c
// pushes apart with a_f (1 - r/r_c) along the line of centres (nearest
// periodic image).
//
// Neighbours come from a cell list: the box is cut into nc cells per axis
// of edge L/nc >= r_c and the cells are hashed into T buckets (T a power of
// two >= 2n).  One pass links every particle into its bucket's list (an atomic
// exchange of the list head); where cells hold many particles another finds
// every particle's successor in ascending index.  Every particle then walks the
// (up to) 27 cells around its own in a fixed order, each cell's particles in
// ascending index (entries of other cells hashed to the same bucket are
// skipped); the 27 cells go to 27 lanes and their sums are combined in a fixed
// order: the result is bitwise reproducible although the first links are not.
// The adjoint kernel uses the same walk.
//
// For a particle or two per cell each pass is a launch's latency (FP64, 4096
// particles: 4.6 and 5 us).  For m of them a pass is a chain of some m loads:
// cutoffs of up to half the box and clusters are accepted, and an insertion sort
// or a new walk for every few particles made 512 per cell 10.9 and 12.9 ms a
// step, the pass over the links 0.53.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "pair_list.hpp"

namespace lbmbp {

__device__ inline uint32_t pair_cell_coord(double r, double L, uint32_t nc) {
    const double s = r - L * floor(r / L);  // wrapped position
    int32_t c = int32_t(floor(s * double(nc) / L));
    c = c < 0 ? 0 : (c >= int32_t(nc) ? int32_t(nc) - 1 : c);
    return uint32_t(c);
}

__device__ inline uint64_t pair_cell(const PairGrid &pg, uint32_t cx, uint32_t cy, uint32_t cz) {
    return (uint64_t(cz) * pg.nc[1] + cy) * pg.nc[0] + cx;
}

// Fibonacci hashing of the cell index into the T buckets.
__device__ inline uint32_t pair_bucket(uint64_t cell, uint32_t T) {
    return uint32_t((cell * 0x9E3779B97F4A7C15ull) >> 32) & (T - 1u);
}

__global__ __launch_bounds__(kPairBlock) void k_pair_link(const double *__restrict__ r, int32_t n,
                                                          PairGrid pg, PairList pl) {
    const int32_t i = int32_t(blockIdx.x * kPairBlock + threadIdx.x);
    if (i >= n) return;
    const uint32_t cx = pair_cell_coord(r[3 * i + 0], pg.L[0], pg.nc[0]);
    const uint32_t cy = pair_cell_coord(r[3 * i + 1], pg.L[1], pg.nc[1]);
    const uint32_t cz = pair_cell_coord(r[3 * i + 2], pg.L[2], pg.nc[2]);
    const uint64_t cell = pair_cell(pg, cx, cy, cz);
    const uint32_t b = pair_bucket(cell, pg.T);
    pl.link[i] = PairLink{cell, atomicExch(&pl.head[b], uint32_t(i)), b};
}

// The lists in ascending index: a particle's successor is the smallest index
// above its own in its bucket.
__global__ __launch_bounds__(kPairBlock) void k_pair_order(int32_t n, PairGrid pg, PairList pl) {
    const uint32_t i = blockIdx.x * kPairBlock + threadIdx.x;
    if (i >= uint32_t(n)) return;
    const PairLink e = pl.link[i];
    uint32_t next = kPairNone, hops = 0;
    bool lowest = true;
    for (uint32_t j = pl.head[e.bucket]; j != kPairNone && hops < pg.n; ++hops) {
        lowest = lowest && j >= i;
        if (j > i) next = min(next, j);
        j = pl.link[j].next;
    }
    pl.sorted[i] = PairLink{e.cell, next, e.bucket};
    if (lowest) pl.first[e.bucket] = i;
}

// A group of kPairLanes lanes serves one particle: lane l visits the l-th of
// its (up to) 27 neighbour cells (offsets in x fastest, then y, z) and calls
// fn(j, d, |d|^2) for every particle j != i of that cell within the cutoff,
// d = r_i - r_j at the nearest image, in ascending j.
constexpr int kPairLanes = 32;

// Whether m particles of one cell cost more in walks over the links, m^2 / 4
// dependent loads, than in one pass over all n particles, some in flight at a
// time (a cluster among 4096 particles, us per step: 64 of them 213 in walks; 128
// of them 731 in walks, 403 in one pass; 256 of them 1853 and 552).
// Positions that are not finite all fall into one cell: without the bound a run
// that diverges would walk n^2 / 4 links per particle.
__device__ inline bool pair_cluster(uint32_t m, uint32_t n) { return uint64_t(m) * m > 2 * uint64_t(n); }

template <bool ORDERED, typename Fn>
__device__ inline void pair_cell_visit(const double *__restrict__ r, const PairGrid &pg,
                                       const PairList &pl, int32_t i, uint32_t l, Fn &&fn) {
    const double ri[3] = {r[3 * i + 0], r[3 * i + 1], r[3 * i + 2]};
    const uint32_t o[3] = {l % 3u, (l / 3u) % 3u, l / 9u};
    uint32_t q[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        // one, two or three distinct cells per axis
        const uint32_t cnt = pg.nc[k] >= 3 ? 3u : pg.nc[k];
        if (o[k] >= cnt) return;
        const uint32_t c = pair_cell_coord(ri[k], pg.L[k], pg.nc[k]);
        q[k] = pg.nc[k] >= 3 ? (c + o[k] + pg.nc[k] - 1u) % pg.nc[k] : (c + o[k]) % pg.nc[k];
    }
    const double rc2 = pg.rc * pg.rc;
    const uint64_t cell = pair_cell(pg, q[0], q[1], q[2]);
    const uint32_t b = pair_bucket(cell, pg.T);
    auto meet = [&](int32_t j) {
        double d[3], rr = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            d[k] = ri[k] - r[3 * j + k];
            d[k] -= pg.L[k] * rint(d[k] / pg.L[k]);
            rr += d[k] * d[k];
        }
        if (rr > 0.0 && rr < rc2) fn(j, d, rr);
    };
    if constexpr (ORDERED) {
        uint32_t hops = 0;
        for (uint32_t next = pl.head[b] == kPairNone ? kPairNone : pl.first[b]; next != kPairNone && hops < pg.n; ++hops) {
            const int32_t j = int32_t(next);
            const PairLink e = pl.sorted[j];
            next = e.next;
            if (j != i && e.cell == cell) meet(j);
        }
    } else {
        // kPairBatch of the cell's particles per walk of the bucket's list (a
        // cell holds one or two as a rule)
        for (int64_t last = -1;;) {
            uint32_t id[kPairBatch];
#pragma unroll
            for (int k = 0; k < kPairBatch; ++k) id[k] = kPairNone;
            uint32_t found = 0;
            uint32_t hops = 0;
            for (uint32_t j = pl.head[b]; j != kPairNone && hops < pg.n; ++hops) {
                const PairLink e = pl.link[j];
                if (e.cell == cell && int64_t(j) > last) {
                    ++found;
                    uint32_t v = j;  // into the sorted batch, the largest drops out
#pragma unroll
                    for (int k = 0; k < kPairBatch; ++k) {
                        const uint32_t lo = min(id[k], v);
                        v = max(id[k], v);
                        id[k] = lo;
                    }
                }
                j = e.next;
            }
            if (__builtin_expect(pair_cluster(found, pg.n), 0)) {
                constexpr uint32_t kAhead = 8;
                for (uint32_t j0 = id[0]; j0 < pg.n; j0 += kAhead) {
                    uint32_t hit = 0;
#pragma unroll
                    for (uint32_t k = 0; k < kAhead; ++k)
                        hit |= uint32_t(pl.link[min(j0 + k, pg.n - 1)].cell == cell && j0 + k < pg.n) << k;
                    for (; hit; hit &= hit - 1) {
                        const int32_t j = int32_t(j0) + __builtin_ctz(hit);
                        if (j != i) meet(j);
                    }
                }
                break;
            }
#pragma unroll
            for (int k = 0; k < kPairBatch; ++k)
                if (id[k] != kPairNone && int32_t(id[k]) != i) meet(int32_t(id[k]));
            if (found <= uint32_t(kPairBatch)) break;
            last = id[kPairBatch - 1];
        }
    }
}

// Sum of v over the kPairLanes lanes of a group, in a fixed butterfly order
// (every lane receives it).
__device__ inline double pair_group_sum(double v) {
#pragma unroll
    for (int m = kPairLanes / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, kPairLanes);
    return v;
}

// F[i] = sum over neighbours of a_f (1 - |d|/r_c) d/|d|.
template <bool ORDERED>
__global__ __launch_bounds__(kPairBlock) void k_pair_force(const double *__restrict__ r, int32_t n,
                                                           PairGrid pg, PairList pl,
                                                           double *__restrict__ F) {
    const int32_t i = int32_t((blockIdx.x * kPairBlock + threadIdx.x) / kPairLanes);
    const uint32_t l = threadIdx.x % kPairLanes;
    if (i >= n) return;  // whole groups leave together
    double f[3] = {0.0, 0.0, 0.0};
    if (l < 27)
        pair_cell_visit<ORDERED>(r, pg, pl, i, l, [&](int32_t, const double (&d)[3], double rr) {
            const double dist = sqrt(rr);
            const double mag = pg.a * (1.0 - dist / pg.rc) / dist;
#pragma unroll
            for (int k = 0; k < 3; ++k) f[k] += mag * d[k];
        });
#pragma unroll
    for (int k = 0; k < 3; ++k) f[k] = pair_group_sum(f[k]);
    if (l == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) F[3 * i + k] = f[k];
}

// Adjoint: with Fb = dJ/dF_C of every particle, rbar[i] += sum over
// neighbours of Jac(d) (Fb[i] - Fb[j]), Jac(d) = a_f [(1/|d| - 1/r_c) I -
// d d^T / |d|^3] (the force of a pair is odd in d, its Jacobian even and
// symmetric).
template <bool ORDERED>
__global__ __launch_bounds__(kPairBlock) void k_adj_pair(const double *__restrict__ r, int32_t n,
                                                         PairGrid pg, PairList pl,
                                                         const double *__restrict__ Fb,
                                                         double *__restrict__ rbar) {
    const int32_t i = int32_t((blockIdx.x * kPairBlock + threadIdx.x) / kPairLanes);
    const uint32_t l = threadIdx.x % kPairLanes;
    if (i >= n) return;
    const double fi[3] = {Fb[3 * i + 0], Fb[3 * i + 1], Fb[3 * i + 2]};
    double g[3] = {0.0, 0.0, 0.0};
    if (l < 27)
        pair_cell_visit<ORDERED>(r, pg, pl, i, l, [&](int32_t j, const double (&d)[3], double rr) {
            const double dist = sqrt(rr);
            const double diag = pg.a * (1.0 / dist - 1.0 / pg.rc);
            const double outer = pg.a / (rr * dist);
            double w[3], dw = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                w[k] = fi[k] - Fb[3 * j + k];
                dw += d[k] * w[k];
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) g[k] += diag * w[k] - outer * d[k] * dw;
        });
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = pair_group_sum(g[k]);
    if (l == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) rbar[3 * i + k] += g[k];
}

}  // namespace lbmbp
