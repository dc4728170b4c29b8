// Two lattice steps in one sweep: the populations of step n are read once, the
// post-collision values of step n stay in LDS, and those of step n + 1 are
// written, in the bits of two single steps (the same node_moments and
// node_relax, the values in between encoded and decoded as in memory).
//
// A single step is bound by HBM: it reads and writes every population (152 B a
// node in FP32).  Here a block takes a tile in x and y with one halo node
// around it and marches in z: the first step of plane p from registers into
// LDS, then the second step of plane p - 1, which pulls its e_z < 0 populations
// from plane p and has kept the others in registers.  Half the bytes per step
// are left, plus the halo, whose lines are mostly in the L2 of the XCD that
// holds the neighbouring tiles (blocks in XCD slabs).  Two steps, ms, against
// two single ones at 256^3: FP32 0.484 / 0.85, BF16 0.31 / 0.41, FP64 0.96 /
// 1.73; FP32 128^3 0.067 / 0.110.  The halo costs 7 to 12% of the lattice in reads
// from memory; with it FP32 and FP64 move 5.6 TB/s (a copy 5.2, the single-step
// sweep 6.4), the address unit busy 70% of the time; without its loads the FP32
// sweep takes 0.23 ms, without its stores 0.37.  16-bit storage moves 3.9 TB/s, the
// vector unit busy 65-70% and the address unit 62% of the time, on 11 to 13
// wavefronts a compute unit; D3Q19 spills 23 to 25 registers.
// Slower were: planes brought to LDS by direct loads (FP32 0.548, BF16 0.395),
// two small blocks per compute unit, non-temporal loads (FP32 0.726, BF16 0.463:
// the halo's lines come twice), a march in alternate directions so that a
// sweep first reads what the last one wrote last (under 1%).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "codec.hpp"
#include "collide.hpp"
#include "replica.hpp"
#include "velocities.hpp"

namespace lbmbp {

// How a storage's sweep is built.  A block is one lane per node of the padded
// tile and one block fills a compute unit: 13 wavefronts leave 128 registers
// each, FP64 takes 11 for its 168, and the post-collision planes take 126 KB of
// LDS in FP32.
//   kBuffers: LDS planes; two need one barrier per plane, one needs two (FP64,
//     where two planes would not fit);
//   kPlanes: planes of populations in flight in registers, loaded that many
//     ahead; 0 loads the next one between the two steps (FP64, for the
//     registers).  A second plane pays where a plane is short (16-bit, 64 x 8
//     tiles at 256^3: 0.324 -> 0.310 ms per sweep) and not where HBM is the
//     limit (FP32 0.484 -> 0.489);
//   kFront: loads sent off before the first step's arithmetic; the rest go one
//     at a time between the relaxed pairs.  All at once they fill the address
//     queue and every wavefront of the block stalls (BF16 0.382 -> 0.324 ms,
//     FP32 0.518 -> 0.484).
template <class T>
struct TwoStepShape {
    static constexpr int kNodes = sizeof(T) == 8 ? 704 : 832;
    static constexpr int kBuffers = sizeof(T) == 8 ? 1 : 2;
    static constexpr int kPlanes = sizeof(T) == 8 ? 0 : (sizeof(T) == 4 ? 1 : 2);
    static constexpr int kFront = sizeof(T) == 2 ? 10 : 6;
    static constexpr bool kForceAhead = sizeof(T) == 4;  // see two_steps_block
};
constexpr uint32_t two_step_nodes(size_t elem) {
    return elem == 8 ? TwoStepShape<double>::kNodes : TwoStepShape<float>::kNodes;
}

__host__ inline uint32_t two_step_threads(const TwoStepTiles &tl) { return ((tl.tx + 2) * (tl.ty + 2) + 63u) & ~63u; }

// A copy that stays a copy: the original's registers are free for the next
// load at once, which the compiler otherwise prevents by reading them in place.
__device__ inline float held_copy(float v) {
    float r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ inline uint32_t held_copy(uint32_t v) {
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ inline uint16_t held_copy(uint16_t v) { return v; }  // decoding moves it
__device__ inline double held_copy(double v) { return v; }

// One block: the nodes [x0, x0 + w) x [y0, y0 + h) x [z0, z0 + d).
// AHEAD: the node forces of a plane are loaded with its populations, from flag
// words loaded a plane before.  Loaded where they are needed they would hold up
// a wavefront, and with it its block, until the loads and stores sent off
// before them are done (4096 particles, FP32: ten steps at 128^3 775 -> 745 us,
// twenty at 256^3 5.80 -> 5.72 ms).  Only FP32 has the 18 registers; the ensembles' sweep,
// with its box table, would spill them (64 boxes 8.17 -> 8.26 ms per 16 steps).
template <class C, bool FORCED, bool NTS, bool AHEAD>
__device__ inline void two_steps_block(const typename C::T *__restrict__ A, typename C::T *__restrict__ B,
                                       const Grid &g, typename C::R omega, typename C::R enc_s,
                                       typename C::R dec_s, const ForceField &f0, const ForceField &f1,
                                       typename C::R Gx, typename C::R Gy, typename C::R Gz, uint32_t x0,
                                       uint32_t y0, uint32_t z0, uint32_t w, uint32_t h, uint32_t d,
                                       typename C::T (&post)[TwoStepShape<typename C::T>::kBuffers][C::V::Q][TwoStepShape<typename C::T>::kNodes]) {
#pragma clang fp contract(on)  // as node_relax
    using T = typename C::T;
    using R = typename C::R;
    using V = typename C::V;
    using S = TwoStepShape<T>;
    constexpr int D = S::kPlanes > 1 ? S::kPlanes : 1;  // sets of load registers
    static_assert(!AHEAD || D == 1, "one set of node-force registers");
    const uint32_t pw = w + 2;  // row pitch of the padded tile in LDS

    auto up = [&](uint32_t z) { return z + 1 == g.nz ? 0u : z + 1; };
    auto down = [&](uint32_t z) { return z == 0 ? g.nz - 1 : z - 1; };
    auto row_bytes = [&](uint32_t y) {
        return ((y & ~g.ymask) * V::Q + (y & g.ymask)) * g.chunk * uint32_t(sizeof(T));
    };
    const uint64_t plane = uint64_t(g.ny) * V::Q * g.chunk * sizeof(T);  // bytes
    const uint32_t popb = g.pstride * uint32_t(sizeof(T));
    const uint32_t nxy = g.nx * g.ny;

    // first step: lane -> node (x0 - 1 + ix, y0 - 1 + iy), one halo node
    // around the tile; lanes past the last node repeat it
    const uint32_t lds1 = min(threadIdx.x, pw * (h + 2) - 1);
    const uint32_t iy = lds1 / pw, ix = lds1 - iy * pw;
    uint32_t X = x0 + ix, Y = y0 + iy;  // node + 1
    X = X == 0 ? g.nx - 1 : (X > g.nx ? 0u : X - 1);
    Y = Y == 0 ? g.ny - 1 : (Y > g.ny ? 0u : Y - 1);
    const uint32_t yo[3] = {row_bytes(Y + 1 == g.ny ? 0u : Y + 1), row_bytes(Y), row_bytes(Y == 0 ? g.ny - 1 : Y - 1)};
    const uint32_t xo[3] = {(X + 1 == g.nx ? 0u : X + 1) * uint32_t(sizeof(T)), X * uint32_t(sizeof(T)),
                            (X == 0 ? g.nx - 1 : X - 1) * uint32_t(sizeof(T))};
    const uint32_t cell1 = Y * g.nx + X;

    // second step: lane -> tile node (x0 + jx, y0 + jy); lanes past the last
    // node of a wavefront that holds any repeat it
    const uint32_t i2 = min(threadIdx.x, w * h - 1);
    const uint32_t jy = i2 / w, jx = i2 - jy * w;
    const uint32_t y2 = y0 + jy;
    const uint32_t own = row_bytes(y2) + (x0 + jx) * uint32_t(sizeof(T));
    const uint32_t cell2 = y2 * g.nx + x0 + jx;
    const bool second = __builtin_amdgcn_readfirstlane(threadIdx.x) < w * h;  // wavefront-uniform
    const uint32_t from[3] = {(jy + 2) * pw + jx + 1, (jy + 1) * pw + jx + 1, jy * pw + jx + 1};  // rows y - e_y

    // raw populations and flag words of the first step at a plane, the flag
    // word of the second step at the plane below; set i of D
    T raw[D][V::Q];
    uint32_t word1[D] = {}, word2[D] = {};
    // AHEAD: the flag words of the plane after, the node forces at the
    // flagged nodes of the plane itself
    uint32_t ahead1 = 0, ahead2 = 0;
    int64_t force1[3] = {}, force2[3] = {};
    auto words_of = [&](uint32_t z, uint32_t zbelow, uint32_t &w1, uint32_t &w2) {
        w1 = f0.mask[(z * nxy + cell1) >> 5];
        w2 = f1.mask[(zbelow * nxy + cell2) >> 5];
    };
    auto force_at = [&](const ForceField &ff, uint32_t word, uint32_t cell, int64_t (&f)[3]) {
        if ((word >> (cell & 31)) & 1u)
            for (int k = 0; k < 3; ++k) f[k] = ff.f[3 * uint64_t(cell) + k];
    };
    const char *src[3];  // planes zp + 1, zp, zp - 1 of the plane being loaded
    auto load_from = [&](uint32_t zp, auto ic) {
        constexpr int i = decltype(ic)::value;
        const uint32_t zs[3] = {up(zp), zp, down(zp)};
        for (int k = 0; k < 3; ++k) src[k] = reinterpret_cast<const char *>(A) + uint64_t(zs[k]) * plane;
        if constexpr (FORCED && AHEAD) {
            word1[i] = ahead1;
            word2[i] = ahead2;
            words_of(zs[0], zp, ahead1, ahead2);
            force_at(f0, word1[i], zp * nxy + cell1, force1);
            force_at(f1, word2[i], zs[2] * nxy + cell2, force2);
        } else if constexpr (FORCED) {
            words_of(zp, zs[2], word1[i], word2[i]);
        }
    };
    auto load_pop = [&](auto ac, auto ic) {
        constexpr int a = decltype(ac)::value, i = decltype(ic)::value;
        uint32_t off = yo[V::ey[a] + 1] + xo[V::ex[a] + 1];
        asm("" : "+v"(off));  // a lane offset to a scalar base, not a 64-bit lane address
        raw[i][a] = *reinterpret_cast<const T *>(src[V::ez[a] + 1] + uint64_t(uint32_t(a) * popb) + off);
    };
    auto load = [&](uint32_t zp, auto ic) {
        load_from(zp, ic);
        static_for<0, V::Q>([&](auto ac) { load_pop(ac, ic); });
    };
    const bool body = Gx != R(0) || Gy != R(0) || Gz != R(0);
    // relaxation at a node of linear index cell with flag bit `flag`
    auto relax = [&](const R (&gv)[V::Q], bool flag, uint32_t cell, const ForceField &ff, const R (&fn)[3], auto &&put) {
        const NodeMoments<C> m = node_moments<C>(gv);
        if (body || (FORCED && __any(flag))) {
            R Fx = Gx, Fy = Gy, Fz = Gz;
            if constexpr (FORCED && AHEAD) {
                if (flag) {
                    Fx += fn[0];
                    Fy += fn[1];
                    Fz += fn[2];
                }
            } else if constexpr (FORCED) {
                if (flag) {
                    Fx += R(double(ff.f[3 * uint64_t(cell) + 0]) * kFixInv);
                    Fy += R(double(ff.f[3 * uint64_t(cell) + 1]) * kFixInv);
                    Fz += R(double(ff.f[3 * uint64_t(cell) + 2]) * kFixInv);
                }
            }
            node_relax<C, true>(gv, m, omega, Fx, Fy, Fz, put);
        } else {
            node_relax<C, false>(gv, m, omega, R(0), R(0), R(0), put);
        }
    };
    uint32_t zp = down(z0);  // plane of the first step
    uint32_t b = 0;          // LDS buffer it writes
    // first step at plane zp, held in set i; w2: the flag word of the second
    // step below it
    auto first_step = [&](uint32_t &w2, R (&fn2)[3], auto ic) {
        constexpr int i = decltype(ic)::value;
        R gv[V::Q];
        static_for<0, V::Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            gv[a] = C::dec(S::kPlanes > 0 ? held_copy(raw[i][a]) : raw[i][a], dec_s);
        });
        const uint32_t w1 = held_copy(word1[i]);
        w2 = held_copy(word2[i]);
        const uint32_t cell = zp * nxy + cell1;
        R fn1[3] = {};
        if constexpr (FORCED && AHEAD) {
            for (int k = 0; k < 3; ++k) {
                fn1[k] = R(double(force1[k]) * kFixInv);
                fn2[k] = R(double(force2[k]) * kFixInv);
            }
        }
        if constexpr (S::kPlanes > 0) {
            load_from(S::kPlanes > 1 ? up(up(zp)) : up(zp), ic);
            static_for<0, S::kFront>([&](auto ac) { load_pop(ac, ic); });
        }
        relax(gv, (w1 >> (cell & 31)) & 1u, cell, f0, fn1, [&](auto ac, R gn) {
            constexpr int a = decltype(ac)::value;
            post[b][a][lds1] = C::enc(gn, enc_s);
            if constexpr (S::kPlanes > 0 && a >= S::kFront) {
                load_pop(ac, ic);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        __syncthreads();
        zp = up(zp);
        if constexpr (S::kPlanes == 0) load(zp, ic);
    };
    auto flip = [&]() {
        if constexpr (S::kBuffers == 2)
            b ^= 1;
        else
            __syncthreads();
    };
    auto pulled = [&](auto ac) {
        constexpr int a = decltype(ac)::value;
        return post[b][a][int(from[V::ey[a] + 1]) - V::ex[a]];
    };

    T pend[V::Q];  // e_z = 0 and +1 of the next target plane
    T next[V::Q];  // e_z = +1 of the plane after
    static_for<0, V::Q>([&](auto ac) { pend[decltype(ac)::value] = next[decltype(ac)::value] = T(0); });
    auto shift = [&]() {
        static_for<0, V::Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            if constexpr (V::ez[a] == 0) pend[a] = pulled(ac);
            if constexpr (V::ez[a] > 0) {
                pend[a] = next[a];
                next[a] = pulled(ac);
            }
        });
    };

    using Set0 = std::integral_constant<int, 0>;
    using Set1 = std::integral_constant<int, D - 1>;
    if constexpr (FORCED && AHEAD) words_of(zp, down(zp), ahead1, ahead2);
    load(zp, Set0{});
    if constexpr (D == 2) load(up(zp), Set1{});
    // the planes below and at z0
    auto start = [&](auto ic) {
        uint32_t w2;
        R fn2[3] = {};
        first_step(w2, fn2, ic);
        if (second) shift();
        flip();
    };
    start(Set0{});
    start(Set1{});
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the loop's waits then count its own accesses only
    // first step one plane above the second step's
    auto both = [&](auto ic) {
        uint32_t w2;
        R fn2[3] = {};
        first_step(w2, fn2, ic);
        const uint32_t zt = down(down(zp));
        R gv[V::Q];
        static_for<0, V::Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            if constexpr (V::ez[a] < 0)
                gv[a] = C::dec(pulled(ac), dec_s);
            else
                gv[a] = C::dec(pend[a], dec_s);
        });
        shift();
        const uint32_t cell = zt * nxy + cell2;
        char *row = reinterpret_cast<char *>(B) + uint64_t(zt) * plane;
        relax(gv, (w2 >> (cell & 31)) & 1u, cell, f1, fn2, [&](auto ac, R gn) {
            constexpr int a = decltype(ac)::value;
            uint32_t off = own;
            asm("" : "+v"(off));
            T *p = reinterpret_cast<T *>(row + uint64_t(uint32_t(a) * popb) + off);
            if constexpr (NTS)
                __builtin_nontemporal_store(C::enc(gn, enc_s), p);
            else
                *p = C::enc(gn, enc_s);
        });
        flip();
    };
    // a wavefront past the tile's nodes has the first step only
    auto first_only = [&](auto ic) {
        uint32_t w2;
        R fn2[3] = {};
        first_step(w2, fn2, ic);
        flip();
    };
    // d planes, the D register sets in turn; each kind of wavefront has a loop
    // of its own, so that its waits know the stores in flight behind the loads
    auto march = [&](auto &&plane_of) {
        for (uint32_t left = d;;) {
            plane_of(Set0{});
            if (--left == 0) break;
            if constexpr (D == 2) {
                plane_of(Set1{});
                if (--left == 0) break;
            }
        }
    };
    if (second)
        march(both);
    else
        march(first_only);
}

// Block b of a box's sweep: tiles in x, then y, then slabs of planes.
struct TwoStepBlock {
    uint32_t x0, y0, z0, w, h, d;
    __device__ inline TwoStepBlock(const TwoStepTiles &tl, const Grid &g, uint32_t b) {
        const uint32_t per = tl.ntx * tl.nty;
        const uint32_t slab = b / per, tile = b - slab * per;
        const uint32_t by = tile / tl.ntx, bx = tile - by * tl.ntx;
        x0 = bx * tl.tx;
        y0 = by * tl.ty;
        z0 = slab * tl.lz;
        w = min(tl.tx, g.nx - x0);
        h = min(tl.ty, g.ny - y0);
        d = min(tl.lz, g.nz - z0);
    }
};

template <class C, bool FORCED, bool NTS>
__global__ __launch_bounds__(TwoStepShape<typename C::T>::kNodes) void k_two_steps(
    const typename C::T *__restrict__ A, typename C::T *__restrict__ B, Grid g, typename C::R omega,
    typename C::R enc_s, typename C::R dec_s, ForceField f0, ForceField f1, typename C::R Gx,
    typename C::R Gy, typename C::R Gz, TwoStepTiles tl, uint32_t order) {
    __shared__ typename C::T post[TwoStepShape<typename C::T>::kBuffers][C::V::Q][TwoStepShape<typename C::T>::kNodes];
    const TwoStepBlock t(tl, g, sweep_block(order));
    two_steps_block<C, FORCED, NTS, TwoStepShape<typename C::T>::kForceAhead>(A, B, g, omega, enc_s, dec_s, f0, f1, Gx, Gy, Gz, t.x0, t.y0, t.z0, t.w, t.h, t.d, post);
}

// Every box of an ensemble (block -> box table); advances the device clock by
// the two steps.
template <class C, bool NTS>
__global__ __launch_bounds__(TwoStepShape<typename C::T>::kNodes) void k_ens_two_steps(
    const typename C::T *__restrict__ A, typename C::T *__restrict__ B, const Replica *__restrict__ reps,
    const uint16_t *__restrict__ blk_rep, ForceField f0, ForceField f1, typename C::R enc_s,
    typename C::R dec_s, EnsClock *clock, int vacf_on) {
    using R = typename C::R;
    __shared__ typename C::T post[TwoStepShape<typename C::T>::kBuffers][C::V::Q][TwoStepShape<typename C::T>::kNodes];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // the steps' last reader of the clock has finished (previous kernel)
        clock->step += 2;
        if (vacf_on) clock->vacf_t += 2;
    }
    const Replica &rp = reps[blk_rep[blockIdx.x]];
    const Grid g = rp.g;
    const TwoStepBlock t(rp.two, g, blockIdx.x - rp.first_two);
    two_steps_block<C, true, NTS, false>(A + rp.pop_off, B + rp.pop_off, g, R(rp.omega), enc_s, dec_s,
                                  f0.box(rp.cell_off, rp.mask_off), f1.box(rp.cell_off, rp.mask_off),
                                  R(0), R(0), R(0), t.x0, t.y0, t.z0, t.w, t.h, t.d, post);
}

}  // namespace lbmbp
