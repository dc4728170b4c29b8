// Two lattice steps in one sweep: the populations of step n are read once, the
// post-collision values of step n stay in LDS, and those of step n + 1 are
// written.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "codec.hpp"
#include "collide.hpp"
#include "replica.hpp"
#include "velocities.hpp"

namespace lbmbp {

// Nodes of a padded tile (lanes of a block and LDS nodes) at most, LDS buffers,
// and whether the loads of the next plane go out before the first step's
// arithmetic.
template <class T>
struct TwoStepShape {
    static constexpr int kNodes = sizeof(T) == 8 ? 704 : 832;
    static constexpr int kBuffers = sizeof(T) == 8 ? 1 : 2;
    static constexpr bool kEarly = sizeof(T) != 8;
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
template <class C, bool FORCED, bool NTS, int NMAX, int BUF, bool EARLY>
__device__ inline void two_steps_block(const typename C::T *__restrict__ A, typename C::T *__restrict__ B,
                                       const Grid &g, typename C::R omega, typename C::R enc_s,
                                       typename C::R dec_s, const ForceField &f0, const ForceField &f1,
                                       typename C::R Gx, typename C::R Gy, typename C::R Gz, uint32_t x0,
                                       uint32_t y0, uint32_t z0, uint32_t w, uint32_t h, uint32_t d,
                                       typename C::T (&post)[BUF][C::V::Q][NMAX]) {
#pragma clang fp contract(on)  // as node_relax
    using T = typename C::T;
    using R = typename C::R;
    using V = typename C::V;
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

    // raw populations and flag words of the first step at plane zp, the flag
    // word of the second step at the plane below
    T raw[V::Q];
    uint32_t word1 = 0, word2 = 0;
    auto load = [&](uint32_t zp) {
        const uint32_t zs[3] = {up(zp), zp, down(zp)};
        static_for<0, V::Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            const char *base = reinterpret_cast<const char *>(A) +
                               (uint64_t(zs[V::ez[a] + 1]) * plane + uint64_t(uint32_t(a) * popb));
            uint32_t off = yo[V::ey[a] + 1] + xo[V::ex[a] + 1];
            asm("" : "+v"(off));
            raw[a] = *reinterpret_cast<const T *>(base + off);
        });
        if constexpr (FORCED) {
            word1 = f0.mask[(zp * nxy + cell1) >> 5];
            word2 = f1.mask[(zs[2] * nxy + cell2) >> 5];
        }
    };
    const bool body = Gx != R(0) || Gy != R(0) || Gz != R(0);
    // relaxation at a node of linear index cell with flag bit `flag`
    auto relax = [&](const R (&gv)[V::Q], bool flag, uint32_t cell, const ForceField &ff, auto &&put) {
        const NodeMoments<C> m = node_moments<C>(gv);
        if (body || (FORCED && __any(flag))) {
            R Fx = Gx, Fy = Gy, Fz = Gz;
            if constexpr (FORCED) {
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
    // first step at plane zp; w2: the flag word of the second step below it
    auto first_step = [&](uint32_t &w2) {
        R gv[V::Q];
        static_for<0, V::Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            gv[a] = C::dec(EARLY ? held_copy(raw[a]) : raw[a], dec_s);
        });
        const uint32_t w1 = held_copy(word1);
        w2 = held_copy(word2);
        if constexpr (EARLY) load(up(zp));
        const uint32_t cell = zp * nxy + cell1;
        relax(gv, (w1 >> (cell & 31)) & 1u, cell, f0, [&](int a, R gn) { post[b][a][lds1] = C::enc(gn, enc_s); });
        __syncthreads();
        zp = up(zp);
        if constexpr (!EARLY) load(zp);
    };
    auto flip = [&]() {
        if constexpr (BUF == 2)
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

    load(zp);
    for (uint32_t k = 0; k < 2; ++k) {
        uint32_t w2;
        first_step(w2);
        if (second) shift();
        flip();
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the loop's waits then count its own accesses only
    if (second) {
        for (uint32_t k = 0; k < d; ++k) {
            uint32_t w2;
            first_step(w2);
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
            relax(gv, (w2 >> (cell & 31)) & 1u, cell, f1, [&](int a, R gn) {
                uint32_t off = own;
                asm("" : "+v"(off));
                T *p = reinterpret_cast<T *>(row + uint64_t(uint32_t(a) * popb) + off);
                if constexpr (NTS)
                    __builtin_nontemporal_store(C::enc(gn, enc_s), p);
                else
                    *p = C::enc(gn, enc_s);
            });
            flip();
        }
    } else {
        for (uint32_t k = 0; k < d; ++k) {
            uint32_t w2;
            first_step(w2);
            flip();
        }
    }
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

template <class C, bool FORCED, bool NTS, int NMAX, int BUF, bool EARLY>
__global__ __launch_bounds__(NMAX) void k_two_steps(
    const typename C::T *__restrict__ A, typename C::T *__restrict__ B, Grid g, typename C::R omega,
    typename C::R enc_s, typename C::R dec_s, ForceField f0, ForceField f1, typename C::R Gx,
    typename C::R Gy, typename C::R Gz, TwoStepTiles tl, uint32_t order) {
    __shared__ typename C::T post[BUF][C::V::Q][NMAX];
    const TwoStepBlock t(tl, g, sweep_block(order));
    two_steps_block<C, FORCED, NTS, NMAX, BUF, EARLY>(A, B, g, omega, enc_s, dec_s, f0, f1, Gx, Gy, Gz, t.x0, t.y0,
                                                      t.z0, t.w, t.h, t.d, post);
}

// Every box of an ensemble (block -> box table); advances the device clock by
// the two steps.
template <class C, bool NTS, int NMAX, int BUF, bool EARLY>
__global__ __launch_bounds__(NMAX) void k_ens_two_steps(
    const typename C::T *__restrict__ A, typename C::T *__restrict__ B, const Replica *__restrict__ reps,
    const uint16_t *__restrict__ blk_rep, ForceField f0, ForceField f1, typename C::R enc_s,
    typename C::R dec_s, EnsClock *clock, int vacf_on) {
    using R = typename C::R;
    __shared__ typename C::T post[BUF][C::V::Q][NMAX];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // the steps' last reader of the clock has finished (previous kernel)
        clock->step += 2;
        if (vacf_on) clock->vacf_t += 2;
    }
    const Replica &rp = reps[blk_rep[blockIdx.x]];
    const Grid g = rp.g;
    const TwoStepBlock t(rp.two, g, blockIdx.x - rp.first_two);
    two_steps_block<C, true, NTS, NMAX, BUF, EARLY>(A + rp.pop_off, B + rp.pop_off, g, R(rp.omega), enc_s, dec_s,
                                                    f0.box(rp.cell_off, rp.mask_off), f1.box(rp.cell_off, rp.mask_off),
                                                    R(0), R(0), R(0), t.x0, t.y0, t.z0, t.w, t.h, t.d, post);
}

}  // namespace lbmbp
