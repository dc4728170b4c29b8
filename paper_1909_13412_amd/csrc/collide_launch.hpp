// Host launch of the stream-collide in every configuration (collide.hpp).  The
// launches are instantiated per storage in collide_<storage>.hip, translation
// units of their own.
#pragma once

#include <hip/hip_runtime.h>

#include "collide.hpp"

namespace lbmbp {

struct CollideArgs {
    const void *A;
    void *B;
    Grid g;
    double omega, enc_s, dec_s, body[3];
    ForceField ff;
    double *mom;      // per-wavefront moment sums (nullptr: none)
    int shape, order; // launch configuration and block order
    unsigned grid;    // blocks
    size_t dyn;       // LDS reserved for the residency cap
    hipStream_t stream;
};

template <class C, bool FORCED>
void launch_stream_collide(const CollideArgs &a);

// Launch configuration k of the stream-collide: CALL(nodes per lane, block,
// non-temporal stores, row-aligned mapping).  Ensembles take k < 8 only.
#define LBM_CONFIG_SWITCH(k, CALL)                  \
    switch (k) {                                    \
        case 1: CALL(1, 256, false, false); break;  \
        case 2: CALL(2, 512, false, false); break;  \
        case 3: CALL(2, 256, false, false); break;  \
        case 4: CALL(1, 512, true, false); break;   \
        case 5: CALL(1, 256, true, false); break;   \
        case 6: CALL(2, 512, true, false); break;   \
        case 7: CALL(2, 256, true, false); break;   \
        case 8: CALL(1, 256, false, true); break;   \
        case 9: CALL(1, 256, true, true); break;    \
        default: CALL(1, 512, false, false); break; \
    }


// Addressing of the sweep (kAddr* in collide.hpp).  The row-aligned mapping
// always addresses by wavefront rows.  The flat mapping does so for 16-bit
// storage when rows are whole wavefronts: there the per-lane index arithmetic
// competes with the collision for the vector unit (FP16 step 1.8%, BF16 0.4%
// faster by rows, measured A/B on one device).  FP32 and FP64 sweeps are
// memory-bound, and per-lane indices measured as fast or faster (FP32 step
// 0.9%: its sum-carrying launches run longer by rows); those are in 32 bits
// unless the lattice holds 2^32 or more elements (Q nx ny nz; boxes beyond
// about 226M nodes).
template <class C>
int sweep_addr(const Grid &g, bool row_mapping) {
    if (row_mapping || (sizeof(typename C::T) == 2 && g.nx % 64 == 0)) return kAddrRow;
    return uint64_t(C::V::Q) * g.ncell >= (uint64_t(1) << 32) ? kAddrLane64 : kAddrLane32;
}

}  // namespace lbmbp
