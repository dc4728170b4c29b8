// Definitions behind collide_launch.hpp, included by collide_<storage>.hip.
#pragma once

#include "collide_launch.hpp"

namespace lbmbp {

template <class C, bool FORCED, bool MOMENTS, int CPT, int BS, bool NTS, bool ROW, int ADDR>
static void launch_collide_addr(const CollideArgs &a) {
    using T = typename C::T;
    using R = typename C::R;
    hipLaunchKernelGGL((k_stream_collide<C, FORCED, MOMENTS, CPT, BS, NTS, ROW, ADDR>), dim3(a.grid), dim3(BS), a.dyn,
                       a.stream, static_cast<const T *>(a.A), static_cast<T *>(a.B), a.g, R(a.omega), R(a.enc_s),
                       R(a.dec_s), a.ff, R(a.body[0]), R(a.body[1]), R(a.body[2]), a.mom, uint32_t(a.order));
}

template <class C, bool FORCED, bool MOMENTS, int CPT, int BS, bool NTS, bool ROW>
static void launch_collide_shape(const CollideArgs &a) {
    if constexpr (ROW) {
        launch_collide_addr<C, FORCED, MOMENTS, CPT, BS, NTS, ROW, kAddrRow>(a);
    } else {
        const int addr = sweep_addr<C>(a.g, ROW);
        if constexpr (sizeof(typename C::T) == 2)
            if (addr == kAddrRow) return launch_collide_addr<C, FORCED, MOMENTS, CPT, BS, NTS, ROW, kAddrRow>(a);
        if (addr == kAddrLane64)
            launch_collide_addr<C, FORCED, MOMENTS, CPT, BS, NTS, ROW, kAddrLane64>(a);
        else
            launch_collide_addr<C, FORCED, MOMENTS, CPT, BS, NTS, ROW, kAddrLane32>(a);
    }
}

template <class C, bool FORCED>
void launch_stream_collide(const CollideArgs &a) {
#define LBM_SHAPE(CPT, BS, NTS, ROW)                                        \
    do {                                                                    \
        if (a.mom)                                                          \
            launch_collide_shape<C, FORCED, true, CPT, BS, NTS, ROW>(a);    \
        else                                                                \
            launch_collide_shape<C, FORCED, false, CPT, BS, NTS, ROW>(a);   \
    } while (0)
    LBM_CONFIG_SWITCH(a.shape, LBM_SHAPE)
#undef LBM_SHAPE
}

}  // namespace lbmbp
