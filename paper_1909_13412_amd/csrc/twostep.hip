// Instantiations of the two-step sweep and of the particle update ahead of it.
#include "twostep_launch.hpp"

#include "lbmbp.h"

namespace lbmbp {

template <class C, bool FORCED, bool NTS>
static void launch_two_steps_as(const TwoStepArgs &a) {
    using T = typename C::T;
    using R = typename C::R;
    using S = TwoStepShape<T>;
    const dim3 grid(a.tl.ntx * a.tl.nty * a.tl.nslab), block(two_step_threads(a.tl));
    hipLaunchKernelGGL((k_two_steps<C, FORCED, NTS, S::kNodes, S::kBuffers, S::kEarly>), grid, block, 0, a.stream,
                       static_cast<const T *>(a.A), static_cast<T *>(a.B), a.g, R(a.omega), R(a.enc_s), R(a.dec_s),
                       a.f0, a.f1, R(a.body[0]), R(a.body[1]), R(a.body[2]), a.tl, kOrderXcdSlabs);
}

template <class C>
void launch_two_steps(const TwoStepArgs &a) {
    if (a.forced)
        a.nts ? launch_two_steps_as<C, true, true>(a) : launch_two_steps_as<C, true, false>(a);
    else
        a.nts ? launch_two_steps_as<C, false, true>(a) : launch_two_steps_as<C, false, false>(a);
}

template <class C, int N>
static void launch_ahead_as(const TwoStepArgs &a, const ParticleArgs &pa) {
    using T = typename C::T;
    using R = typename C::R;
    const dim3 grid(unsigned((pa.n + kAheadParticles - 1) / kAheadParticles));
    hipLaunchKernelGGL((k_particle_ahead<C, N>), grid, dim3(kAheadBlock), 0, a.stream, static_cast<const T *>(a.A), a.g,
                       R(a.omega), R(a.enc_s), R(a.dec_s), R(a.body[0]), R(a.body[1]), R(a.body[2]), pa, a.f0, a.f1);
}

template <class C>
void launch_particle_ahead(const TwoStepArgs &a, const ParticleArgs &pa) {
    if (pa.friction == LBM_FRICTION_STOKESLET_2DX || pa.friction == LBM_FRICTION_STOKESLET_CUBE)
        launch_ahead_as<C, 5>(a, pa);
    else
        launch_ahead_as<C, 4>(a, pa);
}

#define LBM_TWO_STEP(CODEC, VEL)                                       \
    template void launch_two_steps<Cfg<CODEC, VEL>>(const TwoStepArgs &); \
    template void launch_particle_ahead<Cfg<CODEC, VEL>>(const TwoStepArgs &, const ParticleArgs &);
LBM_TWO_STEP(CodecF64, D3Q19)
LBM_TWO_STEP(CodecF32, D3Q19)
LBM_TWO_STEP(CodecBF16, D3Q19)
LBM_TWO_STEP(CodecF16, D3Q19)
LBM_TWO_STEP(CodecF64, D3Q15)
LBM_TWO_STEP(CodecF32, D3Q15)
LBM_TWO_STEP(CodecBF16, D3Q15)
LBM_TWO_STEP(CodecF16, D3Q15)
#undef LBM_TWO_STEP

}  // namespace lbmbp
