// Instantiations of the two-step sweep and of the particle update ahead of it.
#include "twostep_launch.hpp"

#include "lbmbp.h"

namespace lbmbp {

template <class C, bool FORCED, bool NTS>
static void launch_two_steps_as(const TwoStepArgs &a) {
    using T = typename C::T;
    using R = typename C::R;
    const dim3 grid(a.tl.ntx * a.tl.nty * a.tl.nslab), block(two_step_threads(a.tl));
    hipLaunchKernelGGL((k_two_steps<C, FORCED, NTS>), grid, block, 0, a.stream,
                       static_cast<const T *>(a.A), static_cast<T *>(a.B), a.g, R(a.omega), R(a.enc_s), R(a.dec_s),
                       a.f0, a.f1, R(a.body[0]), R(a.body[1]), R(a.body[2]), a.tl, kOrderXcdSlabs);
}

template <class C>
void launch_two_steps(const TwoStepArgs &a) {
    // FP64 reads the (empty) forcing flags of a box without particles too: the
    // kernel without them needs scratch memory (192^3, ms per sweep: 0.568
    // against 0.449)
    if constexpr (sizeof(typename C::T) < 8)
        if (!a.forced)
            return a.nts ? launch_two_steps_as<C, false, true>(a) : launch_two_steps_as<C, false, false>(a);
    a.nts ? launch_two_steps_as<C, true, true>(a) : launch_two_steps_as<C, true, false>(a);
}

template <class C, int N>
static void launch_ahead_as(const TwoStepArgs &a, const ParticleArgs &pa) {
    using T = typename C::T;
    using R = typename C::R;
    const dim3 grid(unsigned((pa.n + AheadShape<N>::kParticles - 1) / AheadShape<N>::kParticles));
    hipLaunchKernelGGL((k_particle_ahead<C, N>), grid, dim3(AheadShape<N>::kBlock), 0, a.stream, static_cast<const T *>(a.A), a.g,
                       R(a.omega), R(a.enc_s), R(a.dec_s), R(a.body[0]), R(a.body[1]), R(a.body[2]), pa, a.f0, a.f1);
}

template <class C>
void launch_particle_ahead(const TwoStepArgs &a, const ParticleArgs &pa) {
    if (pa.friction == LBM_FRICTION_STOKESLET_2DX || pa.friction == LBM_FRICTION_STOKESLET_CUBE)
        launch_ahead_as<C, 5>(a, pa);
    else
        launch_ahead_as<C, 4>(a, pa);
}

template <class C, bool NTS>
static void launch_ens_two_steps_as(const EnsTwoStepArgs &a) {
    using T = typename C::T;
    using R = typename C::R;
    hipLaunchKernelGGL((k_ens_two_steps<C, NTS>), dim3(a.blocks), dim3(a.threads), 0,
                       a.stream, static_cast<const T *>(a.A), static_cast<T *>(a.B), a.reps, a.blk_rep, a.f0, a.f1,
                       R(a.enc_s), R(a.dec_s), a.clock, a.vacf_on);
}

template <class C>
void launch_ens_two_steps(const EnsTwoStepArgs &a) {
    a.nts ? launch_ens_two_steps_as<C, true>(a) : launch_ens_two_steps_as<C, false>(a);
}

template <class C, int N>
static void launch_ens_ahead_as(const EnsTwoStepArgs &a, const ParticleArgs &pa) {
    using T = typename C::T;
    using R = typename C::R;
    const dim3 grid(unsigned((pa.n + AheadShape<N>::kParticles - 1) / AheadShape<N>::kParticles));
    hipLaunchKernelGGL((k_ens_particle_ahead<C, N>), grid, dim3(AheadShape<N>::kBlock), 0, a.stream, static_cast<const T *>(a.A),
                       a.reps, a.part_rep, R(a.enc_s), R(a.dec_s), pa, a.clock, a.f0, a.f1);
}

template <class C>
void launch_ens_particle_ahead(const EnsTwoStepArgs &a, const ParticleArgs &pa) {
    if (pa.friction == LBM_FRICTION_STOKESLET_2DX || pa.friction == LBM_FRICTION_STOKESLET_CUBE)
        launch_ens_ahead_as<C, 5>(a, pa);
    else
        launch_ens_ahead_as<C, 4>(a, pa);
}

#define LBM_ENS_TWO_STEP(CODEC)                                                   \
    template void launch_ens_two_steps<Cfg<CODEC, D3Q19>>(const EnsTwoStepArgs &); \
    template void launch_ens_particle_ahead<Cfg<CODEC, D3Q19>>(const EnsTwoStepArgs &, const ParticleArgs &);
LBM_ENS_TWO_STEP(CodecF64)
LBM_ENS_TWO_STEP(CodecF32)
LBM_ENS_TWO_STEP(CodecBF16)
LBM_ENS_TWO_STEP(CodecF16)
#undef LBM_ENS_TWO_STEP

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
