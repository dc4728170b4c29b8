// Host launches of the two-step sweep (twostep.hpp) and of the particle update
// one step ahead of it (particle.hpp).  They are instantiated in twostep.hip,
// a translation unit of its own.
#pragma once

#include <hip/hip_runtime.h>

#include "collide.hpp"
#include "particle.hpp"
#include "twostep.hpp"

namespace lbmbp {

struct TwoStepArgs {
    const void *A;
    void *B;
    Grid g;
    double omega, enc_s, dec_s, body[3];
    ForceField f0, f1;  // node forces of the first and the second step
    TwoStepTiles tl;
    bool forced;  // particles attached
    bool nts;     // non-temporal stores
    hipStream_t stream;
};

template <class C>
void launch_two_steps(const TwoStepArgs &a);

// pa: the second step's update, whose node forces go to a.f1.
template <class C>
void launch_particle_ahead(const TwoStepArgs &a, const ParticleArgs &pa);

// The same over an ensemble's boxes.
struct EnsTwoStepArgs {
    const void *A;
    void *B;
    const Replica *reps;
    const uint16_t *blk_rep, *part_rep;
    unsigned blocks, threads;
    double enc_s, dec_s;
    ForceField f0, f1;
    EnsClock *clock;
    int vacf_on;
    bool nts;
    hipStream_t stream;
};

template <class C>
void launch_ens_two_steps(const EnsTwoStepArgs &a);
template <class C>
void launch_ens_particle_ahead(const EnsTwoStepArgs &a, const ParticleArgs &pa);

}  // namespace lbmbp
