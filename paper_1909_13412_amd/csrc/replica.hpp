// Device-side tables of ensembles, and the block geometry of the two-step sweep.
#pragma once

#include <stdint.h>

#include "collide.hpp"

namespace lbmbp {

// The blocks of a two-step sweep: tiles of tx x ty nodes in (x, y), lz planes
// deep (the last ones may be smaller).
struct TwoStepTiles {
    uint32_t tx, ty, lz;
    uint32_t ntx, nty, nslab;  // ceil(n / extent)
};

// ---------------------------------------------------------------------------
// Ensembles of independent boxes (replicas) of different sizes, stepped
// together: one stream-collide launch covers every replica's nodes (a block
// never straddles two replicas) and one particle launch covers every
// particle.  Step-dependent values come from a device clock so that a
// captured graph of several steps can be replayed.
// ---------------------------------------------------------------------------
struct Replica {
    Grid g;
    uint64_t pop_off;              // first element of this box in the lattices
    uint64_t cell_off;             // first node in the node-force fields
    uint32_t mask_off;             // first word of its forcing flags
    uint32_t first_block[4];       // first stream-collide block, per launch shape
    TwoStepTiles two;              // its blocks of the two-step sweep
    uint32_t first_two;            // and the first of them
    uint32_t part_off, npart;      // its particles in the concatenated arrays
    uint32_t replica_id;           // Philox third counter word
    uint64_t seed;                 // Philox key
    double omega;                  // 1 / tau
    double R;                      // particle radius
};

struct EnsClock {
    int64_t step;    // Philox first counter word
    int64_t vacf_t;  // VACF sample clock
};

}  // namespace lbmbp
