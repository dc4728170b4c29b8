// The cell list of the pair repulsion (pairs.hpp).
#pragma once

#include <stdint.h>

namespace lbmbp {

constexpr int kPairMax = 65536;  // particles at most
constexpr int kPairBlock = 256;
constexpr uint32_t kPairNone = 0xFFFFFFFFu;

struct PairGrid {
    uint32_t nc[3];  // cells per axis
    uint32_t T;      // buckets (power of two)
    uint32_t n;      // particles: no list is longer
    double L[3];     // box edges
    double a, rc;    // a_f and the cutoff
    uint32_t ordered;  // k_pair_order runs (pair_list_ordered)
};

struct alignas(16) PairLink {
    uint64_t cell;    // the particle's cell
    uint32_t next;    // next particle of its bucket or kPairNone
    uint32_t bucket;
};

// The cell list: the particles of every bucket, linked as they came and, where
// the lists are long, in ascending index.
struct PairList {
    PairLink *link;    // [n] as they came
    PairLink *sorted;  // [n] ascending
    uint32_t *head;    // [T] first of `link` or kPairNone (all none between builds)
    uint32_t *first;   // [T] first of `sorted` where head is one
};

// Particles that a walk of a list takes at a time.
constexpr int kPairBatch = 4;

// Whether the lists are put into ascending order before they are walked: a pass
// of 4 us, and every cell is then one walk instead of one for each kPairBatch
// of its particles.  Us per step, as they came / in order, 4096 particles in
// 32^3: 1 per cell 35.5 / 38.6, 8 per cell 57.3 / 50.1, 64 per cell 533 / 129, 512
// per cell 12895 / 536; 65536 in 128^3: 2 per cell 275 / 284, 16 per cell 854 / 500.
inline bool pair_list_ordered(uint64_t particles, uint64_t cells) { return particles > kPairBatch * cells; }

}  // namespace lbmbp
