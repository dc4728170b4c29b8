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
};

struct alignas(16) PairLink {
    uint64_t cell;    // the particle's cell
    uint32_t next;    // next particle of its bucket or kPairNone
    uint32_t bucket;
};

// The cell list: the particles of every bucket, linked.
struct PairList {
    PairLink *link;  // [n]
    uint32_t *head;  // [T] first particle or kPairNone (all none between builds)
};

}  // namespace lbmbp
