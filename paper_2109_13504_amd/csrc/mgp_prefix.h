// mgp_prefix.h -- the prefix-sum resamplers (multinomial, Algorithm 7;
// systematic, Algorithm 8) as the single-filter entry point and the SIR
// filter enqueue them: one job of R equal-size runs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mgp.h"
#include "mgp_internal.h"

namespace mgp {

constexpr int kMaxLevels = 8;  // levels of the 16-ary search tree: 16^8 = 2^32 > any n

// One resample of R equal-size filters (runs) at once, run r = blockIdx.y:
// a single filter is R = 1. Every run has its own scan region of the same
// layout (byte offsets below) at region + r region_ld.
struct PrefixJob {
    const float* w;           // run r's weights: w + r w_ld
    uint64_t w_ld;
    mgp_stats* stats;         // run r's validation and max: stats[r]
    // Where the finalize step has not run yet (a single filter): the
    // reduction's partials, over which every block of the first kernel does
    // it; block 0 writes stats and st_user. parts null: stats are there.
    const Partial* parts;
    uint32_t nparts;
    FinalizeArgs fin;
    mgp_stats* st_user;
    char* region;
    uint64_t region_ld;
    int32_t* anc;             // run r's ancestors: anc + r anc_ld (null: none)
    uint64_t anc_ld;
    const float* states;      // the particle copy x_bar_i = x_{a_i} of run r: rows of
    float* out;               // d floats at states / out + r rows_ld (states null: none)
    uint64_t rows_ld;
    uint32_t d, vec4;
    uint32_t n;
    uint32_t per, nsum;       // chunks per block of the first kernel, its blocks
    int log2n;                // ceil(log2 n)
    uint32_t key0, key1;
    uint32_t stream0;         // run r draws from stream stream0 + r
    uint64_t o_hdr, o_sum;
    uint64_t o_level[kMaxLevels + 1];  // level k (1..top) of the tree
    uint32_t count[kMaxLevels + 1];    // its entries, padded to a multiple of the fan-out
    uint32_t top_span;                 // count[top] rounded up to a power of two
    int top;                           // the first level of at most kTopMax entries
    uint32_t nsys;                     // blocks of the systematic search
    uint64_t o_start;                  // the group each of them starts in, and the last one's end
};

// Fills the region layout and n, per, nsum, log2n of J for runs of n
// particles; returns the bytes of one run's region.
uint64_t prefix_region(uint32_t n, PrefixJob* J);

// Enqueues the scan and search of a job: R runs, method MGP_MULTINOMIAL or
// MGP_SYSTEMATIC.
int enqueue_prefix(const PrefixJob& J, uint32_t R, int method, hipStream_t s);

}  // namespace mgp
