// mgp_batch_internal.h -- device-side records and host helpers of the
// batched kernels, shared by the batch plan and the serving executor.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "mgp.h"
#include "mgp_device.h"
#include "mgp_internal.h"

namespace mgp {

constexpr uint32_t kNoFilter = 0xFFFFFFFFu;
constexpr uint32_t kBatchMaxN = kWindowMaxN;
constexpr int kMaxXcd = 8;

// Whether a filter's windows have a tail: the reduction, or the SIR filter's
// stage 1, writes it with the weights in hand, so a B still to be found counts
// as many steps.
inline bool record_tail(uint32_t n, uint32_t B_user) { return has_tail(n, B_user ? B_user : ~0u); }

// Per-filter record in device memory (read with scalar loads).
struct FilterDev {
    const float* w;
    int32_t* anc;
    const float* states;
    float* out;
    mgp_stats* stats_user;
    Windows windows;     // Megopolis: the accept loop's weights
    float* copy;         // Megopolis, weights not readable in place: the copy (n + kSeam floats) the reduction makes
    float* seam;         // Megopolis, weights read in place: their seam (2 kSeam floats), else null
    float* tail;         // Megopolis, large odd sizes: the weights once more (n + kSeam floats), on behind either
    uint32_t* offsets;   // Megopolis: b_max entries, else null
    double eps;
    uint32_t n;
    uint32_t B_user;
    uint32_t b_max;
    uint32_t key0, key1;
    uint32_t stream_id;
    uint32_t part_base;  // first partial of this filter
    uint32_t nparts;
    uint32_t chunk;
    uint32_t n_w, n_part;
    uint32_t vec;        // the reduction may use float4 loads
    uint32_t rows4;      // the gather may use float4 rows
    uint32_t pad[3];

    // The Megopolis windows: w in place with its seam at `aux`, or a copy there
    // (w, n and B_user are set).
    void set_windows(bool in_place, float* aux)
    {
        const bool tailed = record_tail(n, B_user);
        copy = in_place ? nullptr : aux;
        // windows past n start on cache lines: the seam's middle, n, lies n mod 32 floats behind one
        seam = in_place ? aux + (tailed ? n % 32u : 0u) : nullptr;
        tail = !tailed ? nullptr : in_place ? seam + kSeam : copy + n;
        windows = in_place ? windows_in_place(w, seam, n) : windows_copy(copy);
    }
};

// Floats of a filter's window region: the seam or copy, and the tail.
inline size_t window_floats(bool in_place, uint32_t n, uint32_t B_user)
{
    const size_t tail = record_tail(n, B_user) ? (size_t)n + (in_place ? 32u : 0u) : 0u;
    return tail + (in_place ? 2u * (size_t)kSeam : (size_t)n + kSeam);
}

// A block of the batched reduction: chunk c of filter f, or (kEndsTile) the
// ends of a Megopolis filter's windows, which run beside its chunks then
// instead of after one of them.
struct RTile {
    uint32_t f, c;
};
constexpr uint32_t kEndsTile = 0xFFFFFFFFu;

struct LTile {
    uint32_t f, start;
};

struct LoopShape {
    int bt, ppt, sched;
};

// Tile table of the accept loop for one launch shape (host side): filters
// placed on `nxcd` XCDs by longest-processing-time first on cost[f], tiles of
// the costlier filters first inside each XCD. Schedule 1 interleaves the XCD
// lists so that block b runs on XCD b mod nxcd (empty slots are kNoFilter);
// schedule 2 concatenates them and fills qoff[0..nxcd].
void build_tile_table(const std::vector<uint32_t>& n, const std::vector<double>& cost, const LoopShape& sh, int nxcd,
                      std::vector<LTile>& table, uint32_t* qoff);

// Enqueues one batched run: the segmented reduction, one finalize block per
// filter, and the accept loop with the fused gather. With n_rt == 0 the
// reduction is skipped: the producer of the weights has already written
// every filter's partials (and, for Megopolis, its seam).
int enqueue_batch(int variant, const LoopShape& sh, const FilterDev* d_fd, uint32_t count, const RTile* d_rt,
                  uint32_t n_rt, Partial* d_parts, mgp_stats* d_stats, const LTile* d_lt, uint32_t grid,
                  const uint32_t* d_qoff, uint32_t* d_qcount, uint32_t nxcd, uint32_t d, hipStream_t s);

// The finalize step alone (one block per filter: the stats record, B, and
// for Megopolis the offsets) over partials already written.
int enqueue_batch_finalize(const FilterDev* d_fd, uint32_t count, Partial* d_parts, mgp_stats* d_stats,
                           uint32_t* d_qcount, hipStream_t s);

bool batch_shape_supported(int variant, const LoopShape& sh);

}  // namespace mgp
