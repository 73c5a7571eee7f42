// mgp_internal.h -- host/device shared definitions of libmgp (not part of the
// public ABI): workspace layout, launch shapes, and the host helpers the
// single-filter, batched and serving paths share.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "mgp.h"
#include "mgp_device.h"

namespace mgp {

constexpr int kVersion = 100;               // 0.1.0
constexpr uint32_t kReduceThreads = 256;    // reduce / finalize block
constexpr uint32_t kLoopThreads = 256;      // accept-loop block (4 waves of 64)
constexpr uint32_t kMaxPartials = 4096;     // reduce blocks per filter, at most
constexpr uint32_t kReduceChunk = 2048;     // weights per reduce block (before the kMaxPartials cap)
constexpr uint32_t kDefaultBMax = 65536;
constexpr uint32_t kBMaxLimit = 1u << 24;

// Workspace layout of a single-filter call (byte offsets, 256-aligned):
//   [stats: mgp_stats][log(eps): f64]
//   [partials: kMaxPartials x Partial]
//   [offsets: b_max x u32]
//   [copy: (2n + 2048) x f32 reserved, Megopolis with n <= kWindowMaxN only.
//    copy[k] = w[k mod n], k < n + kSeam (2n + kSeam with a tail, which the
//    finalize launch writes once B is known). The reduction makes it (kLayoutCopy)
//    or, for a loop that reads the weights in place (kLayoutInPlace), its last
//    2 kSeam entries, the seam; that loop then writes the others, for a prepared
//    loop that may follow, which always reads the copy.]
constexpr size_t kWsStatsOffset = 0;
constexpr size_t kWsLogEpsOffset = 128;
constexpr size_t kWsPartialsOffset = 256;
constexpr uint32_t kWindowReserve = 2048;  // of the reserved 2n + 2048
static_assert(kWindowReserve >= kSeam, "the copy must fit the reserved region");
constexpr int kMegopolisPPT = 4;  // particles per thread of the large Megopolis loop

struct Partial {
    double w_sum;
    float w_max;
    uint32_t bad;
};
static_assert(sizeof(Partial) == 16, "Partial is 16 bytes");

constexpr size_t kWsOffsetsOffset = kWsPartialsOffset + (size_t)kMaxPartials * sizeof(Partial);

struct FinalizeArgs {
    double eps;
    const double* log_eps = nullptr;  // log(eps) if an earlier launch of the call computed it, else null
    uint32_t n;
    uint32_t B_user;
    uint32_t b_max;
    uint32_t make_offsets;
    uint32_t key0, key1;
    uint32_t stream_id;
    uint32_t tag;
};

// Tag tying a workspace's stats and offsets to the call that produced them.
__host__ __device__ inline uint32_t call_tag(uint32_t n, int variant, uint64_t seed, uint32_t stream_id)
{
    uint32_t h = 0x811C9DC5u;
    const uint32_t parts[5] = {n, (uint32_t)variant, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id};
    for (int i = 0; i < 5; ++i) h = (h ^ parts[i]) * 0x01000193u;
    return h | 1u;  // never 0
}

// Validated copy of mgp_params with defaults filled in.
struct Params {
    int variant;
    uint32_t B;
    double eps;
    uint64_t seed;
    uint32_t stream_id;
    uint32_t partition_bytes;
    uint32_t b_max;
    uint32_t segment = 32;  // Megopolis segment width, 32 or 64
};

int fail(int code, const char* fmt, ...);
void clear_error();
int check_launch(const char* what);
int normalize_params(const mgp_params* in, Params* out);
size_t workspace_bytes(uint32_t b_max);
size_t workspace_bytes(uint32_t n, const Params& p);
bool uses_windows(uint32_t n, int variant);
size_t windows_offset(uint32_t b_max);
uint32_t reduce_blocks(uint32_t n);
uint32_t reduce_chunk(uint32_t n, uint32_t blocks);
// Whether a Megopolis loop may read w in place: 128-byte aligned, and none of
// the byte ranges [out, out + bytes) of its outputs overlaps it.
struct OutRange {
    const void* at;
    uint64_t bytes;
};
bool in_place(const float* w, uint32_t n, const OutRange* outs, int count);
bool ranges_overlap(const void* a, uint64_t a_bytes, const void* b, uint64_t b_bytes);
// layout: kLayoutInPlace or kLayoutCopy (Megopolis with windows), else unused.
// copy (other variants): where the reduction also writes the n weights (16-byte aligned), or null.
int enqueue_reduce_finalize(const float* w, uint32_t n, const Params& p, bool make_offsets, uint32_t layout, char* ws,
                            mgp_stats* st_user, hipStream_t stream, float* copy = nullptr);
// The reduction's partials alone, and the arguments of the finalize step that
// the next kernel does over them.
int enqueue_partials(const float* w, uint32_t n, const Params& p, char* ws, uint32_t* nparts, FinalizeArgs* fin,
                     float* copy, hipStream_t stream);
// The accept loop (after the reduction and finalize launches); with rc.states
// set, the particle copy x_bar_i = x_{k_i} runs as its epilogue. anc may be
// null when rc copies the rows. layout: the reduction's; kLayoutCopy for a
// prepared loop.
int enqueue_loop(const float* w, uint32_t n, const Params& p, uint32_t layout, char* ws, int32_t* anc,
                 hipStream_t stream, const RowCopy& rc = RowCopy{});
// The accept loop for m outputs drawn from n weighted inputs (M != N, layout
// kLayoutCopy: m particles do not hold all the weights).
int enqueue_loop_m(const float* w, uint32_t n, uint32_t m, const Params& p, uint32_t layout, char* ws, int32_t* anc,
                   hipStream_t stream, const RowCopy& rc = RowCopy{});
int enqueue_gather(const float* states, uint32_t n_states, uint32_t d, const int32_t* anc, uint32_t n_out,
                   float* out, hipStream_t stream);
// mgp_resample's work: one launch up to 8192 (Megopolis) or 4096 particles,
// leaving nothing in the workspace for a prepared loop; two (the reduction,
// then the accept loop with the finalize step in every block) while that is
// faster; else the reduction + finalize and the accept loop.
int enqueue_resample(const float* w, uint32_t n, const Params& p, char* ws, mgp_stats* st_user, int32_t* anc,
                     hipStream_t stream, const RowCopy& rc = RowCopy{});

}  // namespace mgp
