// mgp_kernels.hip -- single-filter kernels for gfx950 and the C ABI of
// include/mgp.h: weight reduction, B selection and Megopolis offsets, the
// four accept loops, and the particle gather.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <mutex>

#include "mgp.h"
#include "mgp_device.h"
#include "mgp_internal.h"
#include "mgp_reduce.h"

namespace mgp {

// ---------------------------------------------------------------------------
// Errors
// ---------------------------------------------------------------------------
static thread_local char g_err[512];

int fail(int code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

void clear_error() { g_err[0] = '\0'; }

int check_launch(const char* what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(MGP_EHIP, "%s: %s", what, hipGetErrorString(e));
    return MGP_OK;
}

// ---------------------------------------------------------------------------
// 1. Reduction: fp32 max, fp64 sum, invalid-weight flag, per block.
//    The block decomposition depends on n only, so the fp64 sum (and B) is
//    the same on every call.
// ---------------------------------------------------------------------------
// What the reduction launch does beside the reduction, in blocks of their own
// after its nparts blocks, so that they run beside those:
//   - ends != 0: the ends of a Megopolis loop's windows (block nparts);
//   - early_offsets > 0: offsets o_0 .. o_{early_offsets - 1} and log(eps), for
//     a loop that does the finalize step itself. The offsets do not depend on
//     the weights, B only says how many are used.
struct ReduceExtra {
    float* copy;
    float* seam;
    uint32_t ends;
    uint32_t early_offsets;
    uint32_t* offsets;
    double* log_eps;
    FinalizeArgs a;
};

constexpr uint32_t kOffsetsPerBlock = 4096;  // early offsets: four calls per thread

// Block b < nparts reduces w[b*chunk, min(n, (b+1)*chunk)); chunk is a
// multiple of 4 and, with Vec, w is 16-byte aligned so float4 loads stay
// aligned.
template <bool Vec>
__global__ __launch_bounds__(kReduceThreads) void k_reduce(const float* __restrict__ w, uint32_t n,
                                                           uint32_t chunk, uint32_t nparts, Partial* __restrict__ part,
                                                           ReduceExtra x)
{
    if (blockIdx.x >= nparts) {
        const uint32_t e = blockIdx.x - nparts;
        if (x.ends && e == 0) {
            write_window_ends(w, n, x.copy, x.seam, nullptr);
        } else {
            const uint32_t first = (e - x.ends) * kOffsetsPerBlock;
            const uint32_t end = first + kOffsetsPerBlock < x.early_offsets ? first + kOffsetsPerBlock : x.early_offsets;
            if (first < end) draw_offsets(x.a, first, end, threadIdx.x, kReduceThreads, x.offsets);
            if (e == x.ends && threadIdx.x == 0) *x.log_eps = log(x.a.eps);
        }
        return;
    }
    // trailing blocks may start at or past n when chunk was rounded up: their
    // range is empty and they contribute the neutral partial
    const uint64_t start = (uint64_t)blockIdx.x * chunk;
    const uint64_t stop = start + chunk < (uint64_t)n ? start + chunk : (uint64_t)n;
    const uint64_t end = stop > start ? stop : start;
    float mx = 0.0f;
    double s = 0.0;
    uint32_t bad = 0;
    reduce_range<Vec>(w, start, end, x.copy, nullptr, mx, s, bad);
    block_reduce(mx, s, bad);
    if (threadIdx.x == 0) part[blockIdx.x] = Partial{s, mx, bad};
}

// ---------------------------------------------------------------------------
// 2. Finalize: see finalize_one in mgp_reduce.h.
// ---------------------------------------------------------------------------
// Blocks beyond the first write the tail of the weights (has_tail), copy[n + k] =
// src[k mod n], k < n + kSeam. Whether the loop wants it depends on B, so they do
// the step for themselves: a launch of its own after this one, which returned
// where the tail is not wanted, would cost every such call 3 us.
struct TailArgs {
    const float* src;
    float* copy;
};
constexpr uint32_t kTailBlocks = 512;

// Block b's share, by whole float4s of the copy (the first may hold up to three
// places before n, with the values that are there already).
__device__ __forceinline__ void write_tail(const TailArgs& t, uint32_t n, uint32_t b)
{
    constexpr uint32_t kAhead = 4, kStep = 4u * kTailBlocks * kReduceThreads;
    const uint32_t end = 2u * n + kSeam;
    uint32_t p = (n & ~3u) + 4u * (b * kReduceThreads + threadIdx.x);
    for (; p >= n && (uint64_t)p + (kAhead - 1u) * kStep + 4u <= 2ull * n; p += kAhead * kStep) {
        Row4 v[kAhead];
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u)
            v[u] = *reinterpret_cast<const Unaligned4*>(t.src + (p - n) + u * kStep);
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) *reinterpret_cast<Row4*>(t.copy + p + u * kStep) = v[u];
    }
    for (; p < end; p += kStep) {
        Row4 v;
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t k = p + c;  // below 2n + kSeam + 3 < 3n
            v[c] = t.src[k < n ? k : k < 2u * n ? k - n : k - 2u * n];
        }
        *reinterpret_cast<Row4*>(t.copy + p) = v;
    }
}

__global__ __launch_bounds__(kReduceThreads) void k_finalize(const Partial* __restrict__ part, uint32_t nparts,
                                                             FinalizeArgs a, mgp_stats* __restrict__ st,
                                                             mgp_stats* __restrict__ st_user,
                                                             uint32_t* __restrict__ offsets, TailArgs tail)
{
    __shared__ mgp_stats st_local;
    const bool first = blockIdx.x == 0;
    if (!first) a.make_offsets = 0u;
    const uint32_t B = finalize_one<true>(part, nparts, a, first ? st : &st_local, first ? st_user : nullptr, offsets);
    if (!first && has_tail(a.n, B)) write_tail(tail, a.n, blockIdx.x - 1u);
}

// ---------------------------------------------------------------------------
// 3. The accept loop. B and the validity of the weights come from the stats
//    that k_finalize wrote, or (Fin) every block does the finalize step over
//    the reduction's partials: the same sums in the same order, so the same B
//    and stats, which block 0 returns. That saves a launch of 3-5 us and its
//    gap for about 2 us at the start of each block.
// ---------------------------------------------------------------------------
struct LoopStart {
    const mgp_stats* st;   // !Fin: k_finalize's record
    uint32_t tag, b_cap;   // !Fin: what that record must say
    const Partial* parts;  // Fin
    uint32_t nparts;
    FinalizeArgs a;
    mgp_stats* st_ws;      // Fin: the workspace's record
    uint32_t prepares;     // Fin: that record may serve a prepared loop (as k_finalize leaves it), else it is refused
    mgp_stats* st_user;    // Fin: the caller's stats or null
};

// B, or 0 when every ancestor is -1: invalid weights, or (!Fin) a record that
// is not this very call's (n, variant, seed, stream) or a B beyond the
// workspace's offsets.
template <bool Fin>
__device__ __forceinline__ uint32_t loop_start(const LoopStart& l, uint32_t n)
{
    if constexpr (Fin) {
        __shared__ mgp_stats st_local;
        const uint32_t B = finalize_one(l.parts, l.nparts, l.a, &st_local, blockIdx.x == 0 ? l.st_user : nullptr,
                                        nullptr);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            mgp_stats r = st_local;
            if (!l.prepares) r.n = r.tag = 0u;
            *l.st_ws = r;
        }
        return B;
    } else {
        const uint32_t B = l.st->B;
        return l.st->status == MGP_OK && l.st->tag == l.tag && l.st->n == n && B <= l.b_cap ? B : 0u;
    }
}

// One particle per thread, any variant.
template <int V, bool Narrow, bool Fin>
__global__ __launch_bounds__(kLoopThreads) void k_resample(const float* __restrict__ w, uint32_t n, uint32_t m,
                                                           LoopStart ls, const uint32_t* __restrict__ offsets,
                                                           uint32_t key0, uint32_t key1, uint32_t stream_id,
                                                           uint32_t n_w, uint32_t n_part, uint32_t seg_mask,
                                                           int32_t* __restrict__ anc, RowCopy rc)
{
    const uint32_t i = blockIdx.x * kLoopThreads + threadIdx.x;
    const uint32_t B = loop_start<Fin>(ls, n);
    int32_t k = -1;
    if (B > 0) {
        // every lane runs a chain, also past m (C2 shares each group's
        // partition draws across its half-wave): output i starts at input
        // i mod n, i itself when i < n
        const LoopParams<GlobalPtr<const float>> P{global_ptr(w), offset_ptr(offsets), n, B, key0, key1, stream_id,
                                                   n_w, n_part, seg_mask};
        const uint32_t pos = i < n ? i : i % n;
        k = (int32_t)run_chain<V, Narrow, true>(P, i, pos);
    }
    if (i >= m) return;
    if (anc) anc[i] = k;
    if (rc.states) copy_row(rc, i, k);
}

// Where a single filter's Megopolis loop finds its windows, and, for a loop in
// place after which the workspace may serve a prepared loop, the copy that it
// completes.
struct WindowArgs {
    Windows at;
    float* keep;
};

// Megopolis by windows, P particles per thread, rounds of D steps. Rows
// selects the particle copy of the epilogue: 0 none, D4 > 0 rows of D4
// float4s, -1 any row shape (copy_row).
template <int P, int D, int Rows, bool Fin>
__global__ __launch_bounds__(kLoopThreads) void k_megopolis(WindowArgs wa, uint32_t n, uint32_t m, LoopStart ls,
                                                            const uint32_t* __restrict__ offsets, uint32_t key0,
                                                            uint32_t key1, uint32_t stream_id, uint32_t seg_mask,
                                                            int32_t* __restrict__ anc, RowCopy rc)
{
    const uint32_t start = blockIdx.x * (kLoopThreads * P);
    const uint32_t B = loop_start<Fin>(ls, n);
    uint32_t idx[P];
    int32_t k[P];
    bool live[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        idx[p] = start + threadIdx.x + kLoopThreads * p;
        live[p] = idx[p] < m;
        k[p] = -1;
    }
    if (B > 0) {
        // every lane runs, also past m (start < m <= n here): the window
        // keeps those loads in bounds, and only real outputs store
        uint32_t kc[P];
        megopolis_chain<P, (int)kLoopThreads, D, true>(wa.at, offset_ptr(offsets), n, B, key0, key1, stream_id, start, kc,
                                                 seg_mask, wa.keep, has_tail(n, B));
#pragma unroll
        for (int p = 0; p < P; ++p) k[p] = (int32_t)kc[p];
    }
    if (anc) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (live[p]) anc[idx[p]] = k[p];
    }
    if constexpr (Rows > 0) {
        copy_rows_vec4<P, Rows>(rc, idx, k, live);
    } else if constexpr (Rows < 0) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (live[p]) copy_row(rc, idx[p], k[p]);
    }
}

// Few outputs are few waves, which hide fewer round trips to memory: fewer
// particles per thread and longer rounds then. Calls one after the other in a
// graph, us, at B = 4 / 16 / 354 by particles per thread and steps per round:
//            1, 20              2, 10              4, 5
//   2^17     6.8 /  8.6 / 37.6  6.8 /  8.2 / 45.7  7.0 /  9.4 / 69.3
//   2^18     8.1 / 10.5 / 59.6  7.1 /  9.2 / 54.4  7.1 /  9.6 / 68.7
//   2^19    10.5 / 14.6 /  101  8.4 / 11.6 / 85.5  7.9 / 11.1 / 90.5
//   2^20    15.4 / 23.9 /  188 11.0 / 17.2 /  148 10.1 / 16.4 /  150
// Up to 2^16 k_megopolis_split is the fastest (below).
constexpr uint32_t kOneMaxM = 1u << 17;  // one particle per thread
constexpr uint32_t kTwoMaxM = 1u << 18;  // two

// mgp_resample of a small filter in one launch (Megopolis up to kSmallMaxN
// particles, the other variants up to kSmallMaxNOther): every block copies
// the weights into LDS, M[k] = w[k mod n] for k < n + kSmallPad, and repeats the
// reduction of k_reduce and k_finalize chunk by chunk in the same order (so
// the fp64 sum, B and the stats are bit-identical to the three-launch path,
// B by eq. (proposition) of Section 4.1), then runs the chains of its own
// particles against LDS: k_megopolis_split<kSplitSmall> for Megopolis
// (Algorithm 5), k_resample_small for Algorithms 2-4.
constexpr uint32_t kSmallMaxN = 8192;
constexpr uint32_t kSmallMaxNOther = 4096;  // Metropolis, C1, C2: chains without shared indices gain less
constexpr uint32_t kSmallPad = 64;        // a window of 64 particles starts below n
constexpr uint32_t kSmallMaxParts = kSmallMaxN / kReduceChunk;
static_assert(kSmallMaxN % kReduceChunk == 0 && kSmallMaxN <= (uint64_t)kReduceChunk * kMaxPartials,
              "the reduction of a small filter has at most kSmallMaxParts chunks");

// The first steps of the one-launch kernels: the weights into LDS,
// M[k] = w[k mod n], k < n + kSmallPad, then the reduction and B exactly as
// k_reduce and k_finalize compute them (chunks of `chunk` weights with
// k_reduce's thread mapping: float4 folds when fold_vec). Block 0 returns the
// stats. Returns B (0 for invalid weights) in every thread.
__device__ __forceinline__ uint32_t small_prologue(const float* __restrict__ w, uint32_t n, uint32_t nparts,
                                                   uint32_t chunk, uint32_t copy_vec, uint32_t fold_vec,
                                                   const FinalizeArgs& a, mgp_stats* __restrict__ st_ws,
                                                   mgp_stats* __restrict__ st_user, float* __restrict__ M,
                                                   Partial* __restrict__ parts, mgp_stats* __restrict__ st_local)
{
    // 1. the weights: every load of a thread is issued before its first LDS
    //    store (clamped indices, no branch around a load), so the copy costs
    //    one round trip to L2, not one per element
    if (copy_vec) {  // w 16-byte aligned and n % 4 == 0
        constexpr uint32_t kIt = kSmallMaxN / (4u * kLoopThreads);
        const float4* w4 = reinterpret_cast<const float4*>(w);
        const uint32_t last4 = n / 4u - 1u;
        float4 v[kIt];
#pragma unroll
        for (uint32_t it = 0; it < kIt; ++it) {
            const uint32_t k4 = threadIdx.x + it * kLoopThreads;
            v[it] = w4[k4 < last4 ? k4 : last4];
        }
        // lanes past the end store the last element again, to its own place
#pragma unroll
        for (uint32_t it = 0; it < kIt; ++it) {
            const uint32_t k4 = threadIdx.x + it * kLoopThreads;
            const uint32_t c4 = k4 < last4 ? k4 : last4;
            *reinterpret_cast<float4*>(M + 4u * c4) = v[it];
        }
    } else {
        constexpr uint32_t kIt = kSmallMaxN / kLoopThreads;
        float v[kIt];
#pragma unroll
        for (uint32_t it = 0; it < kIt; ++it) {
            const uint32_t k = threadIdx.x + it * kLoopThreads;
            v[it] = w[k < n ? k : n - 1u];
        }
#pragma unroll
        for (uint32_t it = 0; it < kIt; ++it) {
            const uint32_t k = threadIdx.x + it * kLoopThreads;
            const uint32_t c = k < n ? k : n - 1u;
            M[c] = v[it];
        }
    }
    __syncthreads();
    if (threadIdx.x < kSmallPad) M[n + threadIdx.x] = M[threadIdx.x % n];
    __syncthreads();
    // 2. the reduction, one chunk at a time with k_reduce's thread mapping
    for (uint32_t p = 0; p < nparts; ++p) {
        const uint64_t start = (uint64_t)p * chunk;
        const uint64_t stop = start + chunk < (uint64_t)n ? start + chunk : (uint64_t)n;
        const uint64_t end = stop > start ? stop : start;
        float mx = 0.0f;
        double s = 0.0;
        uint32_t bad = 0;
        if (fold_vec)
            reduce_range<true>(M, start, end, nullptr, nullptr, mx, s, bad);
        else
            reduce_range<false>(M, start, end, nullptr, nullptr, mx, s, bad);
        block_reduce(mx, s, bad);
        if (threadIdx.x == 0) parts[p] = Partial{s, mx, bad};
        __syncthreads();
    }
    // 3. B and the stats; block 0 returns them. The workspace record is
    //    marked unusable for mgp_resample_prepared (n = 0): this path leaves
    //    no offsets or windows there.
    const uint32_t B = finalize_one(parts, nparts, a, st_local, blockIdx.x == 0 ? st_user : nullptr, nullptr);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        mgp_stats r = *st_local;
        r.n = 0;
        r.tag = 0;
        *st_ws = r;
    }
    return B;
}

// The split loop's modes: B from k_finalize's record (kSplitPrepared), by the
// finalize step inside every block (kSplitFinalize), or, for n <= kSmallMaxN,
// the whole of mgp_resample in one launch with the weights in LDS
// (kSplitSmall, with small_prologue).
constexpr int kSplitPrepared = 0, kSplitFinalize = 1, kSplitSmall = 2;

// What kSplitSmall needs beside its LoopStart.
struct SmallArgs {
    const float* w;
    uint32_t chunk;     // weights per reduction chunk
    uint32_t copy_vec;  // float4 copies into LDS
    uint32_t fold_vec;  // float4 folds in the reduction
};

constexpr uint32_t kSplitMaxM = 1u << 16;  // beyond, four waves per 64 particles cost more than they hide
// Megopolis by windows for n up to kSplitMaxM, with each particle's work
// spread over four waves. A block serves 64 particles. Waves 1-3 compute the
// particles' u draws (one Philox call per five steps) and their candidates'
// weights, all independent of the chain, for a pass of kSplitPass steps into
// one of two LDS buffers, while wave 0 runs the chains of the pass before from
// the other; its serial part is the product, the compare and two selects per
// step. The chain keeps the number of the last accepted step, and the position
// comes from that step's offset at the end. The arithmetic and the draws are
// those of megopolis_chain: the ancestors are identical.
//
// What bounds it is instruction issue of the producers, on the CUs that have
// one block more than the others: at 20000 particles 160 instructions per u
// block (200 with each window's address worked out by scalar instructions and
// not by one lane per step); loads made a pass ahead, longer passes and more
// producers (7 of them: 18.5 instead of 20.2, but 3% slower at small B) give
// little. Whole calls, us, at B = 4 / 16 / 60 / 354, when the four waves took
// turns with the chain (passes of 20 steps, two barriers each) / now:
//   1000    6.9 / 5.9   7.8 / 6.5   9.5 / 7.8   22.2 / 12.6
//   8192    9.8 / 8.2  10.7 / 8.5  11.8 / 10.2  26.3 / 17.3
//   20000   7.9 / 7.8   8.7 / 8.5  11.3 / 9.9   29.6 / 20.2
//   2^16    9.3 / 8.5  10.1 / 9.4  12.9 / 11.3  38.5 / 28.2
// kSplitSmall reads the candidates from LDS and draws the offsets into LDS too
// (wave 0, two passes ahead).
constexpr uint32_t kSplitProducers = kLoopThreads / 64u - 1u;
constexpr uint32_t kSplitBlocks = 2;  // u blocks of five steps per producer and pass
constexpr uint32_t kSplitPass = 5u * kSplitBlocks * kSplitProducers;
static_assert(kSplitPass <= 64u, "a lane per step of the pass");

template <int Mode>
__global__ __launch_bounds__(kLoopThreads) void k_megopolis_split(WindowArgs wa, uint32_t n, uint32_t m, LoopStart ls,
                                                                  const uint32_t* __restrict__ offsets,
                                                                  uint32_t key0, uint32_t key1, uint32_t stream_id,
                                                                  uint32_t seg_mask, int32_t* __restrict__ anc,
                                                                  SmallArgs f, RowCopy rc)
{
    __shared__ float2 step[2][kSplitPass][64];  // u and the candidate's weight
    const uint32_t lane = threadIdx.x & 63u;
    // the wave's index, known to the compiler as wave-uniform: no divergence
    // between the chains' wave and the producers
    const uint32_t q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t i = blockIdx.x * 64u + lane;
    constexpr bool kOwnOffsets = Mode == kSplitSmall;
    __shared__ uint32_t soffs[2][kOwnOffsets ? kSplitPass : 1];  // the offsets of a pass and the next
    __shared__ __align__(16) float Ms[Mode == kSplitSmall ? kSmallMaxN + kSmallPad : 1];
    uint32_t B;
    if constexpr (Mode == kSplitSmall) {
        // the weights into LDS, the reduction and B (small_prologue)
        __shared__ Partial parts[kSmallMaxParts];
        __shared__ mgp_stats st_local;
        B = small_prologue(f.w, n, ls.nparts, f.chunk, f.copy_vec, f.fold_vec, ls.a, ls.st_ws, ls.st_user, Ms, parts,
                           &st_local);
    } else {
        B = loop_start<Mode == kSplitFinalize>(ls, n);
    }
    if (B == 0) {
        if (q == 0 && i < m) {
            if (anc) anc[i] = -1;
            if (rc.states) copy_row(rc, i, -1);
        }
        return;
    }
    // lanes past m run too (the window keeps their loads in bounds)
    const uint32_t start = blockIdx.x * 64u;
    const uint32_t la4 = (lane & ~seg_mask) * 4u;
    const uint32_t ll4 = (lane & seg_mask) * 4u;
    const Windows W = wa.at;
    // the weight at a window position (byte offset v of the window from position s on)
    auto candidate = [&](uint32_t s, uint32_t v) -> float {
        if constexpr (Mode == kSplitSmall)
            return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Ms) + 4u * s + v);
        else
            return *(GlobalPtr<const float>)(window_at(W, s, n, 64u) + v);
    };
    // the offsets of the pass starting at step c0, drawn as draw_offsets draws
    // them, by the threads t0, t0 + stride, ... of the block
    auto draw_pass = [&](uint32_t c0, uint32_t* dst, uint32_t t0, uint32_t stride) {
        const uint32_t cnt = B - c0 < kSplitPass ? B - c0 : kSplitPass;
        // whole Philox calls: c0 need not be a multiple of four
        for (uint32_t c = c0 / 4u + t0; c < (c0 + cnt + 3u) / 4u; c += stride) {
            const Words x = philox(c, kTagOffset, stream_id, 0u, key0, key1);
            const uint32_t o[4] = {x.x0, x.x1, x.x2, x.x3};
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {
                const uint32_t d = 4u * c + r - c0;  // wraps below c0
                if (d < cnt) dst[d] = uniform_index(o[r], n);
            }
        }
    };
    if constexpr (kOwnOffsets) {
        draw_pass(0u, soffs[0], threadIdx.x, kLoopThreads);
        if (B > kSplitPass) draw_pass(kSplitPass, soffs[1], threadIdx.x, kLoopThreads);
        __syncthreads();
    }
    // A producer's part of the pass from step b0 on: the u blocks q - 1,
    // q - 1 + kSplitProducers, ... of it. Lane l first works out where the window of
    // the pass's step l lies (past B that of step B - 1, which the chain does
    // not read); each of its steps then takes that from its lane.
    auto produce = [&](uint32_t b0, uint32_t buf) {
        const uint32_t cnt = B - b0 < kSplitPass ? B - b0 : kSplitPass;
        const uint32_t sl = lane < cnt ? lane : cnt - 1u;
        uint32_t o = kOwnOffsets ? soffs[buf][sl] : offsets[b0 + sl];
        o = o < n ? o : n - 1u;
        const uint32_t at = window_start(start, o, seg_mask, n);
        const uint32_t rot = (o & seg_mask) * 4u;
        const uint64_t base = kOwnOffsets ? (uint64_t)at * 4u : (uint64_t)window_at(W, at, n, 64u);
        float wj[kSplitBlocks][5];
#pragma unroll
        for (uint32_t t = 0; t < kSplitBlocks; ++t) {
            const uint32_t g = q - 1u + kSplitProducers * t;
            if (g * 5u >= cnt) continue;
#pragma unroll
            for (uint32_t r = 0; r < 5u; ++r) {
                const int s = (int)(g * 5u + r);
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, s);
                const uint32_t v =
                    la4 | ((ll4 + (uint32_t)__builtin_amdgcn_readlane((int)rot, s)) & (seg_mask * 4u));
                if constexpr (kOwnOffsets) {
                    wj[t][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Ms) + lo + v);
                } else {
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> 32), s);
                    wj[t][r] = *(GlobalPtr<const float>)((GlobalPtr<const char>)(((uint64_t)hi << 32) | lo) + v);
                }
            }
        }
#pragma unroll
        for (uint32_t t = 0; t < kSplitBlocks; ++t) {
            const uint32_t g = q - 1u + kSplitProducers * t;
            if (g * 5u >= cnt) continue;
            const UBlock ub = u_block(philox(b0 / 5u + g, kTagU, stream_id, i, key0, key1));
#pragma unroll
            for (uint32_t r = 0; r < 5u; ++r) step[buf][g * 5u + r][lane] = make_float2(ub.u[r], wj[t][r]);
        }
    };
    float wk = candidate(start, lane * 4u);
    if (Mode != kSplitSmall && wa.keep && q == 0) keep_weight(wa.keep, n, i, wk);
    uint32_t last = 0xFFFFFFFFu;  // the last accepted step
    if (q > 0) produce(0u, 0u);
    __syncthreads();
    for (uint32_t b0 = 0, buf = 0; b0 < B; b0 += kSplitPass, buf ^= 1u) {
        if (q > 0) {
            if (b0 + kSplitPass < B) produce(b0 + kSplitPass, buf ^ 1u);
        } else {
            const uint32_t cnt = B - b0 < kSplitPass ? B - b0 : kSplitPass;
            uint32_t at = 0xFFFFFFFFu;
            if (cnt == kSplitPass) {
                float2 x[kSplitPass];
#pragma unroll
                for (uint32_t s = 0; s < kSplitPass; ++s) x[s] = step[buf][s][lane];
#pragma unroll
                for (uint32_t s = 0; s < kSplitPass; ++s) {
                    const float prod = x[s].x * wk;
                    const bool acc = prod <= x[s].y;
                    at = acc ? s : at;
                    wk = acc ? x[s].y : wk;
                }
            } else {
                for (uint32_t s = 0; s < cnt; ++s) {
                    const float2 x = step[buf][s][lane];
                    const float prod = x.x * wk;
                    const bool acc = prod <= x.y;
                    at = acc ? s : at;
                    wk = acc ? x.y : wk;
                }
            }
            last = at != 0xFFFFFFFFu ? b0 + at : last;
            // the producers read the other buffer's offsets now
            if constexpr (kOwnOffsets)
                if (b0 + 2u * kSplitPass < B) draw_pass(b0 + 2u * kSplitPass, soffs[buf], lane, 64u);
        }
        __syncthreads();  // the buffers change sides
    }
    if (q == 0 && i < m) {
        uint32_t k = i;
        if (last != 0xFFFFFFFFu) {
            uint32_t o;
            if constexpr (kOwnOffsets) {
                const Words x = philox(last / 4u, kTagOffset, stream_id, 0u, key0, key1);
                const uint32_t lo = (last & 1u) ? x.x1 : x.x0, hi = (last & 1u) ? x.x3 : x.x2;
                o = uniform_index((last & 2u) ? hi : lo, n);
            } else {
                o = offsets[last];
                o = o < n ? o : n - 1u;
            }
            k = window_start(start, o, seg_mask, n) +
                (la4 | ((ll4 + (o & seg_mask) * 4u) & (seg_mask * 4u))) / 4u;
        }
        const int32_t kn = (int32_t)(k >= n ? k - n : k);
        if (anc) anc[i] = kn;
        if (rc.states) copy_row(rc, i, kn);
    }
}


// Metropolis, C1 and C2 (Algorithms 2-4) for a small filter in one launch:
// the same prologue, then each thread runs its particle's chain of k_resample
// against the weights in LDS.
template <int V>
__global__ __launch_bounds__(kLoopThreads) void k_resample_small(const float* __restrict__ w, uint32_t n,
                                                                 uint32_t nparts, uint32_t chunk, uint32_t copy_vec,
                                                                 uint32_t fold_vec, FinalizeArgs a,
                                                                 mgp_stats* __restrict__ st_ws,
                                                                 mgp_stats* __restrict__ st_user, uint32_t n_w,
                                                                 uint32_t n_part, int32_t* __restrict__ anc,
                                                                 RowCopy rc)
{
    __shared__ __align__(16) float M[kSmallMaxN + kSmallPad];
    __shared__ Partial parts[kSmallMaxParts];
    __shared__ mgp_stats st_local;
    const uint32_t B = small_prologue(w, n, nparts, chunk, copy_vec, fold_vec, a, st_ws, st_user, M, parts, &st_local);
    const uint32_t i = blockIdx.x * kLoopThreads + threadIdx.x;
    int32_t k = -1;  // invalid weights: B == 0
    if (B > 0) {
        // every lane runs a chain (lanes past n from n - 1's group, whose
        // partition draws C2 shares across the half-wave)
        const LoopParams<const float*> P{M, nullptr, n, B, a.key0, a.key1, a.stream_id, n_w, n_part};
        const uint32_t ic = i < n ? i : n - 1u;
        k = (int32_t)run_chain<V, true, true>(P, ic, ic);
    }
    if (i >= n) return;
    if (anc) anc[i] = k;
    if (rc.states) copy_row(rc, i, k);
}

// ---------------------------------------------------------------------------
// 4. Gather: out[i] = states[anc[i]] (rows of d fp32). With d % 4 == 0 and
//    16-byte aligned rows every thread copies one float4; otherwise one
//    float. Out-of-range ancestors give NaN rows.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gather_vec4(const float4* __restrict__ states, uint32_t n_states,
                                                     uint32_t d4, const int32_t* __restrict__ anc, uint64_t total,
                                                     float4* __restrict__ out)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const uint64_t row = t / d4;
        const uint32_t c = (uint32_t)(t - row * d4);
        const int32_t k = anc[row];
        float4 v;
        if (k >= 0 && (uint32_t)k < n_states) {
            v = states[(uint64_t)k * d4 + c];
        } else {
            v = make_float4(NAN, NAN, NAN, NAN);
        }
        // the output is written once and not read here: stream it past the
        // L2 so that the ancestor rows being read stay cached
        __builtin_nontemporal_store(v.x, &out[t].x);
        __builtin_nontemporal_store(v.y, &out[t].y);
        __builtin_nontemporal_store(v.z, &out[t].z);
        __builtin_nontemporal_store(v.w, &out[t].w);
    }
}

__global__ __launch_bounds__(256) void k_gather_scalar(const float* __restrict__ states, uint32_t n_states,
                                                       uint32_t d, const int32_t* __restrict__ anc, uint64_t total,
                                                       float* __restrict__ out)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const uint64_t row = t / d;
        const uint32_t c = (uint32_t)(t - row * d);
        const int32_t k = anc[row];
        __builtin_nontemporal_store((k >= 0 && (uint32_t)k < n_states) ? states[(uint64_t)k * d + c] : NAN, &out[t]);
    }
}

// The same for fewer than 2^31 elements (T: floats or float4s), Per of them to a
// thread: the row comes from a multiplication, t / d = t mult >> shift
// (row_divisor), where a 64-bit division of some hundred instructions per
// element bound rows of odd lengths, and the thread's loads are in flight
// together. us, 2^22 rows in order of a resample at y = 0, 64-bit divisions / now:
// d = 3 34.5 / 24.6, d = 5 54.6 / 39.8, d = 33 442 / 215 (HBM rate), d = 4 and 16
// even; 100003 rows, d = 5: 2.6 / 2.2.
struct RowDivisor {
    uint32_t mult, shift;
};

template <typename T, uint32_t Per>
__global__ __launch_bounds__(256) void k_gather(const T* __restrict__ states, uint32_t n_states, uint32_t d,
                                                RowDivisor by, const int32_t* __restrict__ anc, uint32_t total,
                                                T* __restrict__ out)
{
    const uint32_t first = blockIdx.x * (256u * Per) + threadIdx.x;
    int32_t k[Per];
    uint32_t c[Per];
    T v[Per];
#pragma unroll
    for (uint32_t e = 0; e < Per; ++e) {
        const uint32_t t = first + 256u * e < total ? first + 256u * e : total - 1u;
        const uint32_t row = (uint32_t)(((uint64_t)t * by.mult) >> by.shift);
        c[e] = t - row * d;
        k[e] = anc[row];
    }
#pragma unroll
    for (uint32_t e = 0; e < Per; ++e) {
        const bool in = k[e] >= 0 && (uint32_t)k[e] < n_states;
        const T x = states[(in ? (uint64_t)k[e] * d : 0u) + c[e]];
        v[e] = in ? x : (T)NAN;
    }
#pragma unroll
    for (uint32_t e = 0; e < Per; ++e)
        if (first + 256u * e < total) __builtin_nontemporal_store(v[e], &out[first + 256u * e]);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
uint32_t reduce_blocks(uint32_t n)
{
    // about kReduceChunk weights per block, at most kMaxPartials blocks
    uint64_t g = ((uint64_t)n + kReduceChunk - 1u) / kReduceChunk;
    if (g > kMaxPartials) g = kMaxPartials;
    if (g < 1) g = 1;
    return (uint32_t)g;
}

uint32_t reduce_chunk(uint32_t n, uint32_t blocks)
{
    uint64_t c = ((uint64_t)n + blocks - 1) / blocks;
    c = (c + 3u) & ~(uint64_t)3u;
    return (uint32_t)c;
}

int normalize_params(const mgp_params* in, Params* out)
{
    if (!in) return fail(MGP_EINVAL, "params is NULL");
    if (in->variant < MGP_METROPOLIS || in->variant > MGP_MEGOPOLIS)
        return fail(MGP_EINVAL, "unknown variant %d", in->variant);
    out->variant = in->variant;
    out->B = in->B;
    out->eps = in->epsilon;
    out->seed = in->seed;
    out->stream_id = in->stream_id;
    out->partition_bytes = in->partition_bytes ? in->partition_bytes : 128u;
    out->b_max = in->b_max ? in->b_max : kDefaultBMax;
    out->segment = in->segment ? in->segment : 32u;
    if (out->segment != 32u && out->segment != 64u)
        return fail(MGP_EINVAL, "segment must be 32 or 64 (got %u)", in->segment);
    if (out->partition_bytes < 4u || out->partition_bytes % 4u != 0u)
        return fail(MGP_EINVAL, "partition_bytes must be a positive multiple of 4 (got %u)", out->partition_bytes);
    if (out->b_max > kBMaxLimit) return fail(MGP_ERANGE, "b_max %u above the limit %u", out->b_max, kBMaxLimit);
    if (out->B == 0) {
        if (!(out->eps > 0.0) || !(out->eps <= 1.0))
            return fail(MGP_EINVAL, "epsilon must be in (0, 1] when B is 0 (got %g)", out->eps);
    } else if (out->B > out->b_max) {
        return fail(MGP_ERANGE, "B = %u above b_max = %u", out->B, out->b_max);
    }
    return MGP_OK;
}

size_t workspace_bytes(uint32_t b_max)
{
    return kWsOffsetsOffset + (((size_t)b_max * 4u + 255u) & ~(size_t)255u);
}

bool uses_windows(uint32_t n, int variant) { return variant == kMegopolis && n <= kWindowMaxN; }

size_t windows_offset(uint32_t b_max) { return workspace_bytes(b_max); }

size_t workspace_bytes(uint32_t n, const Params& p)
{
    size_t b = workspace_bytes(p.b_max);
    if (uses_windows(n, p.variant)) b += (((size_t)2 * n + kWindowReserve) * 4u + 255u) & ~(size_t)255u;
    return b;
}

bool ranges_overlap(const void* a, uint64_t a_bytes, const void* b, uint64_t b_bytes)
{
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a && b && a_bytes && b_bytes && a0 < b0 + b_bytes && b0 < a0 + a_bytes;
}

bool in_place(const float* w, uint32_t n, const OutRange* outs, int count)
{
    if (((uintptr_t)w & 127u) != 0) return false;
    for (int k = 0; k < count; ++k)
        if (ranges_overlap(w, 4ull * n, outs[k].at, outs[k].bytes)) return false;
    return true;
}

// The layout for a call that resamples n weights into n ancestors (and rows).
static uint32_t loop_layout(const float* w, uint32_t n, const int32_t* anc, const mgp_stats* st_user,
                            const RowCopy& rc)
{
    const OutRange outs[3] = {{anc, 4ull * n}, {rc.out, 4ull * n * rc.d}, {st_user, sizeof(mgp_stats)}};
    return n >= kSeam && in_place(w, n, outs, 3) ? kLayoutInPlace : kLayoutCopy;
}

static FinalizeArgs finalize_args(uint32_t n, const Params& p, bool make_offsets)
{
    FinalizeArgs a;
    a.n = n;
    a.eps = p.eps;
    a.log_eps = nullptr;
    a.B_user = p.B;
    a.b_max = p.b_max;
    a.make_offsets = make_offsets ? 1u : 0u;
    a.key0 = (uint32_t)p.seed;
    a.key1 = (uint32_t)(p.seed >> 32);
    a.stream_id = p.stream_id;
    a.tag = call_tag(n, p.variant, p.seed, p.stream_id);
    return a;
}

// The reduction launch: partials and, for Megopolis with make_offsets, the
// ends of the windows or the copy; with early > 0 also that many offsets, and
// log(eps). With copy (16-byte aligned, and no windows asked for), the weights
// too. Returns the number of partials through *nparts.
static int enqueue_reduce(const float* w, uint32_t n, const Params& p, bool make_offsets, uint32_t layout,
                          bool early, char* ws, uint32_t* nparts, hipStream_t stream, float* copy = nullptr)
{
    Partial* part = reinterpret_cast<Partial*>(ws + kWsPartialsOffset);
    const uint32_t g = reduce_blocks(n);
    const uint32_t chunk = reduce_chunk(n, g);
    ReduceExtra x{};
    x.copy = copy;
    uint32_t extra = 0;
    if (make_offsets && uses_windows(n, p.variant)) {
        float* at = reinterpret_cast<float*>(ws + windows_offset(p.b_max));
        x.copy = layout == kLayoutCopy ? at : nullptr;
        x.seam = layout == kLayoutInPlace ? at + (n - kSeam) : nullptr;
        x.ends = 1u;
        extra = 1u;
    }
    if (early) {
        x.early_offsets = make_offsets ? (p.B ? p.B : p.b_max) : 0u;
        x.offsets = reinterpret_cast<uint32_t*>(ws + kWsOffsetsOffset);
        x.log_eps = reinterpret_cast<double*>(ws + kWsLogEpsOffset);
        x.a = finalize_args(n, p, false);
        const uint32_t blocks = (x.early_offsets + kOffsetsPerBlock - 1u) / kOffsetsPerBlock;
        extra += blocks ? blocks : 1u;
    }
    const dim3 grid(g + extra);
    if (((uintptr_t)w & 15u) == 0)
        hipLaunchKernelGGL(k_reduce<true>, grid, dim3(kReduceThreads), 0, stream, w, n, chunk, g, part, x);
    else
        hipLaunchKernelGGL(k_reduce<false>, grid, dim3(kReduceThreads), 0, stream, w, n, chunk, g, part, x);
    *nparts = g;
    return check_launch("reduce kernel");
}

int enqueue_reduce_finalize(const float* w, uint32_t n, const Params& p, bool make_offsets, uint32_t layout, char* ws,
                            mgp_stats* st_user, hipStream_t stream, float* copy)
{
    Partial* part = reinterpret_cast<Partial*>(ws + kWsPartialsOffset);
    mgp_stats* st = reinterpret_cast<mgp_stats*>(ws + kWsStatsOffset);
    uint32_t* offs = reinterpret_cast<uint32_t*>(ws + kWsOffsetsOffset);
    uint32_t g = 0;
    int rc = enqueue_reduce(w, n, p, make_offsets, layout, false, ws, &g, stream, copy);
    if (rc) return rc;
    const FinalizeArgs a = finalize_args(n, p, make_offsets);
    TailArgs tail{};
    uint32_t blocks = 1;
    if (make_offsets && uses_windows(n, p.variant) && has_tail(n, p.B ? p.B : p.b_max)) {
        tail.copy = reinterpret_cast<float*>(ws + windows_offset(p.b_max));
        tail.src = layout == kLayoutCopy ? tail.copy : w;
        blocks += kTailBlocks;
    }
    hipLaunchKernelGGL(k_finalize, dim3(blocks), dim3(kReduceThreads), 0, stream, part, g, a, st, st_user, offs, tail);
    return check_launch("finalize kernel");
}

int enqueue_partials(const float* w, uint32_t n, const Params& p, char* ws, uint32_t* nparts, FinalizeArgs* fin,
                     float* copy, hipStream_t stream)
{
    *fin = finalize_args(n, p, false);
    return enqueue_reduce(w, n, p, false, kLayoutInPlace, false, ws, nparts, stream, copy);
}

// The accept loop's launch for m outputs from n inputs, with the finalize
// step done before it (Fin false) or by its blocks.
template <bool Fin>
struct LoopLaunch {
    const float* w;
    uint32_t n, m;
    const Params& p;
    uint32_t layout;
    char* ws;
    LoopStart ls;
    int32_t* anc;
    const RowCopy& rc;
    hipStream_t stream;
    const uint32_t* offs = reinterpret_cast<const uint32_t*>(ws + kWsOffsetsOffset);
    uint32_t k0 = (uint32_t)p.seed, k1 = (uint32_t)(p.seed >> 32);
    uint32_t seg_mask = p.segment - 1u;

    WindowArgs window_args() const
    {
        float* copy = reinterpret_cast<float*>(ws + windows_offset(p.b_max));
        if (layout == kLayoutCopy) return WindowArgs{windows_copy(copy), nullptr};
        return WindowArgs{windows_in_place(w, copy + (n - kSeam), n), !Fin || ls.prepares ? copy : nullptr};
    }

    template <int V>
    void variant() const
    {
        const uint32_t n_w = p.partition_bytes / 4u;
        const uint32_t n_part = (uint32_t)(((uint64_t)n + n_w - 1u) / n_w);
        const dim3 grid((m + kLoopThreads - 1u) / kLoopThreads);
        if (Fin || n <= (1u << 30))  // Fin: n <= kFinMaxN
            hipLaunchKernelGGL((k_resample<V, true, Fin>), grid, dim3(kLoopThreads), 0, stream, w, n, m, ls, offs, k0,
                               k1, p.stream_id, n_w, n_part, seg_mask, anc, rc);
        else
            hipLaunchKernelGGL((k_resample<V, false, false>), grid, dim3(kLoopThreads), 0, stream, w, n, m, ls, offs,
                               k0, k1, p.stream_id, n_w, n_part, seg_mask, anc, rc);
    }

    template <int P, int D, int Rows>
    void windows_rows() const
    {
        const dim3 grid((m + kLoopThreads * P - 1u) / (kLoopThreads * P));
        hipLaunchKernelGGL((k_megopolis<P, D, Rows, Fin>), grid, dim3(kLoopThreads), 0, stream, window_args(), n, m,
                           ls, offs, k0, k1, p.stream_id, seg_mask, anc, rc);
    }

    // by windows, with the epilogue that fits the row copy
    template <int P, int D>
    void windows() const
    {
        const uint32_t d4 = rc.vec4 ? rc.d / 4u : 0u;
        if (!rc.states)
            windows_rows<P, D, 0>();
        else if (d4 == 1u)
            windows_rows<P, D, 1>();
        else if (d4 == 2u)
            windows_rows<P, D, 2>();
        else if (d4 == 4u)
            windows_rows<P, D, 4>();
        else
            windows_rows<P, D, -1>();
    }

    int run() const
    {
        if (uses_windows(n, p.variant) && m <= n) {
            if (m <= kSplitMaxM)
                hipLaunchKernelGGL(k_megopolis_split<(Fin ? kSplitFinalize : kSplitPrepared)>, dim3((m + 63u) / 64u),
                                   dim3(kLoopThreads), 0, stream, window_args(), n, m, ls, offs, k0, k1,
                                   p.stream_id, seg_mask, anc, SmallArgs{}, rc);
            else if (m <= kOneMaxM)
                windows<1, 20>();
            else if (m <= kTwoMaxM)
                windows<2, 10>();
            else
                windows<kMegopolisPPT, 5>();
        } else if (p.variant == kMetropolis) {
            variant<kMetropolis>();
        } else if (p.variant == kC1) {
            variant<kC1>();
        } else if (p.variant == kC2) {
            variant<kC2>();
        } else if constexpr (!Fin) {
            variant<kMegopolis>();  // m > n, or n beyond the windows
        }
        return check_launch("resample kernel");
    }
};

int enqueue_loop(const float* w, uint32_t n, const Params& p, uint32_t layout, char* ws, int32_t* anc,
                 hipStream_t stream, const RowCopy& rc)
{
    return enqueue_loop_m(w, n, n, p, layout, ws, anc, stream, rc);
}

int enqueue_loop_m(const float* w, uint32_t n, uint32_t m, const Params& p, uint32_t layout, char* ws, int32_t* anc,
                   hipStream_t stream, const RowCopy& rc)
{
    LoopStart ls{};
    ls.st = reinterpret_cast<const mgp_stats*>(ws + kWsStatsOffset);
    ls.tag = call_tag(n, p.variant, p.seed, p.stream_id);
    ls.b_cap = p.b_max;
    return LoopLaunch<false>{w, n, m, p, layout, ws, ls, anc, rc, stream}.run();
}

// mgp_resample with n <= kSmallMaxN (Megopolis) or kSmallMaxNOther: one
// launch of k_megopolis_split<kSplitSmall> or k_resample_small. The reduction
// uses the chunks, thread mapping and fold width that enqueue_reduce_finalize
// uses for the same n and weight alignment (float4 folds need a 16-byte
// aligned w).
int enqueue_small(const float* w, uint32_t n, const Params& p, char* ws, mgp_stats* st_user, int32_t* anc,
                  hipStream_t stream, const RowCopy& rc)
{
    const uint32_t g = reduce_blocks(n);
    const uint32_t chunk = reduce_chunk(n, g);
    const bool aligned = ((uintptr_t)w & 15u) == 0;
    const uint32_t copy_vec = (aligned && n % 4u == 0) ? 1u : 0u;
    const uint32_t fold_vec = aligned ? 1u : 0u;
    const FinalizeArgs a = finalize_args(n, p, false);
    mgp_stats* st_ws = reinterpret_cast<mgp_stats*>(ws + kWsStatsOffset);
    const dim3 grid((n + kLoopThreads - 1u) / kLoopThreads);
    const uint32_t n_w = p.partition_bytes / 4u;
    const uint32_t n_part = (uint32_t)(((uint64_t)n + n_w - 1u) / n_w);
    switch (p.variant) {
    case kMegopolis: {
            LoopStart ls{};
            ls.nparts = g;
            ls.a = a;
            ls.st_ws = st_ws;
            ls.st_user = st_user;
            hipLaunchKernelGGL(k_megopolis_split<kSplitSmall>, dim3((n + 63u) / 64u), dim3(kLoopThreads), 0, stream,
                               WindowArgs{}, n, n, ls, nullptr, a.key0, a.key1, p.stream_id, p.segment - 1u, anc,
                               SmallArgs{w, chunk, copy_vec, fold_vec}, rc);
            break;
        }
    case kMetropolis:
        hipLaunchKernelGGL(k_resample_small<kMetropolis>, grid, dim3(kLoopThreads), 0, stream, w, n, g, chunk,
                           copy_vec, fold_vec, a, st_ws, st_user, n_w, n_part, anc, rc);
        break;
    case kC1:
        hipLaunchKernelGGL(k_resample_small<kC1>, grid, dim3(kLoopThreads), 0, stream, w, n, g, chunk, copy_vec,
                           fold_vec, a, st_ws, st_user, n_w, n_part, anc, rc);
        break;
    default:
        hipLaunchKernelGGL(k_resample_small<kC2>, grid, dim3(kLoopThreads), 0, stream, w, n, g, chunk, copy_vec,
                           fold_vec, a, st_ws, st_user, n_w, n_part, anc, rc);
        break;
    }
    return check_launch("resample kernel (one launch)");
}

// mgp_resample does the finalize step inside the loop (two launches instead of
// three) up to these sizes; beyond, the step repeated in every block costs more
// than the launch. Calls one after the other, us, three launches / two, at B = 16:
//   Megopolis   2^15 8.9 / 7.5, 2^17 10.0 / 8.6, 2^20 17.9 / 16.4, 2^21 26.3 / 26.1
//               (B = 354: 285 / 291)
//   Metropolis  2^14 10.2 / 8.7, 2^18 26.2 / 24.9, 2^19 42.8 / 42.8, 2^20 80.6 / 84.0
//   C1, C2      2^14 9.9 / 8.4 and 10.3 / 8.9, 2^18 12.8 / 11.8 and 13.6 / 12.6,
//               2^19 16.5 / 17.1 and 17.9 / 18.9
constexpr uint32_t kFinMaxN = 1u << 20;
constexpr uint32_t kFinMaxNOther = 1u << 18;
constexpr uint32_t kEarlyOffsetsMax = 65536;    // offsets worth drawing before B is known: 16 blocks
constexpr uint32_t kNoPrepareMaxN = 1u << 15;

int enqueue_resample(const float* w, uint32_t n, const Params& p, char* ws, mgp_stats* st_user, int32_t* anc,
                     hipStream_t stream, const RowCopy& rc)
{
    if (n <= (p.variant == kMegopolis ? kSmallMaxN : kSmallMaxNOther))
        return enqueue_small(w, n, p, ws, st_user, anc, stream, rc);
    const bool mego = p.variant == kMegopolis;
    const uint32_t layout = loop_layout(w, n, anc, st_user, rc);
    if (n <= (mego ? kFinMaxN : kFinMaxNOther) && (!mego || p.B || p.b_max <= kEarlyOffsetsMax)) {
        uint32_t g = 0;
        const int err = enqueue_reduce(w, n, p, mego, layout, true, ws, &g, stream);
        if (err) return err;
        LoopStart ls{};
        ls.parts = reinterpret_cast<const Partial*>(ws + kWsPartialsOffset);
        ls.nparts = g;
        ls.a = finalize_args(n, p, false);
        ls.a.log_eps = reinterpret_cast<const double*>(ws + kWsLogEpsOffset);
        ls.st_ws = reinterpret_cast<mgp_stats*>(ws + kWsStatsOffset);
        ls.st_user = st_user;
        // up to 2^15 particles Megopolis has never left a workspace that a prepared loop takes
        ls.prepares = !mego || n > kNoPrepareMaxN ? 1u : 0u;
        return LoopLaunch<true>{w, n, n, p, layout, ws, ls, anc, rc, stream}.run();
    }
    int err = enqueue_reduce_finalize(w, n, p, mego, layout, ws, st_user, stream);
    if (err) return err;
    return enqueue_loop(w, n, p, layout, ws, anc, stream, rc);
}

// 2^31 elements and more: 2^20 blocks, grid-stride.
static uint32_t gather_blocks(uint64_t total)
{
    const uint64_t b = (total + 255u) / 256u;
    return (uint32_t)(b < (1u << 20) ? (b ? b : 1) : (1u << 20));
}

// Floats from which a thread of the gather takes four and not two. us, two /
// four: 100003 rows of 3 2.1 / 2.2, 2^20 rows of 2 4.1 / 4.0, of 5 12.6 / 9.7,
// of 33 63 / 51.
constexpr uint64_t kGatherFour = 1ull << 21;
// float4s to a thread: two, but one from the first to the second number of them.
// us, one / two: 300007 rows of 12 floats (0.9 M) 6.7 / 5.2, 2^20 of 12 (3 M)
// 25.7 / 26.3, 2^23 of 4 (8 M) 98.2 / 100.9, of 8 (17 M) 142 / 146, of 12 (25 M)
// 199 / 198, 2000003 of 64 (32 M) 163 / 157.
constexpr uint64_t kGatherOneFrom = 5ull << 19, kGatherOneTo = 1ull << 24;

// floor(t / d) = t mult >> shift for t < 2^31: with 2^L >= d > 2^(L-1),
// mult = (2^(31+L) + e) / d for some 0 < e <= d fits 32 bits, and the quotient
// is too large by t e / (d 2^(31+L)) < 1 / d.
static RowDivisor row_divisor(uint32_t d)
{
    uint32_t L = 0;
    while (((uint64_t)1 << L) < d) ++L;
    return RowDivisor{(uint32_t)(((uint64_t)1 << (31u + L)) / d + 1u), 31u + L};
}

template <typename T, uint32_t Per>
static void launch_gather(const T* states, uint32_t n_states, uint32_t d, const int32_t* anc, uint64_t total, T* out,
                          hipStream_t stream)
{
    const dim3 grid((uint32_t)((total + 256u * Per - 1u) / (256u * Per)));
    hipLaunchKernelGGL((k_gather<T, Per>), grid, dim3(256), 0, stream, states, n_states, d, row_divisor(d), anc,
                       (uint32_t)total, out);
}

int enqueue_gather(const float* states, uint32_t n_states, uint32_t d, const int32_t* anc, uint32_t n_out,
                   float* out, hipStream_t stream)
{
    if (n_out == 0) return MGP_OK;
    const bool vec = (d % 4u == 0u) && (((uintptr_t)states & 15u) == 0) && (((uintptr_t)out & 15u) == 0);
    const uint64_t total = (uint64_t)n_out * (vec ? d / 4u : d);
    const bool wide = total >= (1ull << 31);  // 64-bit element numbers
    if (vec && wide) {
        hipLaunchKernelGGL(k_gather_vec4, dim3(gather_blocks(total)), dim3(256), 0, stream,
                           reinterpret_cast<const float4*>(states), n_states, d / 4u, anc, total,
                           reinterpret_cast<float4*>(out));
    } else if (wide) {
        hipLaunchKernelGGL(k_gather_scalar, dim3(gather_blocks(total)), dim3(256), 0, stream, states, n_states, d, anc,
                           total, out);
    } else if (vec && total >= kGatherOneFrom && total <= kGatherOneTo) {
        launch_gather<Row4, 1>(reinterpret_cast<const Row4*>(states), n_states, d / 4u, anc, total,
                               reinterpret_cast<Row4*>(out), stream);
    } else if (vec) {
        launch_gather<Row4, 2>(reinterpret_cast<const Row4*>(states), n_states, d / 4u, anc, total,
                               reinterpret_cast<Row4*>(out), stream);
    } else if (total < kGatherFour) {
        launch_gather<float, 2>(states, n_states, d, anc, total, out, stream);
    } else {
        launch_gather<float, 4>(states, n_states, d, anc, total, out, stream);
    }
    return check_launch("gather kernel");
}

}  // namespace mgp

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
using namespace mgp;

extern "C" {

const char* mgp_last_error(void) { return g_err; }

int mgp_version(void) { return kVersion; }

int mgp_workspace_size(int32_t n, const mgp_params* params, size_t* bytes)
{
    clear_error();
    if (!bytes) return fail(MGP_EINVAL, "bytes is NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    Params p;
    int rc = normalize_params(params, &p);
    if (rc) return rc;
    *bytes = workspace_bytes((uint32_t)n, p);
    return MGP_OK;
}

// Whether n_out rows of d floats at out overlap n_in rows at in.
static bool overlaps(const float* in, int32_t n_in, const float* out, int32_t n_out, int32_t d)
{
    const uint64_t in_bytes = (uint64_t)n_in * (uint64_t)d * 4u;
    const uint64_t out_bytes = (uint64_t)n_out * (uint64_t)d * 4u;
    const uintptr_t a0 = (uintptr_t)in, a1 = a0 + in_bytes;
    const uintptr_t b0 = (uintptr_t)out, b1 = b0 + out_bytes;
    return out_bytes && a0 < b1 && b0 < a1;
}

// The row copy of the fused entry points: n rows of d floats from states to
// out; float4 moves when d % 4 == 0 and both buffers are 16-byte aligned.
static int row_copy_args(const float* states, int32_t n, int32_t d, float* out, RowCopy* rc)
{
    if (!states || !out) return fail(MGP_EINVAL, "states_dev and out_dev must not be NULL");
    if (d < 1) return fail(MGP_EINVAL, "d must be >= 1 (got %d)", d);
    if (overlaps(states, n, out, n, d)) return fail(MGP_EINVAL, "out_dev overlaps states_dev");
    rc->states = states;
    rc->out = out;
    rc->d = (uint32_t)d;
    rc->vec4 = (d % 4 == 0 && ((uintptr_t)states & 15u) == 0 && ((uintptr_t)out & 15u) == 0) ? 1u : 0u;
    return MGP_OK;
}

static int check_workspace(void* ws, size_t ws_bytes, uint32_t n, const Params& p)
{
    if (!ws) return fail(MGP_EINVAL, "workspace is NULL");
    if (((uintptr_t)ws & 255u) != 0) return fail(MGP_EINVAL, "workspace must be 256-byte aligned");
    const size_t need = workspace_bytes(n, p);
    if (ws_bytes < need) return fail(MGP_ERANGE, "workspace has %zu bytes, needs %zu", ws_bytes, need);
    return MGP_OK;
}

int mgp_compute_B(const float* w_dev, int32_t n, const mgp_params* params, mgp_stats* stats_dev,
                  void* workspace_dev, size_t workspace_bytes_, void* stream)
{
    clear_error();
    if (!w_dev) return fail(MGP_EINVAL, "w_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    Params p;
    int rc = normalize_params(params, &p);
    if (rc) return rc;
    rc = check_workspace(workspace_dev, workspace_bytes_, (uint32_t)n, p);
    if (rc) return rc;
    // a copy of the weights: the prepared loop must not see them change
    return enqueue_reduce_finalize(w_dev, (uint32_t)n, p, p.variant == kMegopolis, kLayoutCopy,
                                   static_cast<char*>(workspace_dev), stats_dev, static_cast<hipStream_t>(stream));
}

int mgp_resample_prepared(const float* w_dev, int32_t n, const mgp_params* params, int32_t* ancestors_dev,
                          void* workspace_dev, size_t workspace_bytes_, void* stream)
{
    clear_error();
    if (!w_dev || !ancestors_dev) return fail(MGP_EINVAL, "w_dev and ancestors_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    Params p;
    int rc = normalize_params(params, &p);
    if (rc) return rc;
    rc = check_workspace(workspace_dev, workspace_bytes_, (uint32_t)n, p);
    if (rc) return rc;
    return enqueue_loop(w_dev, (uint32_t)n, p, kLayoutCopy, static_cast<char*>(workspace_dev), ancestors_dev,
                        static_cast<hipStream_t>(stream));
}

int mgp_resample(const float* w_dev, int32_t n, const mgp_params* params, int32_t* ancestors_dev,
                 mgp_stats* stats_dev, void* workspace_dev, size_t workspace_bytes_, void* stream)
{
    clear_error();
    if (!w_dev || !ancestors_dev) return fail(MGP_EINVAL, "w_dev and ancestors_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    Params p;
    int rc = normalize_params(params, &p);
    if (rc) return rc;
    rc = check_workspace(workspace_dev, workspace_bytes_, (uint32_t)n, p);
    if (rc) return rc;
    return enqueue_resample(w_dev, (uint32_t)n, p, static_cast<char*>(workspace_dev), stats_dev, ancestors_dev,
                            static_cast<hipStream_t>(stream));
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Allocation-free mgp_resample: the workspace is a fixed array in the code
// object's device memory instead of a caller buffer. Each device that runs
// the library holds its own copy of it until the process ends.
// ---------------------------------------------------------------------------
static_assert(MGP_NOALLOC_SCRATCH_BYTES % 256 == 0, "the scratch size is a multiple of the workspace alignment");
static __device__ __align__(256) unsigned char scratch[MGP_NOALLOC_SCRATCH_BYTES];

namespace mgp {

constexpr int kMaxDevices = 64;

// The device address of `scratch` on the current device, looked up once per
// device (the host-side name of the array is not a device address). Null
// after a failure, with the error message set.
static void* scratch_on_current_device(int* rc)
{
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        *rc = fail(MGP_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
        return nullptr;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        *rc = fail(MGP_EINVAL, "device %d is beyond the %d devices the scratch table covers", dev, kMaxDevices);
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            *rc = fail(MGP_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
            return nullptr;
        }
        addr[dev] = p;
    }
    *rc = MGP_OK;
    return addr[dev];
}

}  // namespace mgp

extern "C" {

int mgp_resample_noalloc(const float* w_dev, int32_t n, const mgp_params* params, int32_t* ancestors_dev,
                         mgp_stats* stats_dev, void* stream)
{
    clear_error();
    if (!w_dev || !ancestors_dev) return fail(MGP_EINVAL, "w_dev and ancestors_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    Params p;
    int rc = normalize_params(params, &p);
    if (rc) return rc;
    const size_t need = workspace_bytes((uint32_t)n, p);
    if (need > (size_t)MGP_NOALLOC_SCRATCH_BYTES)
        return fail(MGP_ERANGE, "n = %d with these params needs %zu bytes of workspace; the static scratch holds %zu",
                    n, need, (size_t)MGP_NOALLOC_SCRATCH_BYTES);
    void* ws = scratch_on_current_device(&rc);
    if (!ws) return rc;
    return enqueue_resample(w_dev, (uint32_t)n, p, static_cast<char*>(ws), stats_dev, ancestors_dev,
                            static_cast<hipStream_t>(stream));
}

int mgp_resample_m(const float* w_dev, int32_t n, int32_t m, const mgp_params* params, int32_t* ancestors_dev,
                   mgp_stats* stats_dev, void* workspace_dev, size_t workspace_bytes_, void* stream)
{
    clear_error();
    if (!w_dev || !ancestors_dev) return fail(MGP_EINVAL, "w_dev and ancestors_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    if (m < 1) return fail(MGP_EINVAL, "m must be >= 1 (got %d)", m);
    Params p;
    int rc = normalize_params(params, &p);
    if (rc) return rc;
    rc = check_workspace(workspace_dev, workspace_bytes_, (uint32_t)n, p);
    if (rc) return rc;
    char* ws = static_cast<char*>(workspace_dev);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t layout = m == n ? loop_layout(w_dev, (uint32_t)n, ancestors_dev, stats_dev, RowCopy{}) : kLayoutCopy;
    rc = enqueue_reduce_finalize(w_dev, (uint32_t)n, p, p.variant == kMegopolis, layout, ws, stats_dev, s);
    if (rc) return rc;
    return enqueue_loop_m(w_dev, (uint32_t)n, (uint32_t)m, p, layout, ws, ancestors_dev, s);
}

int mgp_gather(const float* states_dev, int32_t n_states, int32_t d, const int32_t* ancestors_dev, int32_t n_out,
               float* out_dev, void* stream)
{
    clear_error();
    if (!states_dev || !ancestors_dev || !out_dev) return fail(MGP_EINVAL, "NULL pointer argument");
    if (n_states < 1 || d < 1 || n_out < 0) return fail(MGP_EINVAL, "need n_states >= 1, d >= 1, n_out >= 0");
    if (overlaps(states_dev, n_states, out_dev, n_out, d)) return fail(MGP_EINVAL, "out_dev overlaps states_dev");
    return enqueue_gather(states_dev, (uint32_t)n_states, (uint32_t)d, ancestors_dev, (uint32_t)n_out, out_dev,
                          static_cast<hipStream_t>(stream));
}

int mgp_resample_gather(const float* w_dev, int32_t n, const mgp_params* params, const float* states_dev, int32_t d,
                        int32_t* ancestors_dev, float* out_dev, mgp_stats* stats_dev, void* workspace_dev,
                        size_t workspace_bytes_, void* stream)
{
    clear_error();
    if (!w_dev) return fail(MGP_EINVAL, "w_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    RowCopy rc;
    int err = row_copy_args(states_dev, n, d, out_dev, &rc);
    if (err) return err;
    Params p;
    err = normalize_params(params, &p);
    if (err) return err;
    err = check_workspace(workspace_dev, workspace_bytes_, (uint32_t)n, p);
    if (err) return err;
    return enqueue_resample(w_dev, (uint32_t)n, p, static_cast<char*>(workspace_dev), stats_dev, ancestors_dev,
                            static_cast<hipStream_t>(stream), rc);
}

int mgp_resample_gather_prepared(const float* w_dev, int32_t n, const mgp_params* params, const float* states_dev,
                                 int32_t d, int32_t* ancestors_dev, float* out_dev, void* workspace_dev,
                                 size_t workspace_bytes_, void* stream)
{
    clear_error();
    if (!w_dev) return fail(MGP_EINVAL, "w_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    RowCopy rc;
    int err = row_copy_args(states_dev, n, d, out_dev, &rc);
    if (err) return err;
    Params p;
    err = normalize_params(params, &p);
    if (err) return err;
    err = check_workspace(workspace_dev, workspace_bytes_, (uint32_t)n, p);
    if (err) return err;
    return enqueue_loop(w_dev, (uint32_t)n, p, kLayoutCopy, static_cast<char*>(workspace_dev), ancestors_dev,
                        static_cast<hipStream_t>(stream), rc);
}

}  // extern "C"
