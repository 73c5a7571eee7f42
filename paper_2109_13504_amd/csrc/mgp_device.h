// mgp_device.h -- device-side building blocks of the resampling kernels for
// gfx950: the counter-based generator, the u and index maps, the candidate
// index of each variant, and the accept loop of one particle.
//
// Definitions (Algorithms 2-5 of "The Megopolis Resampler", arXiv 2109.13504):
//   - particle i starts at k = i and runs B steps; at step b a candidate j is
//     drawn and accepted when u * w_k <= w_j (the ratio test u <= w_j / w_k in
//     product form, evaluated in fp32, ties accept);
//   - Metropolis: j ~ U{0, N-1}; C1: j uniform in the partition the particle's
//     32-group drew once; C2: the group redraws its partition every step;
//     Megopolis: j = (i - i mod 32 + o_b - o_b mod 32 + (i + o_b) mod 32) mod N
//     with offsets o_b shared by every particle.
// Random streams: Philox4x32-10 (Salmon et al., SC'11), key = seed,
// counter = (block, tag, stream_id, index). The per-particle index sits in the
// last counter word so that the first round is wave-uniform (scalar unit)
// and rounds 2 and 3 carry one uniform multiply each.
//   tag 0: u, index i, block b/5, five u per call
//   tag 1: j, index i, block b/4, word b%4
//   tag 2: Megopolis offsets, index 0, block b/4, word b%4
//   tag 3: C1 partition, index i/32, block 0, word 0
//   tag 4: C2 partition, index i/32, block b/4, word b%4
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace mgp {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kWeyl0 = 0x9E3779B9u;
constexpr uint32_t kWeyl1 = 0xBB67AE85u;

constexpr uint32_t kTagU = 0u;
constexpr uint32_t kTagJ = 1u;
constexpr uint32_t kTagOffset = 2u;
constexpr uint32_t kTagC1Part = 3u;
constexpr uint32_t kTagC2Part = 4u;

constexpr int kMetropolis = 0;
constexpr int kC1 = 1;
constexpr int kC2 = 2;
constexpr int kMegopolis = 3;

constexpr uint32_t kSegment = 32u;  // weights per wrapped segment (the paper's warp width)

struct Words {
    uint32_t x0, x1, x2, x3;
};

// a ^ b ^ c in one VALU instruction (gfx950 three-input bitwise op, truth
// table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 on counter (c0, c1, c2, c3) with key (k0, k1). Each round
// takes both 32x32 -> 64-bit products as one v_mad_u64_u32 each. With the
// per-lane index in c3 and the other words wave-uniform, rounds 1-3 still
// hold uniform values that the compiler keeps on the scalar unit, so those
// use plain xors; from round 4 on every word is per lane and each pair of
// xors is one three-input op.
__device__ __forceinline__ Words philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                        uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;
        const uint64_t p1 = (uint64_t)kPhiloxM1 * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        uint32_t n0, n2;
        if (r < 3) {
            n0 = hi1 ^ c1 ^ k0;
            n2 = hi0 ^ c3 ^ k1;
        } else {
            n0 = xor3(hi1, c1, k0);
            n2 = xor3(hi0, c3, k1);
        }
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += kWeyl0;
        k1 += kWeyl1;
    }
    return Words{c0, c1, c2, c3};
}

// U{0, n-1} from a 32-bit word: floor(x * n / 2^32).
__device__ __forceinline__ uint32_t uniform_index(uint32_t x, uint32_t n) { return __umulhi(x, n); }

// u = (m + 1) 2^-24 for a 24-bit m; m 2^-24 + 2^-24 is exact, so the fused
// multiply-add rounds nothing.
__device__ __forceinline__ float u_from_bits(uint32_t m) { return __fmaf_rn((float)m, 0x1p-24f, 0x1p-24f); }

// The five u of one tag-0 call.
struct UBlock {
    float u[5];
};

__device__ __forceinline__ UBlock u_block(const Words& x)
{
    UBlock r;
    r.u[0] = u_from_bits(x.x0 >> 8);
    r.u[1] = u_from_bits(x.x1 >> 8);
    r.u[2] = u_from_bits(x.x2 >> 8);
    r.u[3] = u_from_bits(x.x3 >> 8);
    // the low bytes of x0, x1, x2 (in that order from the bottom) as two byte
    // permutations; shifts and masks take four instructions
    const uint32_t low2 = __builtin_amdgcn_perm(x.x1, x.x0, 0x0C0C0400u);
    r.u[4] = u_from_bits(__builtin_amdgcn_perm(x.x2, low2, 0x0C040100u));
    return r;
}

__device__ __forceinline__ uint32_t word(const Words& x, uint32_t r)
{
    return r == 0 ? x.x0 : r == 1 ? x.x1 : r == 2 ? x.x2 : x.x3;
}

// Megopolis candidate: aligned segment of i plus aligned part of o, rotated by
// (i + o) mod S inside the segment (S = seg_mask + 1, 32 or 64, a wave-uniform
// value); the sum is <= i + o <= 2N - 2, so one
// conditional subtraction is the mod N. min(j, j - n) in unsigned arithmetic
// picks j - n exactly when j >= n (n <= 2^31).
__device__ __forceinline__ uint32_t megopolis_index(uint32_t i_aligned, uint32_t i_low, uint32_t o, uint32_t n,
                                                    uint32_t seg_mask)
{
    const uint32_t j = i_aligned + (o & ~seg_mask) + ((i_low + o) & seg_mask);
    const uint32_t jm = j - n;
    return jm < j ? jm : j;
}

// Pointers read from a record in memory (a batch's filters) carry no address
// space, and the compiler then uses FLAT accesses, 64-bit vector addresses
// and, for the wave-uniform offsets, one vector load per lane. These types
// say where the data lie: HBM for weights, states and ancestors, and memory
// that is read-only during the launch, which uniform indices read through the
// scalar unit, for the offsets. On the 512-filter batch (20.7 M particles,
// 1.37e9 particle-steps) a run went from 718 to 668 us.
template <typename T>
using GlobalPtr = __attribute__((address_space(1))) T*;
using OffsetPtr = const __attribute__((address_space(4))) uint32_t*;

template <typename T>
__device__ __forceinline__ GlobalPtr<T> global_ptr(T* p)
{
    return (GlobalPtr<T>)(uintptr_t)p;
}

// A pointer known to the compiler to lie in HBM.
template <typename T>
__device__ __forceinline__ T* in_hbm(T* p)
{
    return (T*)global_ptr(p);
}

__device__ __forceinline__ OffsetPtr offset_ptr(const uint32_t* p) { return (OffsetPtr)(uintptr_t)p; }

// A position in the weights: its byte offset where that fits 32 bits (Narrow,
// n <= 2^30: the scalar-base + 32-bit vector-offset form of a load, with no
// shift left to do), else its index.
template <bool Narrow>
__device__ __forceinline__ uint32_t position(uint32_t j)
{
    return Narrow ? j << 2 : j;
}

template <bool Narrow>
__device__ __forceinline__ float load_weight(GlobalPtr<const float> w, uint32_t at)
{
    if constexpr (Narrow) {
        return *(GlobalPtr<const float>)((GlobalPtr<const char>)w + at);
    } else {
        return w[(size_t)at];
    }
}

// The same from weights kept in LDS.
template <bool Narrow>
__device__ __forceinline__ float load_weight(const float* w, uint32_t at)
{
    static_assert(Narrow, "weights in LDS are few");
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(w) + at);
}

// Per-call parameters of the accept loop (all wave-uniform). Weights is
// GlobalPtr<const float>, or const float* for weights kept in LDS.
template <typename Weights>
struct LoopParams {
    Weights w;
    OffsetPtr offsets;  // Megopolis offsets o_0..o_{B-1}, each < n
    uint32_t n;
    uint32_t B;
    uint32_t key0, key1;
    uint32_t stream_id;
    uint32_t n_w;     // C1/C2: weights per partition
    uint32_t n_part;  // C1/C2: number of partitions, ceil(n / n_w)
    uint32_t seg_mask = kSegment - 1u;  // Megopolis: segment width - 1
};

// o_b, clamped below n so that a workspace not written by this call's
// reduction can never steer a load out of bounds (wave-uniform, scalar unit).
template <typename W>
__device__ __forceinline__ uint32_t offset_at(const LoopParams<W>& P, uint32_t b)
{
    const uint32_t o = P.offsets[b];
    return o < P.n ? o : P.n - 1u;
}

// Steps per unrolled block: Megopolis needs only the 5-step u blocks; the
// others also use 4-step j blocks, so they unroll over lcm(4, 5) = 20.
template <int V>
struct Unroll {
    static constexpr uint32_t value = (V == kMegopolis) ? 5u : 20u;
};

// What a chain carries from block to block, and what is fixed for it.
struct ChainState {
    uint32_t k;  // current ancestor's position
    float wk;    // its weight
};

struct ChainFixed {
    uint32_t i;          // particle (random draws, C1/C2 group)
    uint32_t group;      // i / 32
    uint32_t i_aligned;  // Megopolis: segment base of the start position
    uint32_t i_low;      // Megopolis: place of the start position in its segment
    uint32_t c1_first;   // C1: the first weight of the group's partition
};

// The particle index as an opaque value: an empty volatile asm statement
// that the compiler may not move out of the branch it sits in, so that a
// generator call taking its result stays behind that branch's test instead
// of being computed ahead of it for steps that do not run. No instruction
// is emitted.
__device__ __forceinline__ uint32_t pinned(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// Steps q U .. q U + cnt - 1 of a chain (cnt = U for a whole block; the last
// block of B mod U steps passes Partial and its count). The candidates and
// their weights come first: they do not depend on the chain, so all of the
// block's loads are in flight together; then the serial accept steps.
// Partial skips the steps past cnt (cnt is wave-uniform), including their
// generator calls and loads.
// Even (C1, C2): n is a multiple of the partition size, so that every
// partition has the same width.
template <int V, bool Narrow, bool Shared, bool Even, bool Partial, typename W>
__device__ __forceinline__ void chain_block(const LoopParams<W>& P, const ChainFixed& F, uint32_t q, uint32_t cnt,
                                            ChainState& c)
{
    constexpr uint32_t U = Unroll<V>::value;
    constexpr bool kShare = Shared && V == kC2;
    UBlock ub;
    Words jb{}, pb{};
    uint32_t mine[4];  // kShare: the first weights of the partitions this lane drew
    uint32_t jj[U];
    float wj[U];
    if constexpr (kShare) {
        // lane k (< U / 4) of the half-wave: the call of block q U / 4 + k,
        // and the partitions of its four words, once for all 32 particles
        const uint32_t k = __lane_id() & 31u;
        const Words x = philox(q * (U / 4) + (k < U / 4 ? k : 0u), kTagC2Part, P.stream_id, F.group, P.key0, P.key1);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) mine[r] = uniform_index(word(x, r), P.n_part) * P.n_w;
    }
#pragma unroll
    for (uint32_t s = 0; s < U; ++s) {
        if (Partial && s >= cnt) continue;
        const uint32_t b = q * U + s;
        uint32_t at;
        if constexpr (V == kMegopolis) {
            at = position<Narrow>(megopolis_index(F.i_aligned, F.i_low, offset_at(P, b), P.n, P.seg_mask));
        } else {
            if (s % 4 == 0) {
                const uint32_t blk = q * (U / 4) + s / 4;
                const uint32_t pi = Partial ? pinned(F.i) : F.i;
                jb = philox(blk, kTagJ, P.stream_id, pi, P.key0, P.key1);
                if constexpr (V == kC2 && !kShare) {
                    const uint32_t pg = Partial ? pinned(F.group) : F.group;
                    pb = philox(blk, kTagC2Part, P.stream_id, pg, P.key0, P.key1);
                }
            }
            const uint32_t jw = word(jb, s % 4);
            if constexpr (V == kMetropolis) {
                at = position<Narrow>(uniform_index(jw, P.n));
            } else {
                uint32_t first;
                if constexpr (V == kC1)
                    first = F.c1_first;
                else if constexpr (kShare)
                    first = (uint32_t)__shfl((int)mine[s % 4], (int)((__lane_id() & 32u) + s / 4), 64);
                else
                    first = uniform_index(word(pb, s % 4), P.n_part) * P.n_w;
                const uint32_t rest = P.n - first;  // the last partition is cut at n
                const uint32_t width = Even || rest >= P.n_w ? P.n_w : rest;
                at = position<Narrow>(first + uniform_index(jw, width));
            }
        }
        jj[s] = at;
        wj[s] = load_weight<Narrow>(P.w, at);
    }
#pragma unroll
    for (uint32_t s = 0; s < U; ++s) {
        if (Partial && s >= cnt) continue;
        if (s % 5 == 0) {
            const uint32_t pi = Partial ? pinned(F.i) : F.i;
            ub = u_block(philox(q * (U / 5) + s / 5, kTagU, P.stream_id, pi, P.key0, P.key1));
        }
        const float p = ub.u[s % 5] * c.wk;
        const bool acc = p <= wj[s];
        c.k = acc ? jj[s] : c.k;
        c.wk = acc ? wj[s] : c.wk;
    }
}

// The B-step chain of particle i; returns its ancestor. The chain starts at
// input position pos (i itself when inputs and outputs are the same
// particles, i mod n for M != N resampling): the Megopolis segment
// arithmetic uses pos, the random draws and the C1/C2 group use i. The steps
// run in blocks of U (Unroll), the last B mod U of them as one partial block.
// Shared (C2 only): every lane of the wave runs a chain, and the 32 lanes of
// each half-wave hold the 32 particles of one group (i - lane a multiple of
// 32 within the half-wave). The group's partition draw of each step is the
// same for its 32 particles, so instead of each lane calling the generator
// once per four steps, lane k of the half-wave makes the call of the k-th
// four-step block of the block's twenty steps and the others read its words
// with a cross-lane permute: one call per lane per twenty steps.
template <int V, bool Narrow, bool Shared, bool Even, typename W>
__device__ __forceinline__ void run_blocks(const LoopParams<W>& P, const ChainFixed& F, ChainState& c)
{
    constexpr uint32_t U = Unroll<V>::value;
    const uint32_t nblk = P.B / U;
    for (uint32_t q = 0; q < nblk; ++q) chain_block<V, Narrow, Shared, Even, false>(P, F, q, U, c);
    const uint32_t rest = P.B - nblk * U;
    if (rest) chain_block<V, Narrow, Shared, Even, true>(P, F, nblk, rest, c);
}

template <int V, bool Narrow, bool Shared = false, typename W>
__device__ __forceinline__ uint32_t run_chain(const LoopParams<W>& P, uint32_t i, uint32_t pos)
{
    ChainFixed F;
    F.i = i;
    F.group = i / kSegment;
    F.i_aligned = pos & ~P.seg_mask;
    F.i_low = pos & P.seg_mask;
    F.c1_first = 0;
    if constexpr (V == kC1) {
        const Words px = philox(0u, kTagC1Part, P.stream_id, F.group, P.key0, P.key1);
        F.c1_first = uniform_index(px.x0, P.n_part) * P.n_w;
    }
    ChainState c{position<Narrow>(pos), load_weight<Narrow>(P.w, position<Narrow>(pos))};
    if constexpr (V == kC1 || V == kC2) {
        if (P.n_part * P.n_w == P.n)
            run_blocks<V, Narrow, Shared, true>(P, F, c);
        else
            run_blocks<V, Narrow, Shared, false>(P, F, c);
    } else {
        run_blocks<V, Narrow, Shared, true>(P, F, c);
    }
    return Narrow ? c.k >> 2 : c.k;
}

template <int V, bool Narrow, bool Shared = false, typename W>
__device__ __forceinline__ uint32_t run_chain(const LoopParams<W>& P, uint32_t i)
{
    return run_chain<V, Narrow, Shared>(P, i, i);
}

// ---------------------------------------------------------------------------
// Megopolis by windows of consecutive weights.
//
// A block's T particles start at a multiple of the segment width S, so at a
// step with offset o their candidates (i_aligned + o_aligned + (i + o) mod S)
// mod N (Algorithm 5) are the T consecutive positions from
// s = (start + o_aligned) mod N on, permuted inside segments. s is the same
// for the whole block, so the mod N is one scalar compare and subtraction per
// step, and only a window that runs past the end of the weights needs care:
// it is read from the seam, a copy of the last and first kSeam weights one
// after the other, and every other window from the caller's weights as they
// lie. Each thread carries P particles BT apart that share one vector offset;
// their loads differ only in the immediate byte offset (4 BT p).
//
// The caller's weights are read in place when they are 128-byte aligned (a
// 32-weight segment is then one cache line; elsewhere it would straddle two,
// three lines per wave and step instead of two) and no output overlaps them.
// Otherwise, and for mgp_compute_B, the reduction makes a copy of n + kSeam
// weights, the first kSeam repeated at the end, which serves every window. A
// prepared loop must not see weights changed since: it always reads that copy,
// which a single filter's loop in place completes from the weights it holds
// anyway (`keep`: 4 bytes per weight written past the L2). Against the earlier
// copy M[k] = w[k mod n], k < 2n, for every call, reading in place saves 8 of
// the reduction's 12 bytes per weight (2^24 weights: 13 against 34 us) and
// halves what the loop's reads spread over (a run of the 512-filter batch 668
// to 626 us, an SIR step of 64 x 2^20 particles 1106 to 1043).
//
// Where n is no multiple of 32, a window that wraps begins n mod 32 weights off
// a cache line, and each of its waves reads three lines per step instead of two:
// about half of all windows. From kTailMinN weights and kTailMinSteps particle-
// steps on that costs more than writing the weights once more, as a tail:
// copy[n + k] = w[k mod n], k < n + kSeam. Windows then do not wrap but run on
// past n, from multiples of the segment width. Whole calls, us, without / with a tail: 2^22 + 13, B = 200
// 375 / 378, B = 354 663 / 644; 6 000 001, B = 100 304 / 313, B = 200 561 / 545,
// B = 354 1007 / 943; 15 000 001, B = 64 537 / 540, B = 100 817 / 807, B = 354
// 2950 / 2660; 3 000 001 (12 MB) never gains.
// Byte offsets must fit 32 bits: 4 (2n + 2 kSeam) < 2^32.
// ---------------------------------------------------------------------------
constexpr uint32_t kSeam = 1024;                  // particles per block at most
constexpr uint32_t kWindowMaxN = (1u << 29) - 4096;
constexpr uint32_t kLayoutInPlace = 1u, kLayoutCopy = 2u;  // where the windows lie
constexpr uint32_t kTailMinN = 1u << 21;
constexpr uint64_t kTailMinSteps = 1ull << 30;

// Whether a loop of B steps over n weights has a tail.
__host__ __device__ __forceinline__ bool has_tail(uint32_t n, uint32_t B)
{
    return n > kTailMinN && n % 32u != 0 && (uint64_t)n * B >= kTailMinSteps;
}

// Byte addresses of the weights: position k of a window that starts at s is at
// (s + T <= n ? w : seam) + 4 k.
struct Windows {
    uint64_t w, seam;
};

__host__ __device__ __forceinline__ Windows windows_in_place(const float* w, const float* seam, uint32_t n)
{
    return Windows{(uint64_t)(uintptr_t)w, (uint64_t)(uintptr_t)seam + 4u * (uint64_t)kSeam - 4u * (uint64_t)n};
}

__host__ __device__ __forceinline__ Windows windows_copy(const float* copy)
{
    return Windows{(uint64_t)(uintptr_t)copy, (uint64_t)(uintptr_t)copy};
}

__device__ __forceinline__ GlobalPtr<const char> window_at(const Windows& W, uint32_t s, uint32_t n, uint32_t tile)
{
    return (GlobalPtr<const char>)((s + tile <= n ? W.w : W.seam) + 4u * (uint64_t)s);
}

// s = (start + o_aligned) mod n for start < n, o < n.
__device__ __forceinline__ uint32_t window_start(uint32_t start, uint32_t o, uint32_t seg_mask, uint32_t n)
{
    const uint32_t s = start + (o & ~seg_mask);
    return s >= n ? s - n : s;
}

// The seam of w: seam[k] = w[(n - kSeam + k) mod n], k < 2 kSeam (one block
// writes it).
__device__ __forceinline__ void write_seam(const float* __restrict__ w, uint32_t n, float* __restrict__ seam)
{
    if (n >= kSeam) {  // no division in the usual case
        for (uint32_t k = threadIdx.x; k < 2u * kSeam; k += blockDim.x)
            seam[k] = w[k < kSeam ? n - kSeam + k : k - kSeam];
    } else {
        const uint32_t shift = n - kSeam % n;
        for (uint32_t k = threadIdx.x; k < 2u * kSeam; k += blockDim.x) seam[k] = w[(k + shift) % n];
    }
}

// Completes the copy behind a loop in place: the weight of particle i, unless
// the reduction has written it as part of the seam (n >= kSeam).
__device__ __forceinline__ void keep_weight(float* keep, uint32_t n, uint32_t i, float w)
{
    if (i < n - kSeam) __builtin_nontemporal_store(w, global_ptr(keep) + i);
}

// What the rounds of a thread's chains share (wave-uniform but the last two).
struct WindowLoop {
    Windows W;
    OffsetPtr offs;
    uint32_t key0, key1, stream_id;
    uint32_t start;     // the block's first particle
    uint32_t last;      // n - 1
    uint32_t start4, wrap4, mask4;  // start, the place where windows wrap (n, or none) and the segment mask in bytes
    uint32_t lim4;      // windows that start below it lie in W.w
    uint32_t la4, ll4;  // byte offset of the thread's segment in the window, and of its place in the segment
};

// Steps b0 .. b0 + D - 1 (Partial: b0 .. b0 + cnt - 1), b0 = 5 blk, of
// the chains of particles p0 .. p0 + G - 1 of a thread: candidate loads first
// (they do not depend on the chain), then the draws, then the serial accept
// steps. A step's window takes ten or eleven scalar instructions, all in bytes:
// window_start and window_at, with (i + o) mod S from the unmasked o. Written
// with indices they were 17, and where few waves are in flight a wave's
// instructions are what a step costs. us, then / now: 300 filters of 2^8 to
// 2^12 particles 38.1 / 36.0 (256 x 1) and 65 / 61 (64 x 4); 600 of 2^9 to 2^14
// 98 / 90 (256 x 1); a prepared loop of 100003 particles, B = 354, 38.5 / 32.5.
// Checked: an offset of n or more (a workspace not written by this call) is
// clamped, so that it cannot steer a load out of bounds.
template <int P, int BT, int G, int D, bool Partial, bool Checked>
__device__ __forceinline__ void window_round(const WindowLoop& L, uint32_t blk, uint32_t cnt, int p0,
                                             uint32_t (&kk)[P], float (&wk)[P])
{
    static_assert(D % 5 == 0, "a round covers whole blocks of five u draws");
    const OffsetPtr offs = L.offs + 5u * blk;
    const uint32_t i0 = L.start + threadIdx.x;
    uint32_t o[D];
    uint32_t jb[D];
    float wj[D][G];
#pragma unroll
    for (uint32_t s = 0; s < D; ++s) {
        if (s % 5u == 0) {
            // five offsets at once, not one round trip per step behind its branch
            if (Partial && s >= cnt) continue;
#pragma unroll
            for (uint32_t r = s; r < s + 5u; ++r) o[r] = offs[!Partial || r < cnt ? r : cnt - 1u];
        }
        if (Partial && s >= cnt) continue;
        const uint32_t o4 = (!Checked || o[s] < L.last ? o[s] : L.last) * 4u;
        const uint32_t s4 = L.start4 + (o4 & ~L.mask4), s4n = s4 - L.wrap4;
        const uint32_t at4 = s4 < s4n ? s4 : s4n;  // the difference wraps round below wrap4
        const uint32_t voff = L.la4 | ((L.ll4 + o4) & L.mask4);
        const GlobalPtr<const char> base = (GlobalPtr<const char>)((at4 < L.lim4 ? L.W.w : L.W.seam) + at4);
#pragma unroll
        for (int q = 0; q < G; ++q) wj[s][q] = *(GlobalPtr<const float>)(base + voff + 4u * BT * (p0 + q));
        jb[s] = voff + at4;
    }
#pragma unroll
    for (uint32_t g = 0; g < D / 5; ++g) {
        if (Partial && g * 5u >= cnt) continue;
        UBlock ub[G];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const uint32_t i = (Partial && D > 5) ? pinned(i0 + BT * (p0 + q)) : i0 + BT * (p0 + q);
            ub[q] = u_block(philox(blk + g, kTagU, L.stream_id, i, L.key0, L.key1));
        }
#pragma unroll
        for (uint32_t s = 0; s < 5; ++s) {
            if (Partial && g * 5u + s >= cnt) continue;
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const float prod = ub[q].u[s] * wk[p0 + q];
                const bool acc = prod <= wj[g * 5 + s][q];
                kk[p0 + q] = acc ? jb[g * 5 + s] : kk[p0 + q];
                wk[p0 + q] = acc ? wj[g * 5 + s][q] : wk[p0 + q];
            }
        }
    }
}

// The B-step chains of a thread's particles start + threadIdx.x + BT p, p < P
// (lanes past n run too and return some ancestor), in rounds of D steps. With
// keep, the weights before the seam also go to keep[i]. tail: the windows run on
// past n (has_tail). Checked: as above.
template <int P, int BT, int D, bool Checked>
__device__ __forceinline__ void megopolis_chain(const Windows& W, OffsetPtr offs, uint32_t n, uint32_t B,
                                                uint32_t key0, uint32_t key1, uint32_t stream_id, uint32_t start,
                                                uint32_t (&anc_out)[P], uint32_t seg_mask = kSegment - 1u,
                                                float* keep = nullptr, bool tail = false)
{
    static_assert(BT % 64 == 0 && BT * P <= (int)kSeam, "a block's window must fit the seam");
    static_assert(4 * BT * (P - 1) < 4096, "the immediate offset of the last particle must fit 12 bits");
    // Particles whose loads and draws are in flight together. Eight at once
    // would take 190 registers (two waves per SIMD); in pairs, kept apart by
    // scheduling barriers, 82.
    constexpr int G = P == 8 ? 2 : P;
    const uint32_t t = threadIdx.x;
    const WindowLoop L{W,          offs,   key0,          key1,
                       stream_id,  start,  n - 1u,        start * 4u,
                       tail ? ~0u : n * 4u, seg_mask * 4u,         n >= (uint32_t)(P * BT) ? (n - P * BT) * 4u + 1u : 0u,
                       (t & ~seg_mask) * 4u, (t & seg_mask) * 4u};
    uint32_t kk[P];  // ancestor as the byte offset of particle 0's position
    float wk[P];
    const GlobalPtr<const char> own = window_at(W, start, n, P * BT);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        kk[p] = (start + t) * 4u;
        wk[p] = *(GlobalPtr<const float>)(own + t * 4u + 4u * BT * p);
    }
    if (keep) {
#pragma unroll
        for (int p = 0; p < P; ++p) keep_weight(keep, n, start + t + BT * p, wk[p]);
    }
    uint32_t blk = 0;
    for (; 5u * blk + (uint32_t)D <= B; blk += D / 5) {
#pragma unroll
        for (int p0 = 0; p0 < P; p0 += G) {
            window_round<P, BT, G, D, false, Checked>(L, blk, D, p0, kk, wk);
            if (P > G) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (5u * blk < B) {
#pragma unroll
        for (int p0 = 0; p0 < P; p0 += G) {
            window_round<P, BT, G, D, true, Checked>(L, blk, B - 5u * blk, p0, kk, wk);
            if (P > G) __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t k = kk[p] / 4u + BT * p;
        anc_out[p] = k >= n ? k - n : k;
    }
}

// ---------------------------------------------------------------------------
// The particle copy that closes Algorithms 2-5, x_bar_i = x_{k_i}: rows of d
// fp32 states, row-major, streamed to the output past the L2 (written once,
// never read here). The accept loops run it as an epilogue while the
// ancestors are still in registers; the stand-alone gather runs it over an
// ancestor array. A negative ancestor (invalid weights) gives a NaN row.
// ---------------------------------------------------------------------------
struct RowCopy {
    const float* states;  // input rows; null: nothing is copied
    float* out;           // one row per output particle
    uint32_t d;           // floats per row
    uint32_t vec4;        // d % 4 == 0 and both buffers 16-byte aligned: float4 moves
};

using Row4 = float __attribute__((ext_vector_type(4)));

__device__ __forceinline__ Row4 nan_row4() { return Row4{NAN, NAN, NAN, NAN}; }

// Output row i from input row k, one lane, any d: up to four vectors (or
// four floats) loaded before the first of them is stored, so a row of up to
// 16 floats costs one round trip.
__device__ __forceinline__ void copy_row(const RowCopy& g, uint32_t i, int32_t k)
{
    const uint64_t kr = k < 0 ? 0u : (uint64_t)k;
    if (g.vec4) {
        const uint32_t d4 = g.d >> 2;
        const GlobalPtr<const Row4> src = global_ptr(reinterpret_cast<const Row4*>(g.states)) + kr * d4;
        const GlobalPtr<Row4> dst = global_ptr(reinterpret_cast<Row4*>(g.out)) + (uint64_t)i * d4;
        for (uint32_t c = 0; c < d4; c += 4u) {
            Row4 v[4];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
                if (c + u < d4) v[u] = k < 0 ? nan_row4() : src[c + u];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
                if (c + u < d4) __builtin_nontemporal_store(v[u], dst + c + u);
        }
    } else {
        const GlobalPtr<const float> src = global_ptr(g.states) + kr * g.d;
        const GlobalPtr<float> dst = global_ptr(g.out) + (uint64_t)i * g.d;
        for (uint32_t c = 0; c < g.d; c += 4u) {
            float v[4];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
                if (c + u < g.d) v[u] = k < 0 ? NAN : src[c + u];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
                if (c + u < g.d) __builtin_nontemporal_store(v[u], dst + c + u);
        }
    }
}

// The rows of P outputs of one lane, D4 float4s per row known at compile time
// (g.vec4 set): the loads of G rows are issued before the first of their
// stores. Outputs with live[p] false are skipped.
template <int P, int D4, int G = P>
__device__ __forceinline__ void copy_rows_vec4(const RowCopy& g, const uint32_t (&i)[P], const int32_t (&k)[P],
                                               const bool (&live)[P])
{
    static_assert(P % G == 0, "whole groups");
    const GlobalPtr<const Row4> src = global_ptr(reinterpret_cast<const Row4*>(g.states));
    const GlobalPtr<Row4> dst = global_ptr(reinterpret_cast<Row4*>(g.out));
#pragma unroll
    for (int p0 = 0; p0 < P; p0 += G) {
        Row4 v[G][D4];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int p = p0 + q;
            const uint64_t kr = k[p] < 0 ? 0u : (uint64_t)k[p];
#pragma unroll
            for (int c = 0; c < D4; ++c)
                if (live[p]) v[q][c] = k[p] < 0 ? nan_row4() : src[kr * D4 + c];
        }
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int p = p0 + q;
#pragma unroll
            for (int c = 0; c < D4; ++c)
                if (live[p]) __builtin_nontemporal_store(v[q][c], dst + (uint64_t)i[p] * D4 + c);
        }
    }
}

// The rows of P outputs of one lane, row shape known at run time, in groups
// of at most four rows and eight vectors in flight, kept apart by scheduling
// barriers: eight particles' rows at once would take 190 registers, two waves
// per SIMD for the whole kernel.
template <int P>
__device__ __forceinline__ void copy_rows(const RowCopy& g, const uint32_t (&i)[P], const int32_t (&k)[P],
                                          const bool (&live)[P])
{
    constexpr int G = P < 4 ? P : 4;
    const GlobalPtr<const float> src = global_ptr(g.states);
    const GlobalPtr<float> dst = global_ptr(g.out);
#pragma unroll
    for (int p0 = 0; p0 < P; p0 += G) {
        uint32_t ii[G];
        int32_t kg[G];
        bool lg[G];
#pragma unroll
        for (int q = 0; q < G; ++q) {
            ii[q] = i[p0 + q];
            kg[q] = k[p0 + q];
            lg[q] = live[p0 + q];
        }
        if (g.vec4 && g.d == 4u) {
            copy_rows_vec4<G, 1>(g, ii, kg, lg);
        } else if (g.vec4 && g.d == 8u) {
            copy_rows_vec4<G, 2>(g, ii, kg, lg);
        } else if (g.d == 1u) {
            float v[G];
#pragma unroll
            for (int q = 0; q < G; ++q)
                if (lg[q]) v[q] = kg[q] < 0 ? NAN : src[(uint32_t)kg[q]];
#pragma unroll
            for (int q = 0; q < G; ++q)
                if (lg[q]) __builtin_nontemporal_store(v[q], dst + ii[q]);
        } else {
#pragma unroll
            for (int q = 0; q < G; ++q) {
                if (lg[q]) copy_row(g, ii[q], kg[q]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (P > G) __builtin_amdgcn_sched_barrier(0);
    }
}

}  // namespace mgp
