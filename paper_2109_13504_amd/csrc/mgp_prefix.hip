// mgp_prefix.hip -- the prefix-sum resamplers of the C ABI (include/mgp.h):
// multinomial (Algorithm 7) and systematic (Algorithm 8) resampling, the
// unbiased comparison methods of Section 6.5 and Table 2.
//
// Both give output i the first input j whose inclusive prefix sum of weights
// exceeds a threshold t_i (multinomial: an independent uniform t_i per
// output; systematic: t_i = (i + u) S / N from one uniform u). The weights
// enter the prefix sum as 64-bit fixed point, q = floor(w 2^K), with K from
// the largest weight such that the total S stays below 2^62: integer sums are
// exact in any order, so the parallel scan here and a sequential sum give the
// same prefix and the same ancestors.
//
// The search runs down a 16-ary tree of exclusive sums: level 1 holds the sum
// before every group of 16 inputs, level k that before every 16^k inputs, and
// the top is the first level of at most 2048 entries, which a block keeps in
// LDS. The sums inside a group are not stored: the search adds up the group's
// own 64 bytes of weights. A level of 8 bytes per input would be 16 times
// level 1 (128 of 136 MB at 2^24), written once and read for the last line of
// every descent; this way the scan works on 0.5 byte per input and the last
// line comes from the weights.
//
// Launches, after the reduction of the other resamplers (validation, max,
// fp64 sum):
//   k_prefix_groups   per 1, 4 or 16 chunks of 2048 weights: the fixed-point sum
//                     of each group, and of them all; for a single filter its
//                     blocks also do the finalize step over the reduction's
//                     partials
//   k_prefix_scan     per 2048 groups: the levels' exclusive sums, the header
//                     (up to 32768 inputs the search's blocks do it instead)
//   k_prefix_multinomial   a descent per output, four lanes to a row
//   k_prefix_systematic    1792 outputs per block, whose inputs (thresholds rise
//                     with i) mark in LDS the first output that each of them has
// Whole calls, us, with a level of sums per input and six or seven launches /
// now: multinomial 10^3 19 / 11, 2^16 22 / 17, 2^20 54 / 39, 2^24 626 / 571;
// systematic 10^3 20 / 14, 2^16 24 / 17, 10^7 107 / 58, 2^24 154 / 81, 2^28
// 2551 / 1250. Systematic's search by bisection in LDS, eleven reads and
// 64-bit compares per output, took 44 us of 10^7's 75; the marks take 28.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "mgp.h"
#include "mgp_device.h"
#include "mgp_internal.h"
#include "mgp_prefix.h"
#include "mgp_reduce.h"

namespace mgp {

constexpr uint32_t kPrefixThreads = 256;
constexpr uint32_t kPrefixPer = 8;                        // weights per thread in a chunk
constexpr uint32_t kChunk = kPrefixThreads * kPrefixPer;  // 2048 weights per chunk
constexpr uint32_t kFan = 16;                             // the tree's fan-out: one 128-byte row of sums
constexpr uint32_t kTopMax = 2048;                        // entries of the top level, kept in LDS (16 KB)
constexpr uint32_t kScanGroups = kPrefixThreads * 8;      // groups per block of the scan
constexpr uint32_t kChunksPerScan = kScanGroups * kFan / kChunk;
// Chunks per block of the first kernel: every block of the scan adds up the
// sums that it leaves, so there are to be few of them, and still enough blocks.
// Systematic, us, 1 chunk / 4 / 16: 2^22 41 / 39 / -, 10^7 66 / 64 / -, 2^28
// 1629 / - / 1253, 2^29 4145 / - / 2516.
constexpr uint32_t chunks_per_block(uint32_t n) {  return n < (1u << 22) ? 1u : n < (1u << 25) ? 4u : 16u; }
constexpr uint32_t kTagMultinomial = 6u;
constexpr uint32_t kTagSystematic = 7u;

// What the scan leaves for the search (in the workspace).
struct PrefixHeader {
    uint64_t total;  // S, the sum of the fixed-point weights (0: invalid weights)
    int32_t K;       // the fixed-point exponent
    int32_t valid;   // 1 when the weights passed validation
};

template <typename T>
__device__ __forceinline__ T* at(const PrefixJob& J, uint64_t off)
{
    return reinterpret_cast<T*>(J.region + (uint64_t)blockIdx.y * J.region_ld + off);
}

// K = 62 - ceil(log2 n) - E for w_max = m 2^E, m in [0.5, 1).
__device__ __forceinline__ int fixed_exponent(float w_max, int log2n_ceil)
{
    int E = 0;
    frexp((double)w_max, &E);
    return 62 - log2n_ceil - E;
}

// q = floor(w 2^K) for a finite w >= 0 with q < 2^62, given scale = 2^(K - 32):
// y = w 2^(K - 32) is exact in fp64 (24 bits; K - 32 is between -129 and 178),
// its integer part is the high word and its fraction times 2^32, cut off, the
// low word.
__device__ __forceinline__ uint64_t fixed_weight(float w, double scale)
{
    const double y = (double)w * scale;
    const uint32_t hi = (uint32_t)y;
    const uint32_t lo = (uint32_t)(__builtin_amdgcn_fract(y) * 0x1p32);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

__device__ __forceinline__ double fixed_scale(float w_max, int log2n_ceil)
{
    return ldexp(1.0, fixed_exponent(w_max, log2n_ceil) - 32);
}

// Block-wide exclusive scan of one uint64 per thread; returns the thread's
// exclusive prefix and the block total through *total.
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t* total)
{
    __shared__ uint64_t wave_sums[kPrefixThreads / 64];
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
    uint64_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(x, off, 64);
        if ((int)lane >= off) x += y;
    }
    if (lane == 63u) wave_sums[wv] = x;
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPrefixThreads / 64; ++k) {
        const uint64_t s = wave_sums[k];
        if (k < wv) before += s;
        all += s;
    }
    __syncthreads();  // wave_sums is reused by the next call
    *total = all;
    return before + x - v;
}

// The fixed-point weights of the Per consecutive inputs from `base` on (0 past
// n; Per and base multiples of 4). Whole: base + Per <= n is known.
template <int Per, bool Whole>
__device__ __forceinline__ void load_fixed(const PrefixJob& J, uint64_t base, double scale, uint64_t (&q)[Per])
{
    const GlobalPtr<const float> w = global_ptr(J.w + (uint64_t)blockIdx.y * J.w_ld);
    float v[Per];
    if (Whole) {
#pragma unroll
        for (int e = 0; e < Per; e += 4) {
            const Row4 x = *(GlobalPtr<const Unaligned4>)(w + base + e);
#pragma unroll
            for (int c = 0; c < 4; ++c) v[e + c] = x[c];
        }
    } else {
#pragma unroll
        for (int e = 0; e < Per; ++e) v[e] = base + e < J.n ? w[base + e] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < Per; ++e) q[e] = fixed_weight(v[e], scale);
}

// The same for a block whose threads read Per inputs each from `first` on, one
// after the other: all of them inside n, or each checked.
template <int Per>
__device__ __forceinline__ void load_fixed_tile(const PrefixJob& J, uint64_t first, double scale, uint64_t (&q)[Per])
{
    const uint64_t base = first + (uint64_t)threadIdx.x * Per;
    if (first + (uint64_t)Per * kPrefixThreads <= J.n)
        load_fixed<Per, true>(J, base, scale, q);
    else
        load_fixed<Per, false>(J, base, scale, q);
}

// The sums of the groups of J.per chunks (in level 1's place) and of all of
// them together. Fin: the finalize step of the call comes first, in every
// block.
template <bool Fin>
__global__ __launch_bounds__(kPrefixThreads) void k_prefix_groups(PrefixJob J)
{
    mgp_stats st;
    if constexpr (Fin) {
        __shared__ mgp_stats st_local;
        finalize_one<true>(J.parts, J.nparts, J.fin, &st_local, blockIdx.x == 0 ? J.st_user : nullptr, nullptr);
        if (blockIdx.x == 0 && threadIdx.x == 0) *J.stats = st_local;
        st = st_local;
    } else {
        st = J.stats[blockIdx.y];
    }
    if (st.status != MGP_OK) return;
    const double scale = fixed_scale(st.w_max, J.log2n);
    uint64_t all = 0;
    for (uint32_t p = 0; p < J.per; ++p) {
        const uint32_t chunk = blockIdx.x * J.per + p;
        uint64_t q[kPrefixPer];
        load_fixed_tile(J, (uint64_t)chunk * kChunk, scale, q);
        uint64_t s = 0;
#pragma unroll
        for (uint32_t e = 0; e < kPrefixPer; ++e) s += q[e];
        // two threads hold a group
        const uint64_t both = s + (uint64_t)__shfl_xor((unsigned long long)s, 1, 64);
        const uint64_t g = (uint64_t)chunk * (kChunk / kFan) + threadIdx.x / 2u;
        if (threadIdx.x % 2u == 0 && g < J.count[1]) at<uint64_t>(J, J.o_level[1])[g] = both;
        all += s;
    }
    uint64_t total = 0;
    block_exclusive_scan(all, &total);
    if (threadIdx.x == 0) at<uint64_t>(J, J.o_sum)[blockIdx.x] = total;
}

// Algorithm 8: u = (i + u_t) / N after one draw u_t ~ U[0, 1) per run, in fp64
// with each operation rounded once.
struct SystematicDraw {
    double ut, c;  // u_t, S / N
    double c32;    // c / 2^32
    double inv;    // N / S
    uint64_t S;

    __device__ __forceinline__ SystematicDraw(const PrefixJob& J, uint64_t total) : S(total)
    {
        const Words x = philox(0u, kTagSystematic, J.stream0 + blockIdx.y, 0u, J.key0, J.key1);
        const uint64_t r = (uint64_t)x.x0 | ((uint64_t)x.x1 << 32);
        ut = (double)(r >> 11) * 0x1p-53;
        c = __ddiv_rn((double)S, (double)J.n);
        c32 = c * 0x1p-32;
        inv = __ddiv_rn((double)J.n, (double)S);
    }

    // rises with i
    __device__ __forceinline__ uint64_t threshold(uint32_t i) const
    {
        const uint64_t t = (uint64_t)floor(__dmul_rn(__dadd_rn((double)i, ut), c));
        return t < S ? t : S - 1u;
    }

    // The number of outputs whose threshold is below P (0 <= P <= S), so the
    // first output of the input that starts at P; N or N + 1 when P = S.
    // P N / S - u_t is that crossing to within 2^-18 (each operation, here and in
    // threshold(), is off by 2^-53 of at most 2^31), so only the output nearest
    // to it has to be asked: those before are below P, those after are not. Its
    // threshold is compared as integers, high and low word (c32 scales by a
    // power of two, which rounds nothing), and those that threshold() holds at
    // S - 1 are not below P unless P = S.
    __device__ __forceinline__ uint32_t outputs_below(uint64_t P) const
    {
        const double f = fmax(rint(fma((double)P, inv, -ut)), 0.0);
        const double x = __dmul_rn(__dadd_rn(f, ut), c32);
        const uint32_t hi = (uint32_t)x;
        const uint32_t lo = (uint32_t)(__builtin_amdgcn_fract(x) * 0x1p32);
        const uint64_t t = (uint64_t)lo | ((uint64_t)hi << 32);
        return (uint32_t)f + (t >= P && P < S ? 0u : 1u);
    }
};

// The systematic search: kSysOut outputs per block, of up to kSysTiles tiles of inputs.
constexpr uint32_t kSysPer = 7;
constexpr uint32_t kSysOut = kSysPer * kPrefixThreads;
constexpr uint32_t kSysTiles = 8;

// The exclusive sums of kScanGroups groups, from the chunks' sums before them
// and the groups' own sums, which they replace; the entries of the higher
// levels among them; and, by the block with the last group, every level's
// padding (the largest integer, above any threshold) and the header.
//
// Sys: also where the blocks of the systematic search start. The thread with
// the sum before a group has the first output there (outputs_below), so
// start[b], the group of output b kSysOut, is written by the thread whose group
// has it: about one in 100 of them, against a search from the top of the tree
// at the start of every block. Where a few groups have nearly all outputs, their
// starts lie in a few waves, which write them side by side: sorted weights of
// y = 4, us when a wave wrote one run after the other / now: 2^20 20.5 / 6.9, 2^24
// 37.7 / 11.6.
template <bool Sys>
__global__ __launch_bounds__(kPrefixThreads) void k_prefix_scan(PrefixJob J)
{
    const mgp_stats& st = J.stats[blockIdx.y];
    const bool last = blockIdx.x == gridDim.x - 1u;
    uint64_t* x1 = at<uint64_t>(J, J.o_level[1]);
    const uint32_t g0 = blockIdx.x * kScanGroups + threadIdx.x * 8u;
    uint64_t v[8];
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) v[e] = g0 + e < J.count[1] ? x1[g0 + e] : 0u;
    const uint64_t* sums = at<uint64_t>(J, J.o_sum);
    const uint32_t own = blockIdx.x * (kChunksPerScan / J.per);  // the first sum of this block
    uint64_t before = 0, after = 0;
#pragma unroll 8
    for (uint32_t c = threadIdx.x; c < (Sys ? J.nsum : own); c += kPrefixThreads) {
        const uint64_t x = sums[c];
        before += c < own ? x : 0u;
        after += c < own ? 0u : x;
    }
    // after the loads, which are in bounds whatever it says: one round trip
    // less (2^17 17.1 to 16.6 us, 2^20 38.1 to 37.7, multinomial)
    if (st.status != MGP_OK) {
        if (last && threadIdx.x == 0) *at<PrefixHeader>(J, J.o_hdr) = PrefixHeader{0u, 0, 0};
        return;
    }
    uint64_t base = 0, total = 0, S = 0;
    block_exclusive_scan(before, &base);
    if constexpr (Sys) {
        block_exclusive_scan(after, &S);
        S += base;
    }
    uint64_t s = 0;
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) s += v[e];
    uint64_t run = base + block_exclusive_scan(s, &total);
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) {
        if (g0 + e < J.count[1]) {
            // level k entry m is the sum before input m 16^k
            uint32_t g = g0 + e;
            for (int k = 1; k <= J.top; ++k) {
                at<uint64_t>(J, J.o_level[k])[g] = run;
                if (g % kFan != 0u) break;
                g /= kFan;
            }
        }
        run += v[e];
    }
    if constexpr (Sys) {
        const SystematicDraw draw(J, S);
        uint32_t* start = at<uint32_t>(J, J.o_start);
        const uint32_t lane = threadIdx.x & 63u;
        run -= s;
        uint32_t from = (draw.outputs_below(run) + kSysOut - 1u) / kSysOut;
#pragma unroll
        for (uint32_t e = 0; e < 8u; ++e) {
            // blocks [from, to) start in group g0 + e; the last group with a
            // weight also ends the last block's range
            run += v[e];
            const uint32_t below = draw.outputs_below(run);
            const bool ends = run == S && v[e] > 0u;
            const uint32_t to = ends ? J.nsys + 1u : ((below < J.n ? below : J.n) + kSysOut - 1u) / kSysOut;
            // two by the thread itself, which is all where no group has the
            // outputs of three blocks; the rest of a long run by its wave
            if (from < to) start[from] = g0 + e;
            if (from + 1u < to) start[from + 1u] = g0 + e;
            uint64_t mask = __ballot(from + 2u < to);
            while (mask) {
                const int l = __ffsll((unsigned long long)mask) - 1;
                mask &= mask - 1u;
                const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)from, l) + 2u;
                const uint32_t z = (uint32_t)__builtin_amdgcn_readlane((int)to, l);
                const uint32_t g = (uint32_t)__builtin_amdgcn_readlane((int)(g0 + e), l);
                for (uint32_t b = a + lane; b < z; b += 64u) start[b] = g;
            }
            from = to;
        }
    }
    if (last) {
        for (int k = 1; k <= J.top; ++k) {
            const uint32_t end = (J.count[k] + kFan - 1u) / kFan * kFan;
            const uint32_t m = J.count[k] + threadIdx.x;
            if (m < end) at<uint64_t>(J, J.o_level[k])[m] = ~(uint64_t)0;
        }
        if (threadIdx.x == 0)
            *at<PrefixHeader>(J, J.o_hdr) = PrefixHeader{base + total, fixed_exponent(st.w_max, J.log2n), 1};
    }
}

// Algorithm 7: the threshold of output i of run r, u ~ U[0, S), one 64-bit draw
// per output.
__device__ __forceinline__ uint64_t multinomial_threshold(const PrefixJob& J, uint64_t S, uint32_t i)
{
    const Words x = philox(0u, kTagMultinomial, J.stream0 + blockIdx.y, i, J.key0, J.key1);
    const uint64_t r = (uint64_t)x.x0 | ((uint64_t)x.x1 << 32);
    return __umul64hi(r, S);
}

// Output i of run r: the ancestor and, when the job copies rows, the row
// (a NaN row for invalid weights, a = -1).
__device__ __forceinline__ void emit(const PrefixJob& J, uint32_t i, int32_t a)
{
    const uint64_t r = blockIdx.y;
    if (J.anc) J.anc[r * J.anc_ld + i] = a;
    if (J.states) {
        const RowCopy rc{J.states + r * J.rows_ld, J.out + r * J.rows_ld, J.d, J.vec4};
        copy_row(rc, i, a);
    }
}

using U64x2 = uint64_t __attribute__((ext_vector_type(2)));

// For up to kTopMax groups (32768 inputs), whose level 1 is the top: the scan
// of the groups' sums in LDS by the block that searches them, so that
// k_prefix_scan's launch goes. top[g] is the sum before group g, the largest
// integer from the last group to kTopMax.
__device__ __forceinline__ PrefixHeader scan_in_lds(const PrefixJob& J, uint64_t* top)
{
    const mgp_stats& st = J.stats[blockIdx.y];
    if (st.status != MGP_OK) return PrefixHeader{0u, 0, 0};
    const uint64_t* x1 = at<uint64_t>(J, J.o_level[1]);
    const uint32_t g0 = threadIdx.x * 8u;
    uint64_t v[8], s = 0, total = 0;
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) v[e] = g0 + e < J.count[1] ? x1[g0 + e] : 0u;
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) s += v[e];
    uint64_t run = block_exclusive_scan(s, &total);
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) {
        top[g0 + e] = g0 + e < J.count[1] ? run : ~(uint64_t)0;
        run += v[e];
    }
    __syncthreads();
    return PrefixHeader{total, fixed_exponent(st.w_max, J.log2n), 1};
}
static_assert(kTopMax == kPrefixThreads * 8u, "eight groups per thread");

// x of the lane whose number differs in the bits of Mask (1 or 2): a quad
// permutation on the vector unit.
template <int Mask>
__device__ __forceinline__ uint32_t quad_swap(uint32_t x)
{
    constexpr int kPerm = Mask == 1 ? 0xB1 : 0x4E;  // lanes 1,0,3,2 or 2,3,0,1 of each four
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kPerm, 0xF, 0xF, true);
}

template <int Mask>
__device__ __forceinline__ uint64_t quad_swap(uint64_t x)
{
    return (uint64_t)quad_swap<Mask>((uint32_t)x) | ((uint64_t)quad_swap<Mask>((uint32_t)(x >> 32)) << 32);
}

__device__ __forceinline__ uint64_t shuffle64(uint64_t x, int src)
{
    return (uint64_t)(uint32_t)__shfl((int)(uint32_t)x, src, 64) |
           ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(x >> 32), src, 64) << 32);
}

// The top level of the tree into LDS (k_prefix_scan has run).
__device__ __forceinline__ void load_top(const PrefixJob& J, uint64_t* top)
{
    const uint64_t* lv_top = at<uint64_t>(J, J.o_level[J.top]);
    for (uint32_t k = threadIdx.x; k < J.top_span; k += kPrefixThreads)
        top[k] = k < J.count[J.top] ? lv_top[k] : ~(uint64_t)0;
    __syncthreads();
}

// Multinomial: 64 outputs per wave and pass. Each lane bisects the top level in
// LDS for its own output; the rows below are read by quads, so that one load
// instruction touches 16 lines and not 64 (a row per lane would be bound by
// the address path): lane l serves the outputs r*16 + l/4, r < 4, reading their
// rows' parts l mod 4, and the quad adds up its counts. Requests to L2: one
// line per level below the top and one of weights, two in all up to 2^19
// inputs and three up to 2^23 (five and six with a level of sums per input and
// no level in LDS). What bounds it is VALU issue, about half of it the 64-bit
// sums of the groups' weights. Every lane of the wave runs to the end (outputs
// past n search too, and are not stored). Narrow: n <= 2^30, the byte offsets
// of weights and sums fit 32 bits.
template <bool Narrow, bool OwnScan>
__global__ __launch_bounds__(kPrefixThreads) void k_prefix_multinomial(PrefixJob J, uint32_t passes)
{
    using Off = std::conditional_t<Narrow, uint32_t, uint64_t>;
    __shared__ uint64_t top[kTopMax];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t first = blockIdx.x * kPrefixThreads * passes + threadIdx.x;
    PrefixHeader h;
    if constexpr (OwnScan)
        h = scan_in_lds(J, top);
    else
        h = *at<PrefixHeader>(J, J.o_hdr);
    if (!h.valid) {
        for (uint32_t p = 0; p < passes; ++p)
            if (first + p * kPrefixThreads < J.n) emit(J, first + p * kPrefixThreads, -1);
        return;
    }
    if constexpr (!OwnScan) load_top(J, top);
    const double scale = ldexp(1.0, h.K - 32);
    const uint32_t quad = lane / 4u, part = lane % 4u;
    const GlobalPtr<const char> w = global_ptr(reinterpret_cast<const char*>(J.w + (uint64_t)blockIdx.y * J.w_ld));
    const uint32_t whole = J.n / kFan;  // groups below it can be read by vectors
    for (uint32_t p = 0; p < passes; ++p) {
        const uint32_t i = first + p * kPrefixThreads;
        const uint64_t t_own = multinomial_threshold(J, h.total, i < J.n ? i : J.n - 1u);
        // the last entry <= t; entry 0 is 0
        uint32_t g_own = 0;
        for (uint32_t step = J.top_span / 2u; step > 0; step >>= 1)
            if (top[g_own + step] <= t_own) g_own += step;
        uint64_t t[4], before[4];
        uint32_t g[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int src = (int)(r * 16 + quad);
            before[r] = shuffle64(top[g_own], src);
            t[r] = shuffle64(t_own, src);
            g[r] = (uint32_t)__shfl((int)g_own, src, 64);
        }
        for (int k = J.top - 1; k >= 1; --k) {
            const GlobalPtr<const char> lv = global_ptr(at<const char>(J, J.o_level[k]));
            U64x2 a[4], b[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const Off row = (Off)g[r] * (8u * kFan) + part * 16u;
                a[r] = *(GlobalPtr<const U64x2>)(lv + row);
                b[r] = *(GlobalPtr<const U64x2>)(lv + row + 64u);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                uint32_t c = (a[r].x <= t[r] ? 1u : 0u) + (a[r].y <= t[r] ? 1u : 0u) + (b[r].x <= t[r] ? 1u : 0u) +
                             (b[r].y <= t[r] ? 1u : 0u);
                c += quad_swap<1>(c);
                c += quad_swap<2>(c);
                g[r] = g[r] * kFan + c - 1u;  // entry 0 of a row is <= t
                if (k == 1) {
                    // the largest entry <= t of the row, the sum before the
                    // group (reading it again would cost another request)
                    uint64_t m = a[r].x <= t[r] ? a[r].x : 0u;
                    m = a[r].y <= t[r] ? a[r].y : m;
                    m = b[r].x <= t[r] ? b[r].x : m;
                    m = b[r].y <= t[r] ? b[r].y : m;
                    uint64_t o = quad_swap<1>(m);
                    m = o > m ? o : m;
                    o = quad_swap<2>(m);
                    before[r] = o > m ? o : m;
                }
            }
        }
        // the groups' weights, four to a lane
        Row4 v[4];
        bool inside = true;
#pragma unroll
        for (int r = 0; r < 4; ++r) inside = inside && g[r] < whole;
        if (__all(inside)) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[r] = *(GlobalPtr<const Unaligned4>)(w + ((Off)g[r] * (4u * kFan) + part * 16u));
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) {
                    const uint64_t j = (uint64_t)g[r] * kFan + part * 4u + e;
                    v[r][e] = j < J.n ? *(GlobalPtr<const float>)(w + 4u * j) : 0.0f;
                }
        }
        uint32_t anc = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t p0 = fixed_weight(v[r][0], scale), p1 = p0 + fixed_weight(v[r][1], scale),
                           p2 = p1 + fixed_weight(v[r][2], scale), p3 = p2 + fixed_weight(v[r][3], scale);
            // the sum before the lane's four
            const uint64_t one = quad_swap<1>(p3);
            const uint64_t two = quad_swap<2>(p3 + one);
            const uint64_t base = before[r] + ((part & 1u) ? one : 0u) + ((part & 2u) ? two : 0u);
            uint32_t c = (base + p0 <= t[r] ? 1u : 0u) + (base + p1 <= t[r] ? 1u : 0u) +
                         (base + p2 <= t[r] ? 1u : 0u) + (base + p3 <= t[r] ? 1u : 0u);
            c += quad_swap<1>(c);
            c += quad_swap<2>(c);
            // output l's ancestor is that of r = l / 16 from the quad l mod 16
            const uint32_t x = (uint32_t)__shfl((int)(g[r] * kFan + c), (int)((lane % 16u) * 4u), 64);
            if (lane / 16u == (uint32_t)r) anc = x;
        }
        if (i < J.n) emit(J, i, (int32_t)anc);
    }
}

// The systematic outputs of a block, seven per lane side by side: down the tree,
// then through each group's weights. The few blocks that take it are what the
// launch then waits for, and few waves hide nothing, so the lane's seven searches
// share their round trips down the tree (the weights of seven groups at once
// would take registers from the blocks that do not come here). Whole calls, us,
// sorted weights of y = 4, one search after the other / side by side: 32769
// 36.3 / 20.6, 2^18 51.9 / 23.6, 2^20 62.5 / 27.6, 2^22 86 / 40 (the scan's part
// included).
__device__ __forceinline__ void search_lanes(const PrefixJob& J, const uint64_t* top, double scale,
                                             const SystematicDraw& draw, uint32_t first)
{
    uint64_t t[kSysPer];
    uint32_t g[kSysPer];
#pragma unroll
    for (uint32_t e = 0; e < kSysPer; ++e) {
        const uint32_t i = first + e * kPrefixThreads + threadIdx.x;
        t[e] = draw.threshold(i < J.n ? i : J.n - 1u);
        g[e] = 0;
    }
    for (uint32_t step = J.top_span / 2u; step > 0; step >>= 1)
#pragma unroll
        for (uint32_t e = 0; e < kSysPer; ++e)
            if (top[g[e] + step] <= t[e]) g[e] += step;
    for (int k = J.top - 1; k >= 1; --k) {
        const GlobalPtr<const uint64_t> lv = global_ptr(at<const uint64_t>(J, J.o_level[k]));
#pragma unroll
        for (uint32_t e = 0; e < kSysPer; ++e) g[e] *= kFan;
        for (uint32_t step = kFan / 2u; step > 0; step >>= 1) {
            uint64_t x[kSysPer];
#pragma unroll
            for (uint32_t e = 0; e < kSysPer; ++e) x[e] = lv[g[e] + step];
#pragma unroll
            for (uint32_t e = 0; e < kSysPer; ++e)
                if (x[e] <= t[e]) g[e] += step;
        }
    }
    const GlobalPtr<const float> w = global_ptr(J.w + (uint64_t)blockIdx.y * J.w_ld);
    const uint32_t whole = J.n / kFan;
    const GlobalPtr<const uint64_t> x1 = global_ptr(at<const uint64_t>(J, J.o_level[1]));
#pragma unroll
    for (uint32_t e = 0; e < kSysPer; ++e) {
        float v[kFan];
        uint64_t sum = x1[g[e]];
        if (g[e] < whole) {
#pragma unroll
            for (uint32_t c = 0; c < kFan; c += 4) {
                const Row4 x = *(GlobalPtr<const Unaligned4>)(w + (uint64_t)g[e] * kFan + c);
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) v[c + b] = x[b];
            }
        } else {
#pragma unroll
            for (uint32_t c = 0; c < kFan; ++c) {
                const uint64_t j = (uint64_t)g[e] * kFan + c;
                v[c] = j < J.n ? w[j] : 0.0f;
            }
        }
        uint32_t c = 0;
#pragma unroll
        for (uint32_t b = 0; b < kFan; ++b) {
            sum += fixed_weight(v[b], scale);
            c += sum <= t[e] ? 1u : 0u;
        }
        const uint32_t i = first + e * kPrefixThreads + threadIdx.x;
        if (i < J.n) emit(J, i, (int32_t)(g[e] * kFan + c));
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Systematic: kSysOut outputs per block. Their thresholds rise with i, so their
// ancestors lie between the groups of the block's first output and of the next
// block's, which the scan has left (OwnScan: the block counts them itself over
// its sums in LDS). The block goes through the weights from the one to the
// other in tiles of 2048: N outputs come from N inputs, so 1792 outputs take
// one tile unless their weights are very uneven, and every weight is read about
// once. Each input marks the first of its outputs, if it has any
// (outputs_below of the sums before and after it), and the running maximum of
// the marks is the ancestors. When the weights are more than kSysTiles tiles
// (long runs of very small weights), its lanes search for each output
// (OwnScan: never more than 16 tiles, which it adds up).
template <bool OwnScan>
__global__ __launch_bounds__(kPrefixThreads) void k_prefix_systematic(PrefixJob J)
{
    __shared__ __align__(16) uint64_t stage[kTopMax];
    __shared__ uint32_t s_cnt[kPrefixThreads / 64];
    const uint32_t first = blockIdx.x * kSysOut;
    PrefixHeader h;
    if constexpr (OwnScan)
        h = scan_in_lds(J, stage);
    else
        h = *at<PrefixHeader>(J, J.o_hdr);
    if (!h.valid) {
        for (uint32_t e = 0; e < kSysPer; ++e) {
            const uint32_t i = first + e * kPrefixThreads + threadIdx.x;
            if (i < J.n) emit(J, i, -1);
        }
        return;
    }
    const SystematicDraw draw(J, h.total);
    const uint32_t outs = J.n - first < kSysOut ? J.n - first : kSysOut;
    uint32_t g_lo, g_hi;
    uint64_t base;
    if constexpr (OwnScan) {
        const uint64_t t_lo = draw.threshold(first), t_hi = draw.threshold(first + outs - 1u);
        uint32_t c = 0;  // how many groups start at or below either threshold, at most 2048 each
#pragma unroll
        for (uint32_t e = 0; e < kTopMax / kPrefixThreads; ++e) {
            const uint64_t v = stage[e * kPrefixThreads + threadIdx.x];
            c += (v <= t_lo ? 1u : 0u) + (v <= t_hi ? 0x10000u : 0u);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) c += (uint32_t)__shfl_xor((int)c, off, 64);
        if ((threadIdx.x & 63u) == 0) s_cnt[threadIdx.x >> 6] = c;
        __syncthreads();
        c = 0;
        for (uint32_t k = 0; k < kPrefixThreads / 64u; ++k) c += s_cnt[k];
        g_lo = (c & 0xFFFFu) - 1u;
        g_hi = (c >> 16) - 1u;
        base = stage[g_lo];
        __syncthreads();  // the stage and s_cnt are overwritten next
    } else {
        const uint32_t* start = at<uint32_t>(J, J.o_start) + blockIdx.x;
        g_lo = start[0];
        g_hi = start[1];
        base = at<uint64_t>(J, J.o_level[1])[g_lo];
    }
    const uint64_t lo = (uint64_t)g_lo * kFan, end = ((uint64_t)g_hi + 1u) * kFan;
    const double scale = ldexp(1.0, h.K - 32);
    if (!OwnScan && end - lo > (uint64_t)kSysTiles * kChunk) {  // the same for every lane of the block
        load_top(J, stage);
        search_lanes(J, stage, scale, draw, first);
        return;
    }
    // mark[r]: 1 + the input (from lo on) whose outputs start at first + r, 0: none
    uint32_t* mark = reinterpret_cast<uint32_t*>(stage);
#pragma unroll
    for (uint32_t e = 0; e < kSysPer; ++e) mark[e * kPrefixThreads + threadIdx.x] = 0u;
    for (uint64_t tile = lo; tile < end; tile += kChunk) {
        uint64_t q[kPrefixPer];
        load_fixed_tile(J, tile, scale, q);
#pragma unroll
        for (uint32_t e = 1; e < kPrefixPer; ++e) q[e] += q[e - 1u];
        uint64_t total = 0;
        const uint64_t run = base + block_exclusive_scan(q[kPrefixPer - 1u], &total);
        const uint32_t j = (uint32_t)(tile - lo) + threadIdx.x * kPrefixPer + 1u;
        // places of the block's outputs, 0 to outs
        auto place = [&](uint64_t P) {
            const uint32_t i = draw.outputs_below(P);
            return i < first ? 0u : i - first < outs ? i - first : outs;
        };
        uint32_t from = place(run);
#pragma unroll
        for (uint32_t e = 0; e < kPrefixPer; ++e) {
            const uint32_t to = place(run + q[e]);
            if (from < to) mark[from] = j + e;
            from = to;
        }
        base += total;
    }
    __syncthreads();
    // the running maximum, seven consecutive places per thread
    uint32_t a[kSysPer], m = 0;
#pragma unroll
    for (uint32_t e = 0; e < kSysPer; ++e) {
        const uint32_t x = mark[threadIdx.x * kSysPer + e];
        m = x > m ? x : m;
        a[e] = m;
    }
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)m, off, 64);
        if ((int)lane >= off && y > m) m = y;
    }
    if (lane == 63u) s_cnt[wv] = m;
    __syncthreads();
    uint32_t prev = (uint32_t)__shfl_up((int)m, 1, 64);
    if (lane == 0) prev = 0u;
    for (uint32_t k = 0; k < wv; ++k) prev = s_cnt[k] > prev ? s_cnt[k] : prev;
#pragma unroll
    for (uint32_t e = 0; e < kSysPer; ++e)
        mark[threadIdx.x * kSysPer + e] = (uint32_t)lo - 1u + (a[e] > prev ? a[e] : prev);
    __syncthreads();
    if (!J.states && J.anc) {
        int32_t* anc = J.anc + (uint64_t)blockIdx.y * J.anc_ld + first;
#pragma unroll
        for (uint32_t e = 0; e < kSysPer; ++e) {
            const uint32_t r = e * kPrefixThreads + threadIdx.x;
            if (r < outs) anc[r] = (int32_t)mark[r];
        }
        return;
    }
#pragma unroll 1
    for (uint32_t e = 0; e < kSysPer; ++e) {
        const uint32_t r = e * kPrefixThreads + threadIdx.x;
        if (r < outs) emit(J, first + r, (int32_t)mark[r]);
    }
}

static uint64_t align256(uint64_t b) { return (b + 255u) & ~(uint64_t)255u; }

// The layout of one run's scan region: [header][chunk sums][tree levels
// 1..top][starts of the systematic search's blocks]. Returns the region's size.
uint64_t prefix_region(uint32_t n, PrefixJob* J)
{
    const uint64_t nch = ((uint64_t)n + kChunk - 1u) / kChunk;
    uint64_t o = 0;
    J->o_hdr = o;
    o += 256u;
    J->o_sum = o;
    o += align256(nch * 8u);
    // level k has ceil(n / 16^k) entries; the top is the first with <= kTopMax
    uint64_t cnt = n;
    J->top = 0;
    do {
        cnt = (cnt + kFan - 1u) / kFan;
        ++J->top;
        J->count[J->top] = (uint32_t)cnt;
        J->o_level[J->top] = o;
        o += align256((cnt + kFan - 1u) / kFan * kFan * 8u);
    } while (cnt > kTopMax);
    J->nsys = (uint32_t)(((uint64_t)n + kSysOut - 1u) / kSysOut);
    J->o_start = o;
    o += align256(((uint64_t)J->nsys + 1u) * 4u);
    J->top_span = 1u;
    while (J->top_span < cnt) J->top_span *= 2u;
    J->n = n;
    J->per = chunks_per_block(n);
    J->nsum = (uint32_t)((nch + J->per - 1u) / J->per);
    int L = 0;
    while (((uint64_t)1 << L) < (uint64_t)n) ++L;
    J->log2n = L;
    return o;
}

int enqueue_prefix(const PrefixJob& J, uint32_t R, int method, hipStream_t s)
{
    const dim3 bt(kPrefixThreads);
    if (J.parts)
        hipLaunchKernelGGL(k_prefix_groups<true>, dim3(J.nsum, R), bt, 0, s, J);
    else
        hipLaunchKernelGGL(k_prefix_groups<false>, dim3(J.nsum, R), bt, 0, s, J);
    const bool own_scan = J.top == 1;
    const dim3 scan_grid((J.count[1] + kScanGroups - 1u) / kScanGroups, R);
    if (!own_scan && method == MGP_SYSTEMATIC)
        hipLaunchKernelGGL(k_prefix_scan<true>, scan_grid, bt, 0, s, J);
    else if (!own_scan)
        hipLaunchKernelGGL(k_prefix_scan<false>, scan_grid, bt, 0, s, J);
    int err = check_launch("prefix-sum kernels");
    if (err) return err;
    if (method == MGP_MULTINOMIAL) {
        // four passes per block read the top level once for 1024 outputs, where that leaves enough blocks
        const uint32_t passes = (uint64_t)J.n * R >= (1u << 19) ? 4u : 1u;
        const uint32_t per = kPrefixThreads * passes;
        const dim3 grid((J.n + per - 1u) / per, R);
        if (own_scan)
            hipLaunchKernelGGL((k_prefix_multinomial<true, true>), grid, bt, 0, s, J, passes);
        else if (J.n <= (1u << 30))
            hipLaunchKernelGGL((k_prefix_multinomial<true, false>), grid, bt, 0, s, J, passes);
        else
            hipLaunchKernelGGL((k_prefix_multinomial<false, false>), grid, bt, 0, s, J, passes);
    } else {
        const dim3 grid(J.nsys, R);
        if (own_scan)
            hipLaunchKernelGGL(k_prefix_systematic<true>, grid, bt, 0, s, J);
        else
            hipLaunchKernelGGL(k_prefix_systematic<false>, grid, bt, 0, s, J);
    }
    return check_launch("prefix-sum search kernel");
}

}  // namespace mgp

using namespace mgp;

// The scan room that the single-filter entry point asks for: 8 bytes per input
// (whole chunks) and per entry of the tree down to 16 entries, 16 per chunk, 4
// per 256 outputs. The scan itself uses a tenth of it (prefix_region), and a
// call that needs a copy of its weights half of the rest.
static uint64_t prefix_workspace(uint32_t n)
{
    const uint64_t nch = ((uint64_t)n + kChunk - 1u) / kChunk;
    uint64_t o = 256u + 2u * align256(nch * 8u) + align256(((uint64_t)n / 256u + 2u) * 4u);
    for (uint64_t cnt = n; cnt > kFan;) {
        cnt = (cnt + kFan - 1u) / kFan;
        o += align256((cnt + kFan - 1u) / kFan * kFan * 8u);
    }
    return workspace_bytes(1u) + o + align256(nch * kChunk * 8u);
}

// Up to this size the finalize step runs in every block of k_prefix_groups;
// beyond, it has its own launch, which is nothing there. Systematic, us, in the
// blocks / by itself: 2^22 39 / 40, 10^7 61.5 / 62.2, 2^24 83 / 84.
constexpr uint32_t kPrefixFinMaxN = 1u << 24;

// Multinomial reads a group of 16 weights per output from a random place: one
// cache line where the weights are 64-byte aligned, else two for every other
// group. From this size on that costs more than an aligned copy. us, without /
// with a copy: 2^20 39.6 / 43.6, 2^21 68.7 / 66.7, 2^24 716 / 580 (aligned 566).
constexpr uint32_t kAlignMinN = 1u << 21;

extern "C" {

int mgp_prefix_workspace_size(int32_t n, size_t* bytes)
{
    clear_error();
    if (!bytes) return fail(MGP_EINVAL, "bytes is NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    *bytes = prefix_workspace((uint32_t)n);
    return MGP_OK;
}

int mgp_resample_prefix(const float* w_dev, int32_t n, int32_t method, uint64_t seed, uint32_t stream_id,
                        int32_t* ancestors_dev, mgp_stats* stats_dev, void* workspace_dev, size_t workspace_bytes_,
                        void* stream)
{
    clear_error();
    if (!w_dev || !ancestors_dev) return fail(MGP_EINVAL, "w_dev and ancestors_dev must not be NULL");
    if (n < 1) return fail(MGP_EINVAL, "n must be >= 1 (got %d)", n);
    if (method != MGP_MULTINOMIAL && method != MGP_SYSTEMATIC)
        return fail(MGP_EINVAL, "unknown prefix-sum method %d", method);
    if (!workspace_dev) return fail(MGP_EINVAL, "workspace is NULL");
    if (((uintptr_t)workspace_dev & 255u) != 0) return fail(MGP_EINVAL, "workspace must be 256-byte aligned");
    const uint32_t un = (uint32_t)n;
    PrefixJob J{};
    const uint64_t region_bytes = prefix_region(un, &J);
    const size_t need = prefix_workspace(un);
    if (workspace_bytes_ < need) return fail(MGP_ERANGE, "workspace has %zu bytes, needs %zu", workspace_bytes_, need);
    char* ws = static_cast<char*>(workspace_dev);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // validation, max and fp64 sum: the reduction and finalize step of the
    // other resamplers (one explicit iteration, no offsets, no windows)
    Params p;
    p.variant = kMetropolis;
    p.B = 1;
    p.eps = 0.5;
    p.seed = seed;
    p.stream_id = stream_id;
    p.partition_bytes = 128;
    p.b_max = 1;
    // The search reads the weights while it writes ancestors. Outputs that lie
    // over the weights (ancestors in place, say) are written while other blocks
    // still read there, so such a call scans and searches a copy, which the
    // reduction makes behind the scan's region. So does a large multinomial call
    // whose weights are not 64-byte aligned (kAlignMinN).
    const uint64_t bytes = 4ull * un;
    float* copy = nullptr;
    if (ranges_overlap(w_dev, bytes, ancestors_dev, bytes) ||
        ranges_overlap(w_dev, bytes, stats_dev, sizeof(mgp_stats)) ||
        (method == MGP_MULTINOMIAL && un >= kAlignMinN && ((uintptr_t)w_dev & 63u) != 0))
        copy = reinterpret_cast<float*>(ws + workspace_bytes(1u) + align256(region_bytes));
    J.stats = reinterpret_cast<mgp_stats*>(ws + kWsStatsOffset);
    if (un <= kPrefixFinMaxN) {
        J.parts = reinterpret_cast<const Partial*>(ws + kWsPartialsOffset);
        J.st_user = stats_dev;
        const int err = enqueue_partials(w_dev, un, p, ws, &J.nparts, &J.fin, copy, s);
        if (err) return err;
    } else {
        const int err = enqueue_reduce_finalize(w_dev, un, p, false, kLayoutInPlace, ws, stats_dev, s, copy);
        if (err) return err;
    }
    J.w = copy ? copy : w_dev;
    J.region = ws + workspace_bytes(1u);
    J.anc = ancestors_dev;
    J.key0 = (uint32_t)seed;
    J.key1 = (uint32_t)(seed >> 32);
    J.stream0 = stream_id;
    return enqueue_prefix(J, 1u, method, s);
}

}  // extern "C"
