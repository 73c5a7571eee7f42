// mgp_reduce.h -- device code shared by the single-filter and batched paths:
// the weight reduction (fp32 max, fp64 sum, validation, optional copy) and the finalize step that turns it into B (eq. (proposition)),
// the stats record and the Megopolis offsets.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mgp.h"
#include "mgp_device.h"
#include "mgp_internal.h"

namespace mgp {

__device__ __forceinline__ void fold(float v, float& mx, double& s, uint32_t& bad)
{
    bad |= (!(v >= 0.0f) || v == INFINITY) ? 1u : 0u;
    mx = fmaxf(mx, v);
    s += (double)v;
}

// Every block that calls these has kReduceThreads threads, a constant here: the
// block's size is otherwise one more load from memory before the first step
// (0.8 us of 6.9 of a small filter's call).

// Block-wide reduction of (max, sum, bad); result valid in thread 0.
__device__ __forceinline__ void block_reduce(float& mx, double& s, uint32_t& bad)
{
    __shared__ float smx[kReduceThreads / 64];
    __shared__ double ssum[kReduceThreads / 64];
    __shared__ uint32_t sbad[kReduceThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        s += __shfl_xor(s, off, 64);
        bad |= __shfl_xor(bad, off, 64);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        smx[wv] = mx;
        ssum[wv] = s;
        sbad[wv] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = smx[0];
        s = ssum[0];
        bad = sbad[0];
        for (int k = 1; k < (int)(kReduceThreads / 64); ++k) {
            mx = fmaxf(mx, smx[k]);
            s += ssum[k];
            bad |= sbad[k];
        }
    }
}

// Four floats at any float's address: one access, which the hardware splits
// where it has to.
using Unaligned4 = float __attribute__((ext_vector_type(4), aligned(4)));

// Reduces w[start, end) into (mx, s, bad) per thread and, with a copy or a tail,
// writes copy[i] = w[i], tail[i] = w[i] for the range. With Vec, w + start is
// 16-byte aligned, as copy + start is; tail need not be.
template <bool Vec>
__device__ __forceinline__ void reduce_range(const float* __restrict__ w, uint64_t start, uint64_t end,
                                             float* __restrict__ copy, float* __restrict__ tail, float& mx, double& s,
                                             uint32_t& bad)
{
    if constexpr (Vec) {
        const uint64_t end4 = start + ((end - start) & ~(uint64_t)3);
        for (uint64_t i = start + 4ull * threadIdx.x; i < end4; i += 4ull * kReduceThreads) {
            const float4 v = *reinterpret_cast<const float4*>(w + i);
            if (copy) *reinterpret_cast<float4*>(copy + i) = v;
            if (tail) *reinterpret_cast<Unaligned4*>(tail + i) = Unaligned4{v.x, v.y, v.z, v.w};
            fold(v.x, mx, s, bad);
            fold(v.y, mx, s, bad);
            fold(v.z, mx, s, bad);
            fold(v.w, mx, s, bad);
        }
        for (uint64_t i = end4 + threadIdx.x; i < end; i += kReduceThreads) {
            const float v = w[i];
            if (copy) copy[i] = v;
            if (tail) tail[i] = v;
            fold(v, mx, s, bad);
        }
    } else {
        for (uint64_t i = start + threadIdx.x; i < end; i += kReduceThreads) {
            const float v = w[i];
            if (copy) copy[i] = v;
            if (tail) tail[i] = v;
            fold(v, mx, s, bad);
        }
    }
}

// What a Megopolis loop needs beyond the reduction, by one block: the seam of
// weights read in place, or the repeated first kSeam weights of a copy. With a
// tail, which holds the seam's second half, they are the last kSeam weights and
// those after the tail's n.
__device__ __forceinline__ void write_window_ends(const float* __restrict__ w, uint32_t n, float* __restrict__ copy,
                                                  float* __restrict__ seam, float* __restrict__ tail)
{
    if (tail) {
        for (uint32_t k = threadIdx.x; k < kSeam; k += kReduceThreads) {
            if (seam) seam[k] = w[n - kSeam + k];
            tail[(uint64_t)n + k] = w[k];
        }
        return;
    }
    if (seam) write_seam(w, n, seam);
    if (copy)
        for (uint32_t k = threadIdx.x; k < kSeam; k += kReduceThreads) copy[(uint64_t)n + k] = w[k % n];
}

// ---------------------------------------------------------------------------
// 2. Finalize: combine the partials, pick B by eq. (proposition), write the
//    stats, and generate the Megopolis offsets o_0..o_{B-1} (Algorithm 5's
//    offsets are drawn before the particle loop; here in parallel, four per
//    Philox call).
// ---------------------------------------------------------------------------
// Offsets b of [first, end) (first a multiple of 4), four per call, by the
// threads t, t + stride, ...
__device__ __forceinline__ void draw_offsets(const FinalizeArgs& a, uint32_t first, uint32_t end, uint32_t t,
                                             uint32_t stride, uint32_t* __restrict__ offsets)
{
    for (uint32_t c = first / 4u + t; c < (end + 3u) / 4u; c += stride) {
        const Words x = philox(c, kTagOffset, a.stream_id, 0u, a.key0, a.key1);
        const uint32_t o[4] = {x.x0, x.x1, x.x2, x.x3};
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t b = 4u * c + r;
            if (b < end) offsets[b] = uniform_index(o[r], a.n);
        }
    }
}

// Partials of whole groups of Ahead per thread from `from` on, each group's
// loads in flight together, folded in index order.
template <uint32_t Ahead>
__device__ __forceinline__ void fold_partials(const Partial* __restrict__ part, uint32_t nparts, uint32_t& from,
                                              float& mx, double& s, uint32_t& bad)
{
    for (; from + Ahead * kReduceThreads <= nparts; from += Ahead * kReduceThreads) {
        Partial q[Ahead];
#pragma unroll
        for (uint32_t u = 0; u < Ahead; ++u) q[u] = part[from + u * kReduceThreads + threadIdx.x];
#pragma unroll
        for (uint32_t u = 0; u < Ahead; ++u) {
            mx = fmaxf(mx, q[u].w_max);
            s += q[u].w_sum;
            bad |= q[u].bad;
        }
    }
}

// Returns B (0 for invalid weights) in every thread. Many: where there may be
// thousands of partials, sixteen round trips one after the other otherwise.
// Whole calls, us, before / with it: Megopolis y = 0, 2^22 26.6 / 24.9, 2^23 45.0 /
// 41.5; systematic 10^7 61.3 / 58.0. The loops that do this step themselves
// have 512 at most and stay without (0.2 of 7.7 us at 20000 particles).
template <bool Many = false>
__device__ __forceinline__ uint32_t finalize_one(const Partial* __restrict__ part, uint32_t nparts, const FinalizeArgs& a,
                             mgp_stats* __restrict__ st, mgp_stats* __restrict__ st_user,
                             uint32_t* __restrict__ offsets)
{
    __shared__ uint32_t sB;
    float mx = 0.0f;
    double s = 0.0;
    uint32_t bad = 0;
    uint32_t from = 0;
    if constexpr (Many) {
        fold_partials<8>(part, nparts, from, mx, s, bad);
        fold_partials<4>(part, nparts, from, mx, s, bad);
    }
    for (uint32_t p = from + threadIdx.x; p < nparts; p += kReduceThreads) {
        const Partial q = part[p];
        mx = fmaxf(mx, q.w_max);
        s += q.w_sum;
        bad |= q.bad;
    }
    block_reduce(mx, s, bad);
    if (threadIdx.x == 0) {
        mgp_stats r;
        r.w_sum = s;
        r.w_max = mx;
        r.n = a.n;
        r.clamped = 0;
        r.tag = a.tag;
        r.ratio = 0.0;
        r.b_raw = 0.0;
        if (bad || !(mx > 0.0f)) {
            r.status = MGP_EWEIGHTS;
            r.B = 0;
        } else {
            r.status = MGP_OK;
            const double mean = s / (double)a.n;
            const double ratio = mean / (double)mx;
            r.ratio = ratio;
            if (a.B_user > 0) {
                r.B = a.B_user;
            } else {
                const double raw = ratio >= 1.0 ? 1.0 : (a.log_eps ? *a.log_eps : log(a.eps)) / log1p(-ratio);
                r.b_raw = raw;
                double c = ceil(raw);
                if (c < 1.0) c = 1.0;
                if (c > (double)a.b_max) {
                    c = (double)a.b_max;
                    r.clamped = 1;
                }
                r.B = (uint32_t)c;
            }
        }
        *st = r;
        if (st_user) *st_user = r;
        sB = r.B;
    }
    __syncthreads();
    const uint32_t B = sB;
    if (a.make_offsets && B > 0)
        draw_offsets(a, 0u, B, threadIdx.x, kReduceThreads, offsets);
    return B;
}

}  // namespace mgp
