// What the slow model's kernels do besides for a small batch, so that it costs no launch of its own (one takes as long on the
// device as the whole gate does, and 3 to 4 us on the host): evaluate the gate on the fast model's votes, and copy the labels of
// the flows that are not on the list.  Whole pass, with the label copy as a launch : in this one: 20,011 flows 50.8 : 48.6 us, 10,007 flows
// and a small boosted model 26.1 : 23.7; the gate's figures are at slow_gates().
#pragma once

#include "common.h"

namespace sfsmall {

// Rows the gate takes this way: a block evaluates it for all of them, eight to a thread at a time.  Whole pass, the gate as a launch : in
// this one, us.  bfloat16, 64-200-300-10: 200 rows 18.9 : 17.5, 8,000 25.1 : 23.7, 12,000 25.3 : 24.7, 16,384 25.9 : 25.8; 32-128-64-6
// 15.1 : 13.6, 21.2 : 19.2, 23.5 : 23.3, 24.4 : 25.4.  binary32, whose blocks are more than are resident from 2,048 rows on,
// 32-128-128-4: 4,096 rows 22.8 : 21.4, 5,000 27.0 : 29.3, 16,384 46.4 : 58.1; 32-64-48-10: 16.5 : 15.8, 17.3 : 20.5, 21.5 : 30.5.
constexpr uint32_t kGateRows = 12288, kGateRowsF32 = 4096;
constexpr uint32_t kCopyRows = 65536;   // flows whose labels are copied this way at most: a copying block reads the whole list
constexpr uint32_t kCopySlice = 2048;   // flows of a copying block

// sf_route's gate: the list and its length are written for the caller as by that call
struct GateRows {
    const uint16_t* top;
    const uint16_t* pred;
    uint32_t n, n_vmin;
    uint32_t* esc_idx;
    uint32_t* esc_count;
    uint16_t vmin[SF_MAX_CLASSES];
};
struct NoGate {};

// Whether two arrays share memory.  What these kernels do in one launch the separate calls do one after the other, so an array that
// one of the steps reads and another writes is not for them.
inline bool share(const void* a, uint64_t a_bytes, const void* b, uint64_t b_bytes)
{
    const uint64_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && (x < y ? y - x < a_bytes : x - y < b_bytes);
}

constexpr uint32_t kGateLds = 64 + SF_MAX_CLASSES * 2; // bytes of shared memory

// The gate for all rows by a block of T threads (up to 32 rows a thread, in order): the number of rows that escalate, and with
// write(p) for every position p of the list where it is true the list's entry.  sm: kGateLds bytes, free again behind the caller's next
// barrier, which also has to stand between this and reading the list.
template <uint32_t T, class Mine>
__device__ __forceinline__ uint32_t gate_rows(const GateRows& g, void* sm, Mine mine)
{
    uint32_t* s_wave = reinterpret_cast<uint32_t*>(sm); // [T / 64]
    uint16_t* s_vmin = reinterpret_cast<uint16_t*>(s_wave + 16);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t per = (g.n + T * 8u - 1u) / (T * 8u) * 8u, base = tid * per; // (at most 32)
    const bool one = g.n_vmin == 1u;
    const bool wide = ((reinterpret_cast<uintptr_t>(g.top) | (one ? 0u : reinterpret_cast<uintptr_t>(g.pred))) & 15u) == 0;
    if (tid < SF_MAX_CLASSES) s_vmin[tid] = g.vmin[tid];
    __syncthreads();
    uint32_t mask = 0;
    for (uint32_t j = 0; j < per; j += 8u) {
        const uint32_t at = base + j;
        if (at >= g.n) break;
        uint16_t v[8], p[8];
        if (wide && at + 8u <= g.n) {
            const uint4 w = *reinterpret_cast<const uint4*>(g.top + at), q = *reinterpret_cast<const uint4*>((one ? g.top : g.pred) + at);
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w}, qq[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                v[k] = (uint16_t)(ww[k / 2] >> (16 * (k & 1)));
                p[k] = (uint16_t)(qq[k / 2] >> (16 * (k & 1)));
            }
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 8u; ++k) {
                v[k] = at + k < g.n ? g.top[at + k] : (uint16_t)0xFFFFu;
                p[k] = at + k < g.n && !one ? g.pred[at + k] : (uint16_t)0;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) {
            const uint32_t c = one ? 0u : p[k] < g.n_vmin ? p[k] : g.n_vmin - 1u;
            if (at + k < g.n && v[k] < s_vmin[c]) mask |= 1u << (j + k);
        }
    }
    uint32_t inc = __popc(mask);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d, 64);
        if (lane >= (uint32_t)d) inc += o;
    }
    if (lane == 63u) s_wave[wave] = inc;
    __syncthreads();
    uint32_t total = 0, pos = inc - __popc(mask);
#pragma unroll
    for (uint32_t w = 0; w < T / 64u; ++w) {
        const uint32_t s = s_wave[w];
        pos += w < wave ? s : 0u;
        total += s;
    }
    const auto is_mine = mine(total);
    for (; mask; mask &= mask - 1u, ++pos)
        if (is_mine(pos)) g.esc_idx[pos] = base + (uint32_t)__ffs(mask) - 1u;
    return total;
}

// labels = pred for the flows [lo, lo + kCopySlice) that are not on the list (total entries; CLAMP: a bad one stands for the last
// flow, else for none); the other labels are being written by the blocks beside this one.  bits: kCopySlice / 32 words of shared
// memory.
template <uint32_t T, bool CLAMP>
__device__ __forceinline__ void copy_unlisted(const uint16_t* __restrict__ pred, uint16_t* __restrict__ labels, uint32_t n, const uint32_t* __restrict__ list,
                                              uint32_t total, uint32_t lo, uint32_t* bits)
{
    const uint32_t tid = threadIdx.x;
    if (tid < kCopySlice / 32u) bits[tid] = 0;
    __syncthreads();
    const auto mark = [&](uint32_t f) {
        if (CLAMP) f = f < n ? f : n - 1u;
        f -= lo;
        if (f < kCopySlice) atomicOr(bits + f / 32u, 1u << (f & 31u));
    };
    // (the list's whole 16-byte pieces, four of a thread at a time: tiles wait behind the blocks that copy.  25,848 of 28,720 flows, entry
    // by entry : this 26.5 : 22.1 us)
    const uint32_t pieces = (reinterpret_cast<uintptr_t>(list) & 15u) == 0 ? total / 4u : 0u;
    for (uint32_t e = tid; e < pieces; e += 4u * T) {
        uint4 v[4];
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) {
            const uint32_t at = e + q * T;
            v[q] = reinterpret_cast<const uint4*>(list)[at < pieces ? at : e];
        }
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) mark(v[q].x), mark(v[q].y), mark(v[q].z), mark(v[q].w);
    }
    for (uint32_t e = 4u * pieces + tid; e < total; e += T) mark(list[e]);
    __syncthreads();
    for (uint32_t f = tid; f < kCopySlice && lo + f < n; f += T)
        if (!(bits[f / 32u] >> (f & 31u) & 1u)) labels[lo + f] = pred[lo + f];
}

} // namespace sfsmall
