// Device code of step 1 shared by the stand-alone feature kernel and the fused feature + forest kernel:
// the 32 statistics of one prefix window of a flow whose packets sit in the lane's registers
// (context length k, Section 3.1 of the paper).
//
// Every binary32 operation is issued on its own, in packet order (the files that include this are
// compiled without floating-point contraction); a packet outside a group contributes +0.0 to that
// group's running sums, which leaves them unchanged.
//
// Order statistics (min, max, median of the two directions and of all packets) need sorted values.
// Instead of three sorting networks per quantity (one per group) there is ONE, on keys that carry the
// direction as their top bit and the value of a direction-1 packet complemented: after it the
// direction-0 packets stand first in ascending order, the direction-1 packets behind them in
// DESCENDING order, padding last.  Both directions' statistics are read from that array at
// data-dependent positions; the array, with padding read as the smallest value, is also a bitonic
// sequence (up, then down), so ONE merge stage (log2 N levels instead of a full network) sorts all
// packets together for the third group.  This needs values that order like non-negative integers
// below 2^W: packet sizes (W = 16) and non-negative times (W = 31, the binary32 bit pattern).  A wave
// that holds a time with its sign bit set takes the general path: three full networks on
// order-preserving keys.
//
// The element at a data-dependent rank is read through a per-lane column of shared memory
// (col[i * stride], stride = lanes that share the array, so every lane stays on its own bank).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sffeat {

// A flow's packet records as loaded by the wide path (whole deepest window present, 16-byte aligned)
template <int KMAX>
struct RawPackets {
    uint4 sz[KMAX / 8];
    float4 tm[KMAX / 4];
    uint2 dr[KMAX / 8];
};

template <int KMAX>
__device__ __forceinline__ void load_wide(const uint16_t* size, const float* iat, const uint8_t* dir, uint32_t o, RawPackets<KMAX>& r)
{
#pragma unroll
    for (int c = 0; c < KMAX / 8; ++c) {
        r.sz[c] = *reinterpret_cast<const uint4*>(size + o + 8 * c);
        r.tm[2 * c] = *reinterpret_cast<const float4*>(iat + o + 8 * c);
        r.tm[2 * c + 1] = *reinterpret_cast<const float4*>(iat + o + 8 * c + 4);
        r.dr[c] = *reinterpret_cast<const uint2*>(dir + o + 8 * c);
    }
}

template <int KMAX>
__device__ __forceinline__ void decode_wide(const RawPackets<KMAX>& r, float (&s)[KMAX], float (&t)[KMAX], uint32_t& dmask)
{
    dmask = 0;
#pragma unroll
    for (int c = 0; c < KMAX / 8; ++c) {
        const uint32_t w[4] = {r.sz[c].x, r.sz[c].y, r.sz[c].z, r.sz[c].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s[8 * c + 2 * k] = (float)(w[k] & 0xFFFFu);
            s[8 * c + 2 * k + 1] = (float)(w[k] >> 16);
        }
        const float4 t0 = r.tm[2 * c], t1 = r.tm[2 * c + 1];
        t[8 * c + 0] = t0.x; t[8 * c + 1] = t0.y; t[8 * c + 2] = t0.z; t[8 * c + 3] = t0.w;
        t[8 * c + 4] = t1.x; t[8 * c + 5] = t1.y; t[8 * c + 6] = t1.z; t[8 * c + 7] = t1.w;
        const uint32_t dw[2] = {r.dr[c].x, r.dr[c].y};
#pragma unroll
        for (int k = 0; k < 8; ++k) dmask |= ((dw[k >> 2] >> (8 * (k & 3))) & 1u) << (8 * c + k);
    }
}

// The first `avail` packets from o on, one by one; zeros behind them
template <int KMAX>
__device__ __forceinline__ void load_each(const uint16_t* size, const float* iat, const uint8_t* dir, uint32_t o, int avail, float (&s)[KMAX],
                                          float (&t)[KMAX], uint32_t& dmask)
{
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        if (j < avail) {
            s[j] = (float)size[o + j];
            t[j] = iat[o + j];
            dmask |= (uint32_t)(dir[o + j] & 1u) << j;
        } else {
            s[j] = 0.f;
            t[j] = 0.f;
        }
    }
}

// float -> unsigned key with the same order (negative values: all bits flipped, others: sign set)
__device__ __forceinline__ uint32_t order_key(float x)
{
    const uint32_t b = __float_as_uint(x);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float from_key(uint32_t u)
{
    return __uint_as_float(u ^ ((u & 0x80000000u) ? 0x80000000u : 0xFFFFFFFFu));
}

__device__ __forceinline__ void cmp_swap(uint32_t& lo, uint32_t& hi)
{
    const uint32_t a = lo < hi ? lo : hi, b = lo < hi ? hi : lo;
    lo = a;
    hi = b;
}

// Batcher's odd-even merge sort as a fixed network; every index is a compile-time constant
// after unrolling, so the keys stay in registers.
template <int N>
__device__ __forceinline__ void sort_network(uint32_t (&a)[N])
{
#pragma unroll
    for (int p = 1; p < N; p <<= 1) {
#pragma unroll
        for (int k = p; k >= 1; k >>= 1) {
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k) {
#pragma unroll
                for (int i = 0; i < k; ++i) {
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) cmp_swap(a[i + j], a[i + j + k]);
                }
            }
        }
    }
}

// Sorts a bitonic sequence (ascending, then descending) into ascending order: log2 N levels of N/2 exchanges.
template <int N>
__device__ __forceinline__ void bitonic_merge(uint32_t (&a)[N])
{
#pragma unroll
    for (int k = N / 2; k >= 1; k >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if ((i & k) == 0) cmp_swap(a[i], a[i + k]);
        }
    }
}

__device__ __forceinline__ bool bit_of(uint32_t m, int j) { return (m >> j) & 1u; }

// Group membership comes in two forms, the template parameter WORDS of everything below.
// false: compare and select; the comparisons of a packet are shared by all statistics of its window, which keeps a pair of
//   scalar registers alive per packet and group.  The one-lane kernel takes this form up to 16 packets, where a wave has
//   the registers: 262,149 flows x 16 packets, windows 8 and 16, 28.9 us against 32.8 with words, which are 11 % more
//   vector instructions; 1,048,576 flows, window 16, 62.8 against 70.7.
// true: a word per packet and group that is all ones or zero (one signed bit-field extract), applied with and / xor, and
//   made again from the masks for each part of the statistics.  For 32 packets, where the pairs outnumber a wave's scalar
//   registers (234 spilled), and for the kernels that split the parts between waves with few registers each (48 vector
//   registers spilled in the fused kernel).
__device__ __forceinline__ uint32_t bit_word(uint32_t m, int j) { return (uint32_t)__builtin_amdgcn_sbfe((int)m, (uint32_t)j, 1u); }
// between two parts of the statistics: nothing made from the masks is kept in a register
template <bool WORDS>
__device__ __forceinline__ void forget_words(uint32_t& a, uint32_t& b, uint32_t& c)
{
    if (WORDS) asm volatile("" : "+v"(a), "+v"(b), "+v"(c));
}
// x where bit j of m is set, else +0.0
template <bool WORDS>
__device__ __forceinline__ float masked(float x, uint32_t m, int j)
{
    if (WORDS) return __uint_as_float(__float_as_uint(x) & bit_word(m, j));
    return bit_of(m, j) ? x : 0.f;
}

// Order statistics of one quantity for the three groups (0: direction 0, 1: direction 1, 2: all packets).
// v[i]: the value of packet i as a non-negative integer below 2^W that orders like the value.  valid: the
// window's packets; m1: those of direction 1; m = c0 + c1 packets.  Results are such integers too; for an
// empty group they are meaningless (the caller writes zeros).  lo/hi: the two middle elements (equal for an
// odd count).
template <bool WORDS, int N, int W>
__device__ __forceinline__ void order_stats3(const uint32_t (&v)[N], uint32_t valid, uint32_t m1, int m, int c0, int c1,
                                             uint32_t* col, uint32_t stride, uint32_t (&mn)[3], uint32_t (&mx)[3],
                                             uint32_t (&lo)[3], uint32_t (&hi)[3])
{
    constexpr uint32_t kMask = (1u << W) - 1u;            // W = 31: 0x7FFFFFFF
    constexpr uint32_t kPad = (1u << W) | kMask;          // the largest key; decodes to the value 0
    uint32_t key[N], outside = ~valid;
    forget_words<WORDS>(valid, outside, m1);
#pragma unroll
    for (int i = 0; i < N; ++i) { // direction 1: top bit set and value complemented; outside the window: kPad
        if (WORDS)
            key[i] = (v[i] ^ (bit_word(m1, i) & kPad)) | (bit_word(outside, i) & kPad);
        else
            key[i] = bit_of(valid, i) ? (bit_of(m1, i) ? v[i] ^ kPad : v[i]) : kPad;
    }
    sort_network<N>(key);
#pragma unroll
    for (int i = 0; i < N; ++i) col[i * stride] = key[i];
    // direction 0: ascending at positions [0, c0)
    const int l0 = c0 > 0 ? c0 - 1 : 0;
    mn[0] = key[0];
    mx[0] = col[l0 * stride];
    lo[0] = col[(l0 >> 1) * stride];
    hi[0] = col[(c0 >> 1) * stride];
    // direction 1: descending at positions [c0, m); rank r (ascending) sits at position m - 1 - r
    const int l1 = c1 > 0 ? c1 - 1 : 0;
    const int top = m > 0 ? m - 1 : 0;
    const int p_mx = c0 < N ? c0 : N - 1; // c1 = 0 and c0 = N: the group is empty, any position will do
    mn[1] = col[top * stride] ^ kMask;    // (key & kMask) ^ kMask; the direction bit is cleared below
    mx[1] = col[p_mx * stride] ^ kMask;
    lo[1] = col[(top - (l1 >> 1)) * stride] ^ kMask;
    hi[1] = col[(top - (c1 >> 1) < 0 ? 0 : top - (c1 >> 1)) * stride] ^ kMask;
    mn[1] &= kMask;
    mx[1] &= kMask;
    lo[1] &= kMask;
    hi[1] &= kMask;
    // all packets: decode (padding becomes 0, the smallest value), merge; the padding then stands first
#pragma unroll
    for (int i = 0; i < N; ++i) key[i] = (key[i] ^ bit_word(key[i], W)) & kMask;
    bitonic_merge<N>(key);
#pragma unroll
    for (int i = 0; i < N; ++i) col[i * stride] = key[i];
    const int first = N - m; // number of padding elements
    const int la = m > 0 ? m - 1 : 0;
    const int f = first < N ? first : N - 1;
    mn[2] = col[f * stride];
    mx[2] = key[N - 1];
    lo[2] = col[(f + (la >> 1)) * stride];
    hi[2] = col[(f + (m >> 1) < N ? f + (m >> 1) : N - 1) * stride];
}

// General path for times with the sign bit set somewhere in the wave: one full network per group on
// order-preserving keys, padded with the largest key.
template <int N, int KMAX>
__device__ __forceinline__ void order_stats_signed(const float (&x)[KMAX], uint32_t gm, int cg, uint32_t* col, uint32_t stride,
                                                   float& mn, float& mx, float& lo, float& hi)
{
    uint32_t key[N];
#pragma unroll
    for (int i = 0; i < N; ++i) key[i] = bit_of(gm, i) ? order_key(x[i]) : 0xFFFFFFFFu;
    sort_network<N>(key);
#pragma unroll
    for (int i = 0; i < N; ++i) col[i * stride] = key[i];
    const int last = cg > 0 ? cg - 1 : 0;
    mn = from_key(key[0]);
    mx = from_key(col[last * stride]);
    lo = from_key(col[(last >> 1) * stride]);
    hi = from_key(col[(cg >> 1) * stride]);
}

// Mean and standard deviation of one quantity for the three groups -> dst[k * ds], k = 10 * group (+ 1 for the
// deviation); returns the sum over all packets.  Two ordered passes: the sums, then the squared deviations.
template <bool WORDS, int N, int KMAX>
__device__ __forceinline__ float window_sums(const float (&x)[KMAX], uint32_t valid, uint32_t m0, uint32_t m1, int m, int c0, int c1,
                                             float* dst, uint32_t ds)
{
    const bool e0 = c0 == 0, e1 = c1 == 0, ea = m == 0;
    forget_words<WORDS>(valid, m0, m1);
    float s0 = 0.f, s1 = 0.f, sa = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        sa = sa + masked<WORDS>(x[j], valid, j);
        s0 = s0 + masked<WORDS>(x[j], m0, j);
        s1 = s1 + masked<WORDS>(x[j], m1, j);
    }
    const float n0 = (float)(c0 > 0 ? c0 : 1), n1 = (float)(c1 > 0 ? c1 : 1), na = (float)(m > 0 ? m : 1);
    const float u0 = s0 / n0, u1 = s1 / n1, ua = sa / na;
    forget_words<WORDS>(valid, m0, m1);
    float q0 = 0.f, q1 = 0.f, qa = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        float ug;
        if (WORDS) {
            const uint32_t w1 = bit_word(m1, j);
            ug = __uint_as_float((w1 & __float_as_uint(u1)) | (~w1 & __float_as_uint(u0)));
        } else {
            ug = bit_of(m1, j) ? u1 : u0;
        }
        const float da = x[j] - ua, dg = x[j] - ug;
        const float da2 = da * da, dg2 = dg * dg;
        qa = qa + masked<WORDS>(da2, valid, j);
        q0 = q0 + masked<WORDS>(dg2, m0, j);
        q1 = q1 + masked<WORDS>(dg2, m1, j);
    }
    const float v0 = q0 / n0, v1 = q1 / n1, va = qa / na;
    dst[0 * ds] = e0 ? 0.f : u0;
    dst[1 * ds] = e0 ? 0.f : sqrtf(v0);
    dst[10 * ds] = e1 ? 0.f : u1;
    dst[11 * ds] = e1 ? 0.f : sqrtf(v1);
    dst[20 * ds] = ea ? 0.f : ua;
    dst[21 * ds] = ea ? 0.f : sqrtf(va);
    return sa;
}

// Smallest, largest and median packet size of the three groups -> dst[k * ds], k = 10 * group + 0, 1, 2: sizes as
// 16-bit integers (exact in binary32).
template <bool WORDS, int N, int KMAX>
__device__ __forceinline__ void window_order_sizes(const float (&s)[KMAX], uint32_t valid, uint32_t m1, int m, int c0, int c1,
                                                   uint32_t* col, uint32_t stride, float* dst, uint32_t ds)
{
    uint32_t v[N], a[3], b[3], c[3], d[3];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = (uint32_t)s[i];
    order_stats3<WORDS, N, 16>(v, valid, m1, m, c0, c1, col, stride, a, b, c, d);
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        const int cg = g == 0 ? c0 : (g == 1 ? c1 : m);
        const float lo = (float)c[g], hi = (float)d[g];
        const float two = lo + hi;
        dst[(10 * g + 0) * ds] = cg == 0 ? 0.f : (float)a[g];
        dst[(10 * g + 1) * ds] = cg == 0 ? 0.f : (float)b[g];
        dst[(10 * g + 2) * ds] = cg == 0 ? 0.f : ((cg & 1) ? hi : two * 0.5f);
    }
}

// The same for the times; signed_times: wave-uniform, some lane of the wave holds a time with its sign bit set.
template <bool WORDS, int N, int KMAX>
__device__ __forceinline__ void window_order_times(const float (&t)[KMAX], uint32_t valid, uint32_t m0, uint32_t m1, int m, int c0,
                                                   int c1, bool signed_times, uint32_t* col, uint32_t stride, float* dst, uint32_t ds)
{
    if (!signed_times) {
        uint32_t v[N], a[3], b[3], c[3], d[3];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = __float_as_uint(t[i]);
        order_stats3<WORDS, N, 31>(v, valid, m1, m, c0, c1, col, stride, a, b, c, d);
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            const int cg = g == 0 ? c0 : (g == 1 ? c1 : m);
            const float lo = __uint_as_float(c[g]), hi = __uint_as_float(d[g]);
            const float two = lo + hi;
            dst[(10 * g + 0) * ds] = cg == 0 ? 0.f : __uint_as_float(a[g]);
            dst[(10 * g + 1) * ds] = cg == 0 ? 0.f : __uint_as_float(b[g]);
            dst[(10 * g + 2) * ds] = cg == 0 ? 0.f : ((cg & 1) ? hi : two * 0.5f);
        }
    } else {
#pragma unroll 1
        for (int g = 0; g < 3; ++g) {
            const uint32_t gm = g == 0 ? m0 : (g == 1 ? m1 : valid);
            const int cg = g == 0 ? c0 : (g == 1 ? c1 : m);
            float mn, mx, lo, hi;
            order_stats_signed<N, KMAX>(t, gm, cg, col, stride, mn, mx, lo, hi);
            const float two = lo + hi;
            dst[(10 * g + 0) * ds] = cg == 0 ? 0.f : mn;
            dst[(10 * g + 1) * ds] = cg == 0 ? 0.f : mx;
            dst[(10 * g + 2) * ds] = cg == 0 ? 0.f : ((cg & 1) ? hi : two * 0.5f);
        }
    }
}

// The 32 statistics of one prefix window of m <= N packets -> dst[k * ds], k = 10*g + 5*q + stat, then
// total bytes (k = 30) and packet count (k = 31).  Each result is stored as soon as it is known (the
// sorting networks need the registers).  signed_times: wave-uniform, some lane of the wave holds a time
// with its sign bit set.  dst and col must not overlap.
template <bool WORDS, int N, int KMAX>
__device__ __forceinline__ void window_stats(const float (&s)[KMAX], const float (&t)[KMAX], uint32_t dmask, int m,
                                             bool signed_times, uint32_t* col, uint32_t stride, float* dst, uint32_t ds)
{
    static_assert(N <= KMAX, "window network larger than the register file of the flow");
    static_assert(N <= 32, "packets of a window are the bits of a word");
    const uint32_t valid = m >= 32 ? ~0u : ((1u << m) - 1u);
    const uint32_t m1 = dmask & valid, m0 = ~dmask & valid;
    const int c1 = __popc(m1), c0 = m - c1;
    const float bytes = window_sums<WORDS, N, KMAX>(s, valid, m0, m1, m, c0, c1, dst, ds);
    window_sums<WORDS, N, KMAX>(t, valid, m0, m1, m, c0, c1, dst + 5 * ds, ds);
    dst[30 * ds] = bytes; // every partial sum is an integer below 2^24, so this is exact
    dst[31 * ds] = (float)m;
    window_order_sizes<WORDS, N, KMAX>(s, valid, m1, m, c0, c1, col, stride, dst + 2 * ds, ds);
    window_order_times<WORDS, N, KMAX>(t, valid, m0, m1, m, c0, c1, signed_times, col, stride, dst + 7 * ds, ds);
}

} // namespace sffeat
