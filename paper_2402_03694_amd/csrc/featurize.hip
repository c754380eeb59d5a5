// Step 1: per-flow statistics of the first k packets (context length k, Section 3.1 of the
// paper) and the unpacking of raw header bits (Section 4.1).
//
// One lane owns one flow and keeps its packets in registers; the statistics of a window are
// computed by the shared device code in featurize_core.h (ordered sums, one sorting network and
// one merge stage per quantity for the order statistics), so the result does not depend on how
// flows are spread over lanes.  A window of more than 32 packets is worked on by the whole wave
// (a sort across the lanes; see below).  Where lanes are few or flows ragged, four waves split the statistics of 64
// flows instead (featurize_parts).  Feature rows are staged in shared memory per window and written out as full
// 128-byte runs.
#include "common.h"
#include "featurize_core.h"

namespace {

constexpr int kWave = 64;      // flows per block (one wave)
constexpr int kRow = 33;       // staged row stride in floats (32 + 1 keeps lanes on distinct banks)

struct FeatArgs {
    uint32_t n_flows;
    uint32_t n_pkts;
    const uint32_t* off;
    const uint16_t* size;
    const float* iat;
    const uint8_t* dir;
    uint32_t n_windows;
    uint32_t depth[SF_MAX_WINDOWS];
    float* feat;
    uint32_t ld;
    uint32_t wide_ok; // the packet arrays start on 16-byte (size, time) and 8-byte (direction) boundaries
    uint32_t store16; // feat is 16-byte aligned and ld a multiple of 4: rows can be written in 16-byte pieces
};

__device__ __forceinline__ void flow_range(const FeatArgs& a, uint32_t i, uint32_t& o, uint32_t& n)
{
    uint32_t b = a.off[i], e = a.off[i + 1];
    b = b < a.n_pkts ? b : a.n_pkts; // clamp: malformed offsets must not leave the arrays
    e = e < a.n_pkts ? e : a.n_pkts;
    e = e < b ? b : e;
    o = b;
    n = e - b;
}

// ---- windows deeper than 32 packets ---------------------------------------------------------------------
// A lane keeps at most 32 packets in registers (a 64-element network per lane needs more registers than a
// lane has, and its straight-line code no longer fits the instruction cache).  A flow whose window holds
// more than 32 packets is worked on by the whole wave instead, in two steps:
//   order statistics  lane p holds packet p; six arrays (quantity x group, padded with the largest key) are
//                     sorted at once by a bitonic network across the lanes, and the flow's values are parked
//                     in shared memory;
//   ordered sums      for up to kSlots parked flows at once: six lanes per flow, each walking one
//                     (quantity, group) chain packet by packet.
// The arithmetic per value is the one of sffeat::window_stats.

constexpr uint32_t kSlots = 10;                 // flows whose chains run side by side (6 lanes each)
constexpr uint32_t kSlotWords = 2 * kWave + 8;  // parked per flow: 64 sizes, 64 times, then lane, packets, direction mask

__device__ __forceinline__ uint32_t lane_value(uint32_t x, int p) { return (uint32_t)__builtin_amdgcn_readlane((int)x, p); }

// the value of lane (lane ^ J): within four lanes and across half a row of 16 by a data-parallel move,
// otherwise through the shared-memory crossbar
template <uint32_t J>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t v)
{
    if (J == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    if (J == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
    if (J == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false); // row_ror:8
    return (uint32_t)__shfl_xor((int)v, (int)J, kWave);
}

template <uint32_t K, uint32_t J>
__device__ __forceinline__ void sort6_step(uint32_t (&key)[6], uint32_t lane)
{
    const bool up = (lane & K) == 0; // (K = 64: every lane)
    const bool lower = (lane & J) == 0;
    uint32_t other[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) other[c] = from_lane_xor<J>(key[c]);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        const uint32_t lo = key[c] < other[c] ? key[c] : other[c], hi = key[c] < other[c] ? other[c] : key[c];
        key[c] = lower == up ? lo : hi;
    }
}
template <uint32_t K, uint32_t J>
__device__ __forceinline__ void sort6_merge(uint32_t (&key)[6], uint32_t lane)
{
    sort6_step<K, J>(key, lane);
    if constexpr (J > 1) sort6_merge<K, J / 2>(key, lane);
}
// Six independent arrays of one key per lane, each sorted ascending by lane; the six exchanges of a step are
// issued together so that their latencies overlap.
__device__ __forceinline__ void wave_sort6(uint32_t (&key)[6], uint32_t lane)
{
    sort6_merge<2, 1>(key, lane);
    sort6_merge<4, 2>(key, lane);
    sort6_merge<8, 4>(key, lane);
    sort6_merge<16, 8>(key, lane);
    sort6_merge<32, 16>(key, lane);
    sort6_merge<64, 32>(key, lane);
}

// lane p's packet of a window of m packets that start at packet o (zeros past the window), as loaded: nothing
// is computed from it here, so that the request can be issued a whole flow ahead of its use
struct LanePacket {
    uint32_t sz, d;
    float tm;
};
__device__ __forceinline__ LanePacket long_flow_load(const FeatArgs& a, uint32_t o, int m, uint32_t lane)
{
    LanePacket r = {0u, 0u, 0.f};
    if ((int)lane < m) {
        r.sz = a.size[o + lane];
        r.tm = a.iat[o + lane];
        r.d = a.dir[o + lane];
    }
    return r;
}

// Sort keys of a window of m packets (32 < m <= 64), lane p holding packet p: array c = 3 * quantity + group,
// padded with the largest key; c0 / c1: packets of direction 0 / 1.  The values are parked in slot[] for the
// chains.  Every lane of the wave takes part, m and src_lane are the same in all of them.
__device__ __forceinline__ void long_flow_keys(const LanePacket& pk, int m, uint32_t src_lane, uint32_t lane, uint32_t* slot,
                                               uint32_t (&key)[6], int& c0, int& c1)
{
    const bool valid = (int)lane < m;
    const float sz = (float)pk.sz, tm = pk.tm;
    const uint32_t d = pk.d & 1u;
    const uint64_t vmask = __ballot(valid), m1 = __ballot(valid && d != 0), m0 = vmask & ~m1;
    c1 = __popcll(m1);
    c0 = m - c1;
    slot[lane] = __float_as_uint(sz);
    slot[kWave + lane] = __float_as_uint(tm);
    if (lane == 0u) {
        slot[2 * kWave + 0] = src_lane;
        slot[2 * kWave + 1] = (uint32_t)m;
        slot[2 * kWave + 2] = (uint32_t)m1;
        slot[2 * kWave + 3] = (uint32_t)(m1 >> 32);
    }
#pragma unroll
    for (uint32_t c = 0; c < 6u; ++c) {
        const uint32_t g = c % 3u, q = c / 3u;
        const uint64_t gm = g == 0 ? m0 : (g == 1 ? m1 : vmask);
        const bool in = (gm >> lane) & 1ull;
        key[c] = in ? (q ? sffeat::order_key(tm) : (uint32_t)sz) : 0xFFFFFFFFu;
    }
}

// Order statistics from the keys -> dst[10g + 5q + 2..4]
__device__ __forceinline__ void long_flow_order_stats(uint32_t (&key)[6], int m, int c0, int c1, uint32_t lane, float* dst)
{
    wave_sort6(key, lane);
#pragma unroll
    for (uint32_t c = 0; c < 6u; ++c) {
        const uint32_t g = c % 3u, q = c / 3u;
        const int cg = g == 0 ? c0 : (g == 1 ? c1 : m);
        const int last = cg > 0 ? cg - 1 : 0;
        const uint32_t k_mn = lane_value(key[c], 0), k_mx = lane_value(key[c], last);
        const uint32_t k_lo = lane_value(key[c], last >> 1), k_hi = lane_value(key[c], cg >> 1);
        const float mn = q ? sffeat::from_key(k_mn) : (float)k_mn, mx = q ? sffeat::from_key(k_mx) : (float)k_mx;
        const float lo = q ? sffeat::from_key(k_lo) : (float)k_lo, hi = q ? sffeat::from_key(k_hi) : (float)k_hi;
        const float two = lo + hi;
        if (lane == 0u) {
            dst[10u * g + 5u * q + 2u] = cg == 0 ? 0.f : mn;
            dst[10u * g + 5u * q + 3u] = cg == 0 ? 0.f : mx;
            dst[10u * g + 5u * q + 4u] = cg == 0 ? 0.f : ((cg & 1) ? hi : two * 0.5f);
        }
    }
}

// Means, standard deviations, byte and packet counts of the n_slots parked flows -> their staged rows
// (tile + lane_of_flow * kRow).  Lane 6k + c carries chain c (quantity c / 3, group c % 3) of slot k.
__device__ __forceinline__ void long_flow_chains(const uint32_t* park, uint32_t n_slots, uint32_t lane, float* tile)
{
    const uint32_t k = lane / 6u, c = lane - 6u * k;
    if (k >= n_slots) return;
    const uint32_t g = c % 3u, q = c / 3u;
    const uint32_t* slot = park + k * kSlotWords;
    const uint32_t src_lane = slot[2 * kWave + 0];
    const int m = (int)slot[2 * kWave + 1];
    const uint64_t m1 = (uint64_t)slot[2 * kWave + 2] | ((uint64_t)slot[2 * kWave + 3] << 32);
    const uint64_t valid = m >= 64 ? ~0ull : ((1ull << m) - 1ull);
    const uint64_t in_mask = g == 0 ? valid & ~m1 : (g == 1 ? m1 : valid);
    const int cg = __popcll(in_mask);
    const float ng = (float)(cg > 0 ? cg : 1);
    const float* x = reinterpret_cast<const float*>(slot) + q * kWave;
    float sum = 0.f;
    for (int p = 0; p < kWave; p += 4) {
        const float4 v = *reinterpret_cast<const float4*>(x + p);
        const uint32_t in4 = (uint32_t)(in_mask >> p) & 15u;
        sum = sum + ((in4 & 1u) ? v.x : 0.f);
        sum = sum + ((in4 & 2u) ? v.y : 0.f);
        sum = sum + ((in4 & 4u) ? v.z : 0.f);
        sum = sum + ((in4 & 8u) ? v.w : 0.f);
    }
    const float mean = sum / ng;
    float acc = 0.f;
    for (int p = 0; p < kWave; p += 4) {
        const float4 v = *reinterpret_cast<const float4*>(x + p);
        const uint32_t in4 = (uint32_t)(in_mask >> p) & 15u;
        const float d0 = v.x - mean, d1 = v.y - mean, d2 = v.z - mean, d3 = v.w - mean;
        const float e0 = d0 * d0, e1 = d1 * d1, e2 = d2 * d2, e3 = d3 * d3;
        acc = acc + ((in4 & 1u) ? e0 : 0.f);
        acc = acc + ((in4 & 2u) ? e1 : 0.f);
        acc = acc + ((in4 & 4u) ? e2 : 0.f);
        acc = acc + ((in4 & 8u) ? e3 : 0.f);
    }
    const float var = acc / ng;
    float* dst = tile + src_lane * kRow;
    dst[10u * g + 5u * q + 0u] = cg == 0 ? 0.f : mean;
    dst[10u * g + 5u * q + 1u] = cg == 0 ? 0.f : sqrtf(var);
    if (c == 2u) { // sizes, all packets
        dst[30] = sum;
        dst[31] = (float)m;
    }
}

// KMAX: packets a lane keeps in registers.  LONG: windows may be deeper than that (up to 64 packets); flows
// with more than KMAX packets in a window then go through long_window_stats.
// (second launch bound: waves per SIMD the register allocation aims for.  Three up to 16 packets per flow.
// Two with 32 packets, in 231 registers and none spilled: two waves cover each other's memory latency; three would leave
// a lane 168.  One where long flows go through the whole-wave path: that kernel's time is
// a single wave's latency, which spills only lengthen.)
template <int KMAX, bool LONG>
__global__ __launch_bounds__(kWave, (KMAX <= 16 ? 3 : (LONG ? 1 : 2))) void featurize_wave(FeatArgs a)
{
    constexpr bool WORDS = KMAX > 16; // form of the group masks, see featurize_core.h
    static_assert(!LONG || KMAX == 32, "the whole-wave path takes over above 32 packets");
    __shared__ uint32_t sort_col[KMAX * kWave]; // [rank][lane]
    __shared__ float tile[kWave * kRow];        // [lane][33]
    const uint32_t lane = threadIdx.x;
    const uint32_t tile0 = blockIdx.x * kWave;
    const uint32_t i = tile0 + lane;
    const bool live = i < a.n_flows;
    uint32_t o = 0, n = 0;
    if (live) flow_range(a, i, o, n);
    const uint32_t dmax = a.depth[a.n_windows - 1];
    const int avail_w = (int)(n < dmax ? n : dmax);              // packets of the deepest window
    const int avail = avail_w < KMAX ? avail_w : KMAX;           // of which the lane holds in registers
    float s[KMAX], t[KMAX];
    uint32_t dmask = 0;
    if (avail == KMAX && (o & 7u) == 0 && a.wide_ok) {
        // whole window present and 16-byte aligned (array bases included): wide loads
        sffeat::RawPackets<KMAX> raw;
        sffeat::load_wide<KMAX>(a.size, a.iat, a.dir, o, raw);
        sffeat::decode_wide<KMAX>(raw, s, t, dmask);
    } else {
        sffeat::load_each<KMAX>(a.size, a.iat, a.dir, o, avail, s, t, dmask);
    }
    // a time with its sign bit set anywhere in the wave: the order statistics take the general path
    uint32_t sign_bits = 0;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) sign_bits |= __float_as_uint(t[j]);
    const bool signed_times = __any((int)(sign_bits >> 31));
    uint32_t* col = sort_col + lane;
    float* row = tile + lane * kRow;
    uint32_t rows = a.n_flows - tile0;
    rows = rows < (uint32_t)kWave ? rows : (uint32_t)kWave;
    for (uint32_t w = 0; w < a.n_windows; ++w) {
        const int dw = (int)a.depth[w];
        const int m_w = avail_w < dw ? avail_w : dw;
        const bool long_flow = LONG && m_w > KMAX;
        const int m = long_flow ? 0 : m_w; // (the lane's own result for such a flow is overwritten below)
        // the smallest network that covers every lane's window (wave-uniform choice)
        if (KMAX >= 32 && __any(m > 16))
            sffeat::window_stats<WORDS, (KMAX >= 32 ? 32 : KMAX), KMAX>(s, t, dmask, m, signed_times, col, kWave, row, 1u);
        else if (KMAX >= 16 && __any(m > 8))
            sffeat::window_stats<WORDS, (KMAX >= 16 ? 16 : KMAX), KMAX>(s, t, dmask, m, signed_times, col, kWave, row, 1u);
        else
            sffeat::window_stats<WORDS, 8, KMAX>(s, t, dmask, m, signed_times, col, kWave, row, 1u);
        if (LONG) {
            // (the sort scratch of the lanes' own windows is free by now: the long flows' values are parked there)
            static_assert(!LONG || kSlots * kSlotWords <= (uint32_t)KMAX * kWave, "parked flows fit the sort scratch");
            uint64_t todo = __ballot(long_flow);
            // the packets of the next long flow are requested while the current one is sorted
            int l = todo ? __ffsll((unsigned long long)todo) - 1 : 0;
            int m_l = todo ? (int)lane_value((uint32_t)m_w, l) : 0;
            LanePacket cur = long_flow_load(a, lane_value(o, l), m_l, lane);
            while (todo) {
                uint32_t n_slots = 0;
                while (todo && n_slots < kSlots) {
                    todo &= todo - 1ull;
                    const int l_next = todo ? __ffsll((unsigned long long)todo) - 1 : 0;
                    const int m_next = todo ? (int)lane_value((uint32_t)m_w, l_next) : 0;
                    uint32_t key[6];
                    int c0, c1;
                    long_flow_keys(cur, m_l, (uint32_t)l, lane, sort_col + n_slots * kSlotWords, key, c0, c1);
                    // (requested only now, behind the wait for the current flow's packets, and pinned here: the
                    // request then flies while the current flow is sorted)
                    __builtin_amdgcn_sched_barrier(0);
                    const LanePacket next = long_flow_load(a, lane_value(o, l_next), m_next, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    long_flow_order_stats(key, m_l, c0, c1, lane, tile + l * kRow);
                    ++n_slots;
                    cur = next;
                    l = l_next;
                    m_l = m_next;
                }
                long_flow_chains(sort_col, n_slots, lane, tile);
            }
        }
        __syncthreads();
        if (a.store16) {
            // eight lanes write one staged row (32 consecutive floats = one 128-byte run) as 16-byte pieces:
            // a store instruction of the wave covers eight rows
            const uint32_t c4 = (lane & 7u) * 4u;
            for (uint32_t r = lane >> 3; r < rows; r += 8u) {
                const float* src = tile + r * kRow + c4;
                *reinterpret_cast<float4*>(a.feat + (size_t)(tile0 + r) * a.ld + 32u * w + c4) =
                    make_float4(src[0], src[1], src[2], src[3]);
            }
        } else {
            // half a wave writes one staged row, a float per lane
            const uint32_t c = lane & 31u, half = lane >> 5;
            for (uint32_t r = half; r < rows; r += 2)
                a.feat[(size_t)(tile0 + r) * a.ld + 32u * w + c] = tile[r * kRow + c];
        }
        __syncthreads();
    }
}

// Staged packets of a tile: one column per flow, rows 0..KMAX-1 the sizes, KMAX..2 KMAX-1 the times, then the
// direction bits and the packet count.  Four words of padding per row: the lanes of a wave that write a row pair
// each for eight flows then fall on 64 different banks.
__host__ __device__ constexpr uint32_t stage_stride(uint32_t fpb) { return fpb + 4u; }
__host__ __device__ constexpr uint32_t stage_words(uint32_t kmax, uint32_t fpb) { return (2u * kmax + 2u) * stage_stride(fpb); }

// (The fused feature + forest kernel has a staging and a part of its own: sharing these two functions with it moved its
// blocks and made its whole pass 0.5 % slower, 703 -> 707 us on 1,048,576 flows.)
// One part of one window's statistics for one flow per lane: kind 0 / 2: sums of sizes / times, kind 1 / 3: order
// statistics of sizes / times.  x: the quantity; col: scratch column, a word every `stride`; dst: where the window's
// statistics go, one every `ds` floats.
template <int N, int KMAX>
__device__ __forceinline__ void window_part(uint32_t kind, const float (&x)[KMAX], uint32_t dmask, int m, uint32_t* col, uint32_t stride,
                                            float* dst, uint32_t ds)
{
    const uint32_t valid = N >= 32 && m >= 32 ? ~0u : (1u << m) - 1u, m1 = dmask & valid, m0 = ~dmask & valid;
    const int c1 = __popc(m1), c0 = m - c1;
    if ((kind & 1u) == 0u) {
        const float sum = sffeat::window_sums<true, N, KMAX>(x, valid, m0, m1, m, c0, c1, dst + (kind ? 5u : 0u) * ds, ds);
        if (kind == 0u) {
            dst[30u * ds] = sum; // (bytes: every partial sum is an integer below 2^24, so this is exact)
            dst[31u * ds] = (float)m;
        }
    } else if (kind == 1u) {
        sffeat::window_order_sizes<true, N, KMAX>(x, valid, m1, m, c0, c1, col, stride, dst + 2u * ds, ds);
    } else {
        // a time with its sign bit set anywhere in the wave: the order statistics take the general path
        uint32_t sign_bits = 0;
#pragma unroll
        for (int j = 0; j < KMAX; ++j) sign_bits |= __float_as_uint(x[j]);
        const bool signed_times = __any((int)(sign_bits >> 31));
        sffeat::window_order_times<true, N, KMAX>(x, valid, m0, m1, m, c0, c1, signed_times, col, stride, dst + 7u * ds, ds);
    }
}

// Fetches the packets of flows flow0 .. flow0 + FPB - 1 (up to dmax <= KMAX of each) into the staged form, by a block of BS
// lanes, several pieces per lane.
template <uint32_t FPB, uint32_t BS, int KMAX>
__device__ __forceinline__ void stage_packets(const FeatArgs& c, uint32_t flow0, uint32_t* behind)
{
    constexpr uint32_t SS = stage_stride(FPB);
    const uint32_t n_flows = c.n_flows, dmax = c.depth[c.n_windows - 1u];
    constexpr uint32_t P = KMAX / 2; // lanes that fetch one flow's packets, two packets each
    static_assert(P <= 16 && FPB * P % BS == 0, "every flow's packets are fetched by lanes of one wave, all lanes take part");
    constexpr uint32_t IT = FPB * P / BS;
    // consecutive lanes hold consecutive packets of a flow and the flows follow each other in memory, so the loads of a
    // wave are one contiguous piece (flows longer than the window leave gaps); all offsets are requested before the first
    // packet, all packets before the first is used
    uint32_t b[IT], e[IT];
#pragma unroll
    for (uint32_t it = 0; it < IT; ++it) {
        const uint32_t f = (threadIdx.x + it * BS) / P;
        // a slot past the last flow works on the last flow (its loads stay inside the arrays)
        const uint32_t flow = flow0 + f < n_flows ? flow0 + f : n_flows - 1u;
        b[it] = c.off[flow];
        e[it] = c.off[flow + 1];
    }
    uint32_t sz[IT], dd[IT], avail[IT]; // two sizes, two direction bytes
    float2 tm[IT];
#pragma unroll
    for (uint32_t it = 0; it < IT; ++it) {
        const uint32_t q = threadIdx.x + it * BS, p = q % P;
        const uint32_t b1 = b[it] < c.n_pkts ? b[it] : c.n_pkts; // clamp: malformed offsets must not leave the arrays
        uint32_t e1 = e[it] < c.n_pkts ? e[it] : c.n_pkts;
        e1 = e1 < b1 ? b1 : e1;
        const uint32_t n = e1 - b1, o = b1 + 2u * p;
        avail[it] = n < dmax ? n : dmax;
        sz[it] = 0u;
        dd[it] = 0u;
        tm[it] = make_float2(0.f, 0.f);
        if (2u * p + 1u < avail[it] && (o & 1u) == 0 && c.wide_ok) {
            sz[it] = *reinterpret_cast<const uint32_t*>(c.size + o);
            tm[it] = *reinterpret_cast<const float2*>(c.iat + o);
            dd[it] = *reinterpret_cast<const uint16_t*>(c.dir + o);
        } else if (2u * p < avail[it]) {
            const bool two = 2u * p + 1u < avail[it];
            sz[it] = c.size[o] | (two ? (uint32_t)c.size[o + 1u] << 16 : 0u);
            tm[it] = make_float2(c.iat[o], two ? c.iat[o + 1u] : 0.f);
            dd[it] = c.dir[o] | (two ? (uint32_t)c.dir[o + 1u] << 8 : 0u);
        }
    }
#pragma unroll
    for (uint32_t it = 0; it < IT; ++it) {
        const uint32_t q = threadIdx.x + it * BS, f = q / P, p = q % P;
        uint32_t d = ((dd[it] & 1u) | ((dd[it] >> 7) & 2u)) << (2u * p);
#pragma unroll
        for (uint32_t k = 1; k < P; k *= 2) d |= (uint32_t)__shfl_xor((int)d, (int)k, 64);
        float* st = reinterpret_cast<float*>(behind) + f;
        st[(2u * p) * SS] = (float)(sz[it] & 0xFFFFu);
        st[(2u * p + 1u) * SS] = (float)(sz[it] >> 16);
        st[(KMAX + 2u * p) * SS] = tm[it].x;
        st[(KMAX + 2u * p + 1u) * SS] = tm[it].y;
        if (p == 0u) {
            behind[2u * KMAX * SS + f] = d;
            behind[(2u * KMAX + 1u) * SS + f] = avail[it];
        }
    }
}

// Windows of up to KMAX packets.  A block works on 64 flows with four waves: the packets are fetched once, coalesced, into
// shared memory; then each wave computes one independent part of every window for all 64 flows (ordered sums or order
// statistics, of sizes or times), with one quantity in registers.
// What bounds it: vector arithmetic in large batches, in small ones a wave's latency, which this makes a quarter.  With one
// lane per flow, as all batches went before and large ones still do (see sf_featurize), all four parts are one wave's
// serial chain.  The kernel, before -> after: 20,011 ragged flows, windows 3, 9, 20: 19.7 -> 13.4 us; 250,007 ragged flows,
// windows 8, 16: 37-40 -> 32.6 us; 1,048,576 of those 138 -> 133 us.  (A second tile instead of the second barrier per
// window: 13.4 -> 12.8 us and 133 -> 141; 64 registers per lane for 16 packets, eight waves per SIMD with 20 spilled:
// 133 -> 190.)
// LONG: windows may be deeper than KMAX = 32 (up to 64 packets); a flow that has more is worked on by a whole wave, see above, the
// long flows of the 64 dealt out to the four waves.  One lane per flow : this, windows 8 and 64: 97 ragged flows 25.6 : 15.6 us, 65,536 36.1 :
// 30.7; 65,536 of 64 packets 149 : 91; the rest at long_lanes_pay.
template <int KMAX, bool LONG>
__device__ __forceinline__ void feature_parts(const FeatArgs& a)
{
    static_assert(!LONG || KMAX == 32, "the whole-wave path takes over above 32 packets");
    constexpr uint32_t SS = stage_stride(kWave);
    constexpr uint32_t kStage = stage_words(KMAX, kWave), kSort = 2u * KMAX * kWave; // two of the waves sort
    constexpr uint32_t kPark = LONG ? 4u * kSlots * kSlotWords : 0u, kMost = kStage > kSort ? kStage : kSort;
    __shared__ uint32_t space[kMost > kPark ? kMost : kPark];
    __shared__ float tile[kWave * kRow]; // [lane][33]
    const uint32_t tid = threadIdx.x, slot = tid % kWave, flow0 = blockIdx.x * kWave;
    const uint32_t kind = __builtin_amdgcn_readfirstlane(tid / kWave);
    stage_packets<kWave, 4 * kWave, KMAX>(a, flow0, space);
    __syncthreads();
    float x[KMAX];
    const float* st = reinterpret_cast<const float*>(space) + slot + (kind >> 1) * KMAX * SS;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) x[j] = st[j * SS];
    const uint32_t dmask = space[2u * KMAX * SS + slot];
    const int avail = (int)space[(2u * KMAX + 1u) * SS + slot];
    __syncthreads(); // the staged packets are in registers: their space is scratch now
    uint32_t o = 0; // where a long flow's packets start
    if (LONG && flow0 + slot < a.n_flows) {
        uint32_t n;
        flow_range(a, flow0 + slot, o, n);
    }
    uint32_t* col = space + (kind >> 1) * (KMAX * kWave) + slot; // the lane's own column
    float* row = tile + slot * kRow;
    uint32_t rows = a.n_flows - flow0;
    rows = rows < (uint32_t)kWave ? rows : (uint32_t)kWave;
#pragma unroll 1
    for (uint32_t w = 0; w < a.n_windows; ++w) {
        // nothing made from the packets for one window is kept for another (registers)
#pragma unroll
        for (int j = 0; j < KMAX; ++j) asm volatile("" : "+v"(x[j]));
        const int dw = (int)a.depth[w];
        const int m_w = avail < dw ? avail : dw;
        const bool long_flow = LONG && m_w > KMAX && flow0 + slot < a.n_flows;
        const int m = LONG && m_w > KMAX ? 0 : m_w; // (what the lane makes of such a flow is overwritten below)
        // the smallest network that covers every lane's window (wave-uniform choice)
        if (KMAX >= 32 && __any(m > 16))
            window_part<KMAX, KMAX>(kind, x, dmask, m, col, kWave, row, 1u);
        else if (KMAX >= 16 && __any(m > 8))
            window_part<(KMAX >= 16 ? 16 : KMAX), KMAX>(kind, x, dmask, m, col, kWave, row, 1u);
        else
            window_part<8, KMAX>(kind, x, dmask, m, col, kWave, row, 1u);
        __syncthreads();
        if (LONG && __ballot(long_flow) != 0ull) { // (the same flows in all four waves)
            // (the sort columns are free by now: the long flows' values are parked there)
            uint32_t* park = space + kind * (kSlots * kSlotWords);
            uint64_t todo = __ballot(long_flow), mine = 0;
            for (uint32_t q = 0; todo; ++q) { // every fourth is this wave's
                const uint64_t low = todo & (0ull - todo);
                todo ^= low;
                if ((q & 3u) == kind) mine |= low;
            }
            if (mine) {
                const uint32_t lane = slot;
                // the packets of the next long flow are requested while the current one is sorted
                int l = __ffsll((unsigned long long)mine) - 1;
                int m_l = (int)lane_value((uint32_t)m_w, l);
                LanePacket cur = long_flow_load(a, lane_value(o, l), m_l, lane);
                while (mine) {
                    uint32_t n_slots = 0;
                    while (mine && n_slots < kSlots) {
                        mine &= mine - 1ull;
                        const int l_next = mine ? __ffsll((unsigned long long)mine) - 1 : 0;
                        const int m_next = mine ? (int)lane_value((uint32_t)m_w, l_next) : 0;
                        uint32_t key[6];
                        int c0, c1;
                        long_flow_keys(cur, m_l, (uint32_t)l, lane, park + n_slots * kSlotWords, key, c0, c1);
                        // (requested only now, behind the wait for the current flow's packets, and pinned here: the
                        // request then flies while the current flow is sorted)
                        __builtin_amdgcn_sched_barrier(0);
                        const LanePacket next = long_flow_load(a, lane_value(o, l_next), m_next, lane);
                        __builtin_amdgcn_sched_barrier(0);
                        long_flow_order_stats(key, m_l, c0, c1, lane, tile + l * kRow);
                        ++n_slots;
                        cur = next;
                        l = l_next;
                        m_l = m_next;
                    }
                    long_flow_chains(park, n_slots, lane, tile);
                }
            }
            __syncthreads();
        }
        if (a.store16) {
            // eight lanes write one staged row (32 consecutive floats = one 128-byte run) as 16-byte pieces
            const uint32_t c4 = (tid & 7u) * 4u;
            for (uint32_t r = tid >> 3; r < rows; r += kWave / 2) {
                const float* src = tile + r * kRow + c4;
                *reinterpret_cast<float4*>(a.feat + (size_t)(flow0 + r) * a.ld + 32u * w + c4) =
                    make_float4(src[0], src[1], src[2], src[3]);
            }
        } else {
            // half a wave writes one staged row, a float per lane
            for (uint32_t r = tid >> 5; r < rows; r += kWave / 8)
                a.feat[(size_t)(flow0 + r) * a.ld + 32u * w + (tid & 31u)] = tile[r * kRow + (tid & 31u)];
        }
        __syncthreads();
    }
}

template <int KMAX>
__global__ __launch_bounds__(4 * kWave, KMAX == 8 ? 8 : KMAX == 16 ? 6 : 4) void featurize_parts(FeatArgs a)
{
    feature_parts<KMAX, false>(a);
}
// WAVES per SIMD asked of the compiler: 4 leave 128 registers, 13 spilled; 2 take 144 (three blocks a unit) and spill none, which pays while
// the blocks are no more than that: windows 8 and 64, 97 ragged flows 15.9 -> 14.2 us, 16,384 17.4 -> 15.7, 49,152 24.7 -> 23.5, 41,000 of 40 packets
// 73.8 -> 72.7; with four blocks a unit it is the other way, 65,536 30.1 : 31.5, 300,000 of 40 packets 358 : 389.
template <int WAVES>
__global__ __launch_bounds__(4 * kWave, WAVES) void featurize_long(FeatArgs a)
{
    feature_parts<32, true>(a);
}

// Raw header bits -> one byte per bit.  A thread unpacks one header word (32 features).
__global__ __launch_bounds__(256) void unpack_raw(uint32_t n_flows, uint32_t n_pkts, const uint32_t* __restrict__ off,
                                                  const uint32_t* __restrict__ hdr, uint32_t hdr_words,
                                                  uint32_t raw_pkts, uint32_t raw_bits, uint8_t* __restrict__ raw)
{
    const uint32_t words = (raw_bits + 31) / 32; // words per packet that carry features
    const uint64_t total = (uint64_t)n_flows * raw_pkts * words;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
         g += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t wq = (uint32_t)(g % words);
        const uint64_t fp = g / words;
        const uint32_t j = (uint32_t)(fp % raw_pkts);
        const uint32_t i = (uint32_t)(fp / raw_pkts);
        uint32_t b = off[i], e = off[i + 1];
        b = b < n_pkts ? b : n_pkts;
        e = e < n_pkts ? e : n_pkts;
        const uint32_t n = e > b ? e - b : 0;
        const uint32_t word = j < n ? hdr[(size_t)(b + j) * hdr_words + wq] : 0u;
        uint8_t* dst = raw + ((size_t)i * raw_pkts + j) * raw_bits + 32u * wq;
        const uint32_t nb = raw_bits - 32u * wq < 32u ? raw_bits - 32u * wq : 32u;
        for (uint32_t k = 0; k < nb; ++k) {
            // feature bit 32*wq + k: byte k/8 of the word, bit 7-(k%8) of that byte
            dst[k] = (uint8_t)((word >> (8u * (k >> 3) + 7u - (k & 7u))) & 1u);
        }
    }
}

// One lane per flow or four waves per 64 flows (parts)?  Below two waves per SIMD of lanes the parts win everywhere
// (65,536 flows: 1.05 to 1.25 times as fast).  From there, lanes : parts in microseconds; "ragged": flows of
// geometric length, mean 10.
//   a deepest window of 8 or 16 packets and flows of one length that is a multiple of 8 (told from the totals, as the lengths
//     are on the device): the lanes load whole windows in 16-byte pieces.  1,048,576 flows: windows 8, 16,
//     104 : 120; window 8, 40 : 48.
//   else the lanes load packet by packet, each from its own flow, which pays as long as what they read at once stays in the
//     first-level cache:
//     up to 4 packets, and from 2,048 flows per unit up to 6 (1,048,576 ragged, window 4, 44 : 50; window 8 the other
//     way, 53 : 49);
//     up to 12 packets, or short flows, from 1,536 flows per unit (1,048,576 ragged, windows 5, 10, 120 : 133; but
//     180,000 25.1 : 24.3, and windows 8, 16, 1,048,576, 139 : 134).
//   windows of 17 to 32 packets: flows of one length that fill 32 (wide loads; 4,194,304 x 32 packets, four windows: 1.11 ms against 1.22;
//     1,000,000, windows 8, 32, 150 : 169), and short flows, up to 18 packets on average, 22 in the largest batches (1,000,000 ragged with a mean
//     of 10, windows 8, 20, 170 : 210; of 17 191 : 222, with windows 8, 16, 24, 32 341 : 340; 2,000,000 of 20 packets 338 : 345).  The others read
//     packet by packet past the first-level cache: 1,000,000 of 20 packets, windows 8, 20, 186 : 178, of 24, windows 8, 24, 214 : 178, of 50,
//     windows 10, 30, 484 : 194; ragged with a mean of 25, windows 8, 32, 265 : 228; 131,072 of them 42.5 : 32.5.
bool one_lane_pays(uint32_t dmax, uint32_t per_unit, uint32_t n_flows, uint64_t n_pkts)
{
    if (per_unit < 2u * 4u * kWave) return false;
    const uint64_t len = n_pkts / n_flows;
    if (dmax > 16) return n_pkts <= (per_unit >= 6000u ? 22ull : 18ull) * n_flows || (dmax == 32 && n_pkts % n_flows == 0 && len % 8u == 0 && len >= 32);
    if (dmax % 8u == 0 && n_pkts % n_flows == 0 && len % 8u == 0 && len >= dmax) return true;
    if (dmax <= 8) return dmax <= 4 || (dmax <= 6 && per_unit >= 2048u);
    return per_unit >= 1536u && (dmax <= 12 || (dmax < 16 && n_pkts <= 12ull * n_flows));
}

// The same for windows deeper than 32 packets: lanes where most waves have no long flow and the batch is large enough that one
// wave's chain of latencies no longer counts, the later the longer the flows.  Lanes : parts, us.
//   flows of one length (none longer than 32), from 192 flows a unit up to 12 packets (123,008 of 4, window 64, 10.7 : 16.9; 50,800 of 12 9.5 :
//     11.0), from 320 up to 15 (121,512 of 13, windows 18 and 64, 24.4 : 31.5), from 768 of 16, from 1,536 above (1,170,295 of 24, windows 2, 16, 64, 293 : 401; 457,367 of 20, four windows, 164 : 201; but
//     120,000 of 24 1.28 times as long), and from 320 where they fill 32 (wide loads; 1,199,700, window 64, 136 : 237);
//   ragged ones by their mean: up to 2 packets 256 flows a unit, 8 384 (108,635 of 4.8, windows 3 and 42, 28.4 : 33.7), 12 512 (262,144 of 10, windows 8 and
//     64, 79.5 : 92.8), 15 1,024, 18 2,048 (1,042,169 of 16.9, windows 8, 29, 64, 501 : 563); but a mean of 17, 131,072 flows, 82.9 : 69.3, 400,000
//     181 : 169, of 25 267 : 213.
// Flows longer than 32 packets go in parts: 262,144 of 64, window 64, 387 : 287; 300,000 of 50, windows 20 and 50, 565 : 358.
bool long_lanes_pay(uint32_t per_unit, uint32_t n_flows, uint64_t n_pkts)
{
    const uint64_t len = n_pkts / n_flows;
    if (n_pkts % n_flows == 0) return len <= 32 && per_unit >= (len <= 12 ? 192u : len <= 15 || len == 32 ? 320u : len == 16 ? 768u : 1536u);
    const auto mean_to = [=](uint32_t m) { return n_pkts <= (uint64_t)m * n_flows; };
    return mean_to(18) && per_unit >= (mean_to(2) ? 256u : mean_to(8) ? 384u : mean_to(12) ? 512u : mean_to(15) ? 1024u : 2048u);
}

} // namespace

extern "C" int sf_featurize(sf_ctx* ctx, const sf_packets* pk, const sf_feat_cfg* cfg, float* feat,
                            uint32_t feat_ld, uint8_t* raw)
{
    if (!ctx) return sf::fail(nullptr, SF_EINVAL, "sf_featurize: ctx is NULL");
    if (!pk || !cfg) return sf::fail(ctx, SF_EINVAL, "sf_featurize: packets or config is NULL");
    if (cfg->n_windows < 1 || cfg->n_windows > SF_MAX_WINDOWS)
        return sf::fail(ctx, SF_EINVAL, "sf_featurize: n_windows %u outside 1..%d", cfg->n_windows, SF_MAX_WINDOWS);
    for (uint32_t w = 0; w < cfg->n_windows; ++w) {
        if (cfg->depth[w] < 1 || cfg->depth[w] > SF_MAX_DEPTH_PKTS)
            return sf::fail(ctx, SF_EINVAL, "sf_featurize: depth[%u] = %u outside 1..%d", w, cfg->depth[w],
                            SF_MAX_DEPTH_PKTS);
        if (w && cfg->depth[w] <= cfg->depth[w - 1])
            return sf::fail(ctx, SF_EINVAL, "sf_featurize: depths must be strictly increasing");
    }
    if (feat_ld < 32 * cfg->n_windows)
        return sf::fail(ctx, SF_EINVAL, "sf_featurize: feat_ld %u < %u", feat_ld, 32 * cfg->n_windows);
    if (pk->n_pkts >> 32) return sf::fail(ctx, SF_EINVAL, "sf_featurize: n_pkts exceeds 32-bit offsets");
    if (pk->n_flows == 0) return SF_OK;
    if (!feat || !pk->flow_off) return sf::fail(ctx, SF_EINVAL, "sf_featurize: feat or flow_off is NULL");
    if (pk->n_pkts && (!pk->pkt_size || !pk->pkt_iat || !pk->pkt_dir))
        return sf::fail(ctx, SF_EINVAL, "sf_featurize: packet arrays missing");
    if (raw) {
        if (!pk->pkt_hdr || pk->hdr_words == 0 || pk->hdr_words > SF_HDR_WORDS_MAX)
            return sf::fail(ctx, SF_EINVAL, "sf_featurize: raw output needs pkt_hdr with 1..%d words per packet",
                            SF_HDR_WORDS_MAX);
        if (cfg->raw_pkts == 0 || cfg->raw_bits == 0 || cfg->raw_bits > 32 * pk->hdr_words)
            return sf::fail(ctx, SF_EINVAL, "sf_featurize: raw_pkts/raw_bits do not fit the header words");
    }

    FeatArgs a;
    a.n_flows = pk->n_flows;
    a.n_pkts = (uint32_t)pk->n_pkts;
    a.off = pk->flow_off;
    a.size = pk->pkt_size;
    a.iat = pk->pkt_iat;
    a.dir = pk->pkt_dir;
    a.n_windows = cfg->n_windows;
    for (int w = 0; w < SF_MAX_WINDOWS; ++w) a.depth[w] = w < (int)cfg->n_windows ? cfg->depth[w] : 0;
    a.feat = feat;
    a.ld = feat_ld;
    a.wide_ok = (((uintptr_t)a.size | (uintptr_t)a.iat) & 15u) == 0 && ((uintptr_t)a.dir & 7u) == 0;
    a.store16 = ((uintptr_t)feat & 15u) == 0 && (feat_ld & 3u) == 0;
    const uint32_t dmax = cfg->depth[cfg->n_windows - 1];
    const uint32_t grid = (a.n_flows + kWave - 1) / kWave;
    const uint32_t per_unit = a.n_flows / (uint32_t)ctx->n_cu;
    const bool lanes = one_lane_pays(dmax, per_unit, a.n_flows, pk->n_pkts);
    if (dmax > 32 && long_lanes_pay(per_unit, a.n_flows, pk->n_pkts))
        featurize_wave<32, true><<<grid, kWave, 0, ctx->stream>>>(a);
    else if (dmax > 32 && grid <= 3u * (uint32_t)ctx->n_cu)
        featurize_long<2><<<grid, 4 * kWave, 0, ctx->stream>>>(a);
    else if (dmax > 32)
        featurize_long<4><<<grid, 4 * kWave, 0, ctx->stream>>>(a);
    else if (dmax > 16 && lanes)
        featurize_wave<32, false><<<grid, kWave, 0, ctx->stream>>>(a);
    else if (dmax > 16)
        featurize_parts<32><<<grid, 4 * kWave, 0, ctx->stream>>>(a);
    else if (dmax > 8 && lanes)
        featurize_wave<16, false><<<grid, kWave, 0, ctx->stream>>>(a);
    else if (dmax > 8)
        featurize_parts<16><<<grid, 4 * kWave, 0, ctx->stream>>>(a);
    else if (lanes)
        featurize_wave<8, false><<<grid, kWave, 0, ctx->stream>>>(a);
    else
        featurize_parts<8><<<grid, 4 * kWave, 0, ctx->stream>>>(a);
    SF_LAUNCH_CHECK(ctx, "featurize");
    if (raw) {
        const uint64_t total = (uint64_t)a.n_flows * cfg->raw_pkts * ((cfg->raw_bits + 31) / 32);
        uint64_t blocks = (total + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        unpack_raw<<<(uint32_t)blocks, 256, 0, ctx->stream>>>(a.n_flows, a.n_pkts, pk->flow_off, pk->pkt_hdr,
                                                              pk->hdr_words, cfg->raw_pkts, cfg->raw_bits, raw);
        SF_LAUNCH_CHECK(ctx, "unpack_raw");
    }
    return SF_OK;
}
