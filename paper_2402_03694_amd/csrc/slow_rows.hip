// Step 5, register form (Sections 3.1 and 4.4 of the paper: only the uncertain flows reach the slow model): up to 128 input
// values, hidden widths up to 512, long lists.  A wave takes 64 rows through all three layers with the activations in its
// registers; what moves is the weights, once per 256 rows through shared memory.
//
// Why: the tile form (slow_tiles.h) keeps 128 rows in shared memory and splits the columns over its waves, so each layer's
// activations are written out, waited for by all waves and read back, and nothing overlaps that: 34 % of the matrix rate.
// Here the weights are the first operand of v_mfma_f32_32x32x16_bf16, which leaves a lane with columns of one activation row, and with
// the weights' rows read in the order of sftiles::weight_lane these are eight consecutive columns: exactly what the lane has to supply as
// the second operand of the next layer.  So the results of 32 columns become, through relu and rounding, two operands of the next
// layer without leaving the lane; the second layer's go straight into the last layer's sums.  There is no
// exchange between waves but the weights.
//   - 4 waves a block, one per SIMD, 512 registers each: the second layer's operands of 64 rows (up to 256 registers, most of
//     them accumulation registers), two sets of sums for 32 columns (32 x 2) and the last layer's sums (32).
//   - the weights pass through shared memory in pieces of NB1 fragments (1 KB: 32 columns x 16 k), four pieces deep, each wave
//     fetching its share two pieces before it is stored; one barrier a piece, in its middle part, where nobody waits long.  A
//     fragment read feeds two MFMAs: 64 bytes a clock per unit of what shared memory gives.
//   - with one wave per SIMD what is not an MFMA has to be issued while one runs, at most seven instructions each (32 clocks).
//     The code is laid out step by step for that: the columns before pass through relu two values a step, weights, biases and
//     the next pass's input are requested and stored a few instructions a step.  (All at once between two column blocks the
//     same work took 77,000 clocks a pass instead of 55,000; 39,000 are MFMAs.)
// What bounds it: power.  263,551 rows through 64-512-512-10 176 -> 138 us, a million 609 -> 466 us (1.29 PFLOP/s, the
// clock falls to 1.8 GHz); 300,000 rows 64-128-128-10 96 -> 49, 96-300-200-10 151 -> 103, 128-512-512-10 222 -> 183 us.
// Eight waves of 32 rows each (two per SIMD, 256 registers) read every fragment twice as often and were no faster.
// A block's rows are a run of row blocks of 32, at most one more than another block's: passes of eight row blocks, then one of four
// where three or four are left, or a tile of one or two.
#include "slow_rows.h"

namespace {

using sfmlp::bf16x8;
using sfmlp::f32x16;
using sfrows::RowsArgs;

using sftiles::pack_bf16;
typedef __attribute__((ext_vector_type(4))) uint32_t v4u;

constexpr int kWaves = 4; // waves per block, one per SIMD
constexpr int kFrag = 4; // weight fragments a wave holds: this step's and the next three
constexpr int kBufs = 4; // weight pieces in shared memory

__device__ __forceinline__ bf16x8 operand(v4u x) { return __builtin_bit_cast(bf16x8, x); }
__device__ __forceinline__ v4u frag4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return v4u{a, b, c, d}; }

// NB1: column blocks of the first layer, in fours; KS1: k-steps of the first layer, 4 or 8 (as its weights are ordered); EXACT: the
// first layer has all NB1 column blocks and the second an even number, so that no piece has fragments past the end (which read
// as zeros): 2 % of the pass at 512-512, so made for that width only.
template <int NB1, int KS1, bool EXACT>
struct Rows {
    static constexpr int KS2 = 2 * NB1;        // k-steps of layer 2
    static constexpr int STAGE = NB1 / kWaves; // 16-byte elements of a piece per thread
    static constexpr int PIECES = 2 * KS1;     // input: 32 rows in requests of one 16-byte element per lane
    static constexpr int LPR = 4 * KS1;        // lanes of a request that share a row
    static constexpr int RPP = 64 / LPR;       // rows of a request
    static constexpr int AT_ONCE = NB1 <= 8 ? 4 : NB1 == 12 || (KS1 == 8 && EXACT) ? 2 : 1; // requests per column block of layer 2 (registers)
    static constexpr int RELU = 17 / (KS2 - 4) + 1;                  // pairs of results a step of layer 2 works on
    static constexpr int SYNC = NB1 - 4 > STAGE ? NB1 - 4 : NB1 - 1; // the step of a piece with the barrier
    // (for 16 column blocks of which some may be missing, eight fewer: 2 registers spilled instead of 18, 3 to 5 % faster)
    static constexpr int AREGS = 2 * KS2 - (KS1 == 4 || (NB1 == 16 && !EXACT) ? 10 : 2); // operands of layer 2 that stand in accumulation registers
    static_assert(KS1 % 4 == 0 && NB1 % 4 == 0, "pieces come in fours");
    static_assert(2 + 16 / RELU <= KS2 - 3, "the columns before are done when the operands of the last layer are replaced");

    const RowsArgs& a;
    v4u* ring; // [kBufs][NB1][64]
    v4u* xin;  // this wave's input fragments [2][KS1][64]
    const float *b1, *b2, *b3;
    uint32_t lane, wave, half, swz; // swz: lane with bits 2 and 3 exchanged
    uint32_t nb2p;
    v4u st[2][STAGE]; // pieces on their way from memory
    v4u fb[kFrag];
    float4 bias[4];     // of the next columns
    float4 mu, is;      // the input map of the lane's columns

    __device__ __forceinline__ const v4u* w1s() const { return reinterpret_cast<const v4u*>(a.w1s); }
    __device__ __forceinline__ const v4u* w2s() const { return reinterpret_cast<const v4u*>(a.w2s); }
    __device__ __forceinline__ const v4u* w3s() const { return reinterpret_cast<const v4u*>(a.w3s); }
    __device__ __forceinline__ const v4u* zeros() const { return w3s() + a.ks3 * 64u; } // (a fragment of zeros follows the last layer)

    // a piece of the weights: fragments from p on, zeros from the limit on
    struct Src {
        const v4u* p;
        uint32_t limit;
    };
    __device__ __forceinline__ Src piece1(uint32_t c) const // piece c of layer 1
    {
        const uint32_t n = a.nb1 * KS1, f = c * NB1;
        return {w1s() + (size_t)f * 64u, n > f ? n - f : 0u};
    }
    __device__ __forceinline__ Src piece2(uint32_t nb, uint32_t h) const // half h of column block nb of layer 2
    {
        const uint32_t n = nb < a.nb2 ? a.ks2 : 0u, f = h * NB1;
        return {w2s() + ((size_t)nb * (EXACT ? (uint32_t)KS2 : a.ks2) + f) * 64u, n > f ? n - f : 0u};
    }
    __device__ __forceinline__ Src pick(bool first, const Src& x, const Src& y) const { return {first ? x.p : y.p, first ? x.limit : y.limit}; }
    __device__ __forceinline__ void request(const Src& src, v4u (&s)[STAGE], int u)
    {
        const uint32_t j = wave * STAGE + u;
        const v4u* p = EXACT || j < src.limit ? src.p + wave * STAGE * 64u : zeros() - u * 64;
        s[u] = p[lane + u * 64u];
    }
    __device__ __forceinline__ void put(const v4u (&s)[STAGE], int u, int b) { ring[(b * NB1 + wave * STAGE + u) * 64u + lane] = s[u]; }

    // what a step does for the weights beside its MFMAs: pos: the fragment's place in its piece, c: the piece's number (mod 4)
    __device__ __forceinline__ void feed(const Src& src, int pos, int c)
    {
        if (pos < STAGE) {
            put(st[c & 1], pos, (c + 2) & 3);
            request(src, st[c & 1], pos);
        }
    }
    // fragment of three steps on, into the place of the one before
    __device__ __forceinline__ void read_ahead(int pos, int c)
    {
        const int p = pos + kFrag - 1, b = p < NB1 ? c : c + 1;
        fb[p % kFrag] = ring[((b & 3) * NB1 + p % NB1) * 64u + swz];
    }
    // every wave's share of the piece after the next is in shared memory, nobody reads the one before this one
    static __device__ __forceinline__ void sync()
    {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC37F); // at most the last three reads outstanding
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    // input element of request p for the rows whose flows lane r holds in flow
    __device__ __forceinline__ uint32_t flow_of(int p, uint32_t flow) const { return (uint32_t)__shfl((int)flow, (int)(p * RPP + lane / LPR), 64); }
    __device__ __forceinline__ float4 load_piece(uint32_t f)
    {
        const uint32_t k = 4u * (lane % LPR);
        return *reinterpret_cast<const float4*>(a.feat + (size_t)f * a.feat_ld + (k < a.n_in ? k : 0u));
    }
    // one element of a request through the input map
    __device__ __forceinline__ float map_one(float z, float m, float s) const
    {
        const float d = (4u * (lane % LPR) < a.n_in ? z : 0.f) - m;
        float t = d * s;
        t = t < -a.clamp_z ? -a.clamp_z : t;
        return t > a.clamp_z ? a.clamp_z : t;
    }
    __device__ __forceinline__ void put_piece(int p, const float4& v)
    {
        const uint32_t r = p * RPP + lane / LPR, k = 4u * (lane % LPR);
        // fragment (r / 32, k / 16), lane r % 32 + 32 * (k / 8 % 2)
        uint32_t* dst = reinterpret_cast<uint32_t*>(xin + ((r >> 5) * KS1 + (k >> 4)) * 64u + (r & 31u) + 32u * ((k >> 3) & 1u)) + ((k & 4u) >> 1);
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
    }
    __device__ __forceinline__ void store_piece(int p, float4 v)
    {
        put_piece(p, make_float4(map_one(v.x, mu.x, is.x), map_one(v.y, mu.y, is.y), map_one(v.z, mu.z, is.z), map_one(v.w, mu.w, is.w)));
    }

    // requests p to n - 1, several at a time
    __device__ __forceinline__ void input_pieces(uint32_t p, uint32_t n, uint32_t flow)
    {
        for (; p < n; p += 4u) {
            float4 v[4];
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u) v[u] = load_piece(flow_of(p + u < n ? p + u : n - 1u, flow));
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u) store_piece(p + u < n ? p + u : n - 1u, v[u]);
        }
    }

    // element v of a lane is column 16 (v / 8) + 8 (lane / 32) + v % 8 of its 32
    __device__ __forceinline__ void read_bias(const float* b, int g) { bias[g] = *reinterpret_cast<const float4*>(b + 16 * (g >> 1) + 4 * (g & 1) + 8u * half); }
    __device__ __forceinline__ f32x16 start() const
    {
        f32x16 c;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            c[4 * g + 0] = bias[g].x;
            c[4 * g + 1] = bias[g].y;
            c[4 * g + 2] = bias[g].z;
            c[4 * g + 3] = bias[g].w;
        }
        return c;
    }
    // elements 2 t and 2 t + 1 of a block's results, as bfloat16
    static __device__ __forceinline__ uint32_t relu_pair(const f32x16& c, int t)
    {
        uint32_t y = sftiles::relu_pair(c[2 * t], c[2 * t + 1]);
        asm volatile("" : "+v"(y)); // made here, in the shadow of this step's MFMA, and not where it is used
        return y;
    }
    static __device__ __forceinline__ v4u relu_frag(const f32x16& c, int e)
    {
        return frag4(relu_pair(c, 4 * e), relu_pair(c, 4 * e + 1), relu_pair(c, 4 * e + 2), relu_pair(c, 4 * e + 3));
    }
    static __device__ __forceinline__ void keep(bf16x8& dst, const v4u& v, int at)
    {
        // (the compiler's own choice moves operands between the two kinds of registers)
        dst = operand(v);
        if (at < AREGS) asm volatile("" : "+a"(dst));
        else asm volatile("" : "+v"(dst));
    }

    // 32 * MI rows from row0 on through the model; flow: lane r's input row; next_row0: the wave's first row in the next pass, whose
    // input is in shared memory when this one ends.  Rows from row_end on repeat the last one and store nothing.
    template <int MI>
    __device__ __forceinline__ void pass(uint32_t row0, uint32_t row_end, uint32_t& flow, uint32_t next_row0)
    {
        asm volatile("" : "+v"(lane)); // nothing made from it is kept from pass to pass
        half = lane >> 5;
        swz = sftiles::weight_lane(lane);
        const uint32_t own = row0 + lane; // this lane's row (MI = 1: of the first 32 lanes)
        const bool own_ok = own < row_end && (MI == 2 || lane < 32u);
        uint32_t dst = flow;
        if (a.scatter) dst = a.scatter[own < row_end ? own : row_end - 1u];
        // the next pass's flows
        const uint32_t nr = next_row0 + lane;
        uint32_t nf = a.esc_idx[nr < row_end ? nr : row_end - 1u];
        nf = nf < a.n_rows ? nf : a.n_rows - 1u;

        bf16x8 act[MI][KS2];
        f32x16 acc[2][MI];
        {
            v4u x[MI][KS1];
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int s = 0; s < KS1; ++s) x[i][s] = xin[(i * KS1 + s) * 64u + lane];
#pragma unroll
            for (int cb = 0; cb < NB1; ++cb) {
                uint32_t h[4];
#pragma unroll
                for (int s = 0; s < KS1; ++s) {
                    const int f = cb * KS1 + s, pos = f % NB1, c = f / NB1;
                    const bf16x8 w = operand(fb[pos % kFrag]);
                    const int T = 8 / KS1; // pairs of the columns before per MFMA
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        acc[cb & 1][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, operand(x[i][s]), s ? acc[cb & 1][i] : start(), 0, 0, 0);
                        if (i == 0) read_ahead(pos, c);
                        if (i == MI - 1) {
                            if (pos < STAGE) feed(c + 4 < KS1 ? piece1(c + 4) : piece2((c + 4 - KS1) >> 1, c & 1), pos, c);
#pragma unroll
                            for (int g = 0; g < 4; ++g)
                                if (s == g / 2) read_bias(cb + 1 < NB1 ? b1 + (cb + 1) * 32 : b2, g); // (after its last use)
                        }
                        if (cb > 0) {
#pragma unroll
                            for (int t = (s * MI + i) * T; t < (s * MI + i + 1) * T; ++t) {
                                h[t & 3] = relu_pair(acc[(cb & 1) ^ 1][t >> 3], t & 7);
                                if ((t & 3) == 3)
                                    keep(act[t >> 3][2 * (cb - 1) + ((t >> 2) & 1)], frag4(h[0], h[1], h[2], h[3]), (t >> 3) * KS2 + 2 * (cb - 1) + ((t >> 2) & 1));
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (pos == SYNC) sync();
                }
            }
#pragma unroll
            for (int t = 0; t < 2 * MI; ++t) keep(act[t >> 1][2 * (NB1 - 1) + (t & 1)], relu_frag(acc[(NB1 - 1) & 1][t >> 1], t & 1), (t >> 1) * KS2 + 2 * (NB1 - 1) + (t & 1));
        }
        f32x16 out[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                out[i][v] = b3[16 * (v >> 3) + 8u * half + (v & 7)];
                acc[1][i][v] = 0.f;
            }
        v4u v3a = v4u{0, 0, 0, 0}, v3b = v3a; // operands of the last layer for the columns before: zeros at first
        float4 in[AT_ONCE]; // the next pass's input on its way from memory: requests piece, piece + 1, ...
        uint32_t in_flow[AT_ONCE], piece = 0, nb = 0;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) in[u] = load_piece(flow_of(u, nf));
        do {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const bool more = nb + 2u < nb2p;
                Src src[2];
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2)
                    src[h2] = pick(more, piece2(nb + q + 2u, h2), piece1(2 * q + h2));
                uint32_t h[4];
#pragma unroll
                for (int s = 0; s < KS2; ++s) {
                    const int pos = s % NB1, c = 2 * q + s / NB1;
                    const bf16x8 w = operand(fb[pos % kFrag]);
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        acc[q][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, act[i][s], s ? acc[q][i] : start(), 0, 0, 0);
                        if (i == 0) {
                            read_ahead(pos, c);
                            // the columns before: relu, and on into the last layer
#pragma unroll
                            for (int t = (s - 2) * RELU; t < (s - 1) * RELU; ++t) {
                                if (t < 0 || t > 8 * MI) continue;
                                if (t > 0 && (t & 3) == 0) {
                                    const int z = t - 1;
                                    out[z >> 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand((z >> 2) & 1 ? v3b : v3a), operand(frag4(h[0], h[1], h[2], h[3])), out[z >> 3], 0, 0, 0);
                                }
                                if (t < 8 * MI) h[t & 3] = relu_pair(acc[q ^ 1][t >> 3], t & 7);
                            }
                        }
                        if (i == MI - 1) {
                            feed(src[s / NB1], pos, c);
                            // the next columns' bias (after the last pair: the next pass's first), this block's operands of the last layer
#pragma unroll
                            for (int g = 0; g < 4; ++g)
                                if (s == KS2 - 4 + g) read_bias(q == 0 || more ? b2 + (nb + q + 1u) * 32u : b1, g);
                            if (s == KS2 - 3) v3a = w3s()[2u * (nb + q) * 64u + swz];
                            if (s == KS2 - 2) v3b = w3s()[(2u * (nb + q) + 1u) * 64u + swz];
                            // the next pass's input
#pragma unroll
                            for (int u = 0; u < AT_ONCE; ++u) {
                                if (s == KS2 - 8) in[u].x = map_one(in[u].x, mu.x, is.x);
                                if (s == KS2 - 7) in[u].y = map_one(in[u].y, mu.y, is.y);
                                if (s == KS2 - 6) in[u].z = map_one(in[u].z, mu.z, is.z);
                                if (s == KS2 - 5) in[u].w = map_one(in[u].w, mu.w, is.w);
                                if (s == KS2 - 4) put_piece(piece + u, in[u]);
                                if (s == KS2 - 3 && u == 0) piece = piece + AT_ONCE < (uint32_t)(PIECES * MI) ? piece + AT_ONCE : (uint32_t)(PIECES * MI - AT_ONCE); // (the last ones again)
                                if (s == KS2 - 3) in_flow[u] = flow_of(piece + u, nf);
                                if (s == KS2 - 1) in[u] = load_piece(in_flow[u]);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (pos == SYNC) sync();
                }
            }
            nb += 2u;
        } while (nb < nb2p); // (at least one pair)
#pragma unroll
        for (int t = 0; t < 2 * MI; ++t)
            out[t >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(t & 1 ? v3b : v3a), operand(relu_frag(acc[1][t >> 1], t & 1)), out[t >> 1], 0, 0, 0);
        // what is left of the next pass's input
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) store_piece(piece + u, in[u]);
        input_pieces(piece + AT_ONCE, PIECES * MI, nf);
        uint32_t label = 0;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const uint32_t row = row0 + i * 32u + (lane & 31u);
            float* lg = a.logits + (size_t)row * a.c;
            const bool write = a.logits && row < row_end;
            uint32_t best = 8u * half;
            float bv = label_start(half, out[i][0]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (16u * e >= a.c) break;
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const uint32_t c = 16u * e + 8u * half + v;
                    const float y = out[i][8 * e + v];
                    const bool there = c < a.c;
                    if (write && there) lg[c] = y;
                    const bool take = there && y > bv;
                    bv = take ? y : bv;
                    best = take ? c : best;
                }
            }
            best = label_of(best, bv);
            if (i == 0 || half) label = best;
        }
        if (own_ok && dst < a.n_labels) a.labels[dst] = (uint16_t)label;
        flow = nf;
    }
};

template <int NB1, int KS1, bool EXACT>
__global__ __launch_bounds__(kWaves * 64, 1) void mlp_rows(RowsArgs a)
{
    using R = Rows<NB1, KS1, EXACT>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint32_t total = *a.esc_count;
    total = total < a.esc_cap ? total : a.esc_cap;
    const uint32_t rb_total = (total + 31u) / 32u;
    const uint32_t rb_lo = rb_total / gridDim.x, rb_rem = rb_total % gridDim.x;
    const uint32_t rb_first = blockIdx.x * rb_lo + (blockIdx.x < rb_rem ? blockIdx.x : rb_rem);
    const uint32_t rb_count = rb_lo + (blockIdx.x < rb_rem ? 1u : 0u);
    if (rb_count == 0) return;
    const uint32_t row_begin = rb_first * 32u;
    uint32_t row_end = (rb_first + rb_count) * 32u;
    row_end = row_end < total ? row_end : total;

    const uint32_t tid = threadIdx.x;
    // shared memory: biases, input fragments, weight pieces; in place of the last two a tile
    float *const b1 = reinterpret_cast<float*>(smem), *const b2 = b1 + 512, *const b3 = b2 + 512;
    v4u* const xall = reinterpret_cast<v4u*>(b3 + 32);
    for (uint32_t q = tid; q < 512u; q += kWaves * 64u) {
        b1[q] = q < a.h1 ? a.b1[q] : 0.f;
        b2[q] = q < a.h2 ? a.b2[q] : 0.f;
        if (q < 32u) b3[q] = q < a.c ? a.b3[q] : 0.f;
    }
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // passes of 256 rows (64 a wave), then one of 256 or 128 for three and more row blocks, or a tile for one or two
    const uint32_t rest = rb_count % 8u;
    const uint32_t n_full = rb_count / 8u + (rest > 4u ? 1u : 0u);
    const bool low = rest == 3u || rest == 4u, tile = rest == 1u || rest == 2u;
    if (n_full || low) {
        R r = {a};
        r.ring = xall + kWaves * 2 * KS1 * 64;
        r.xin = xall + wave * 2 * KS1 * 64;
        r.b1 = b1;
        r.b2 = b2;
        r.b3 = b3;
        r.lane = tid & 63u;
        r.wave = wave;
        r.half = r.lane >> 5;
        r.swz = sftiles::weight_lane(r.lane);
        r.nb2p = (a.nb2 + 1u) & ~1u;
        // first pieces of the weights
        v4u first[2][R::STAGE];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int u = 0; u < R::STAGE; ++u) r.request(r.piece1(c), c < 2 ? first[c] : r.st[c - 2], u);
        const bool low_first = rb_count <= 4u; // the height of the first pass decides the wave's rows
        uint32_t flow;
        {
            const uint32_t row = row_begin + wave * (low_first ? 32u : 64u) + r.lane;
            flow = a.esc_idx[row < row_end ? row : row_end - 1u];
            flow = flow < a.n_rows ? flow : a.n_rows - 1u;
        }
        {
            const uint32_t k = 4u * (r.lane % R::LPR);
            const bool map = a.mu && k < a.n_in; // (n_in is a multiple of 4)
            r.mu = map ? make_float4(a.mu[k], a.mu[k + 1u], a.mu[k + 2u], a.mu[k + 3u]) : make_float4(0.f, 0.f, 0.f, 0.f);
            r.is = map ? make_float4(a.inv_sigma[k], a.inv_sigma[k + 1u], a.inv_sigma[k + 2u], a.inv_sigma[k + 3u]) : make_float4(1.f, 1.f, 1.f, 1.f);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int u = 0; u < R::STAGE; ++u) r.put(first[c], u, c);
        __syncthreads();
#pragma unroll
        for (int f = 0; f < kFrag - 1; ++f) r.fb[f] = r.ring[f * 64u + r.swz];
#pragma unroll
        for (int g = 0; g < 4; ++g) r.read_bias(b1, g);
        r.input_pieces(0u, low_first ? R::PIECES : 2 * R::PIECES, flow);
        uint32_t base = row_begin;
        for (uint32_t p = 0; p < n_full; ++p, base += 256u) {
            const bool low_next = p + 1u == n_full && low;
            r.template pass<2>(base + wave * 64u, row_end, flow, base + 256u + wave * (low_next ? 32u : 64u));
        }
        if (low) r.template pass<1>(base + wave * 32u, row_end, flow, base + wave * 32u);
    }
    if (tile) {
        sftiles::FusedSmem m;
        m.s_b1 = b1;
        m.s_b2 = b2;
        m.s_b3 = b3;
        m.H = reinterpret_cast<uint16_t*>(xall);
        m.s_flow = reinterpret_cast<uint32_t*>(m.H + 64 * sftiles::LDH);
        m.s_mu = reinterpret_cast<float*>(m.s_flow + 2 * sftiles::FBM);
        m.s_is = m.s_mu + sftiles::HMAX;
        __syncthreads(); // the passes are done with the shared memory
        for (uint32_t q = tid; q < 128u; q += kWaves * 64u) { // (n_in is at most 128)
            m.s_mu[q] = (a.mu && q < a.n_in) ? a.mu[q] : 0.f;
            m.s_is[q] = (a.mu && q < a.n_in) ? a.inv_sigma[q] : 1.f;
        }
        const uint32_t first = row_begin + n_full * 256u;
        // (columns split over the waves as evenly as whole column blocks allow)
        if (NB1 < 16 && a.nb2 <= (uint32_t)NB1) {
            if (rest == 1u)
                sftiles::run_tiles<kWaves, NB1 / kWaves, 1>(a, m, wave, first, 1u, row_end);
            else
                sftiles::run_tiles<kWaves, NB1 / kWaves, 2>(a, m, wave, first, 1u, row_end);
        } else {
            if (rest == 1u)
                sftiles::run_tiles<kWaves, 16 / kWaves, 1>(a, m, wave, first, 1u, row_end);
            else
                sftiles::run_tiles<kWaves, 16 / kWaves, 2>(a, m, wave, first, 1u, row_end);
        }
    }
}

constexpr size_t kTileLds = (size_t)64 * sftiles::LDH * 2 + 2 * sftiles::FBM * 4 + 2 * sftiles::HMAX * 4;

} // namespace

namespace sfrows {

template <int NB1, int KS1, bool EXACT>
static int launch(sf_ctx* ctx, int slot, const RowsArgs& a)
{
    size_t lds = ((size_t)kBufs * NB1 * 64 + kWaves * 2 * KS1 * 64) * 16;
    lds = (lds > kTileLds ? lds : kTileLds) + (512 + 512 + 32) * 4;
    auto* kernel = mlp_rows<NB1, KS1, EXACT>;
    SF_ALLOW_LDS(ctx, slot, kernel);
    const uint32_t rb_cap = (a.esc_cap + 31u) / 32u;
    uint32_t grid = (uint32_t)ctx->n_cu;
    if (grid > rb_cap) grid = rb_cap;
    kernel<<<grid, kWaves * 64, lds, ctx->stream>>>(a);
    SF_LAUNCH_CHECK(ctx, "mlp_rows");
    return SF_OK;
}

int run(sf_ctx* ctx, const RowsArgs& a)
{
    const int slot = sf::kLdsRows + (a.n_in > 64u ? 5 : 0);
    const bool exact = a.nb1 == 16u && a.nb2 % 2u == 0; // (every piece is whole)
    if (a.n_in <= 64u) {
        if (a.nb1 <= 4u) return launch<4, 4, false>(ctx, slot, a);
        if (a.nb1 <= 8u) return launch<8, 4, false>(ctx, slot + 1, a);
        if (a.nb1 <= 12u) return launch<12, 4, false>(ctx, slot + 2, a);
        return exact ? launch<16, 4, true>(ctx, slot + 3, a) : launch<16, 4, false>(ctx, slot + 4, a);
    }
    if (a.nb1 <= 4u) return launch<4, 8, false>(ctx, slot, a);
    if (a.nb1 <= 8u) return launch<8, 8, false>(ctx, slot + 1, a);
    if (a.nb1 <= 12u) return launch<12, 8, false>(ctx, slot + 2, a);
    return exact ? launch<16, 8, true>(ctx, slot + 3, a) : launch<16, 8, false>(ctx, slot + 4, a);
}

} // namespace sfrows
