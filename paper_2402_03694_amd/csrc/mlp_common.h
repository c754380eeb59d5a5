// Pieces shared by the layer-by-layer MLP kernels: the argument block of one layer and the
// builder of the A operand (8 consecutive K values of one escalated row as bfloat16), which reads
// a bfloat16 activation matrix, or gathers and standardises a feature row, or unpacks header bits.
#pragma once

#include "common.h"
#include "slow_label.h"

namespace sfmlp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4; // (an array of uint4 the compiler may keep in memory)

constexpr int BM = 128; // rows per block

enum { A_BF16 = 0, A_FEAT = 1, A_RAW = 2 };

struct LayerArgs {
    // rows
    const uint32_t* esc_idx;  // row e reads the input row esc_idx[e] (clamped below n_rows) ...
    const uint32_t* scatter;  // ... and its label goes to labels[scatter[e]]; NULL = the same index
    const uint32_t* esc_count;
    uint32_t esc_cap;
    uint32_t row_begin; // first escalated row of this chunk
    uint32_t rows_cap;  // rows the chunk's activations hold (a multiple of BM)
    uint32_t n_rows;    // rows of the input (feature matrix or flows of the packet arrays)
    uint32_t n_labels;  // entries of labels; a label index outside is not written
    // A operand
    const uint16_t* a_bf16; // [rows_in_chunk][lda]
    uint32_t lda;
    const float* feat;
    uint32_t feat_ld;
    const float* mu;
    const float* inv_sigma;
    float clamp;
    const uint32_t* off;
    const uint32_t* hdr;
    uint32_t hdr_words, raw_bits, raw_pkts, n_pkts;
    // weights
    const uint16_t* w; // [N][K] bfloat16 bit patterns
    const float* bias;
    uint32_t N, K;
    // output
    uint16_t* h_out; // [rows_in_chunk][ldh] bfloat16
    uint32_t ldh;
    float* logits;   // [esc_cap][classes] or NULL
    uint16_t* labels;
    const uint16_t* pred; // labels = pred for all n_labels flows first, by the first hidden layer's launch; NULL = they stay
    // The second hidden layer may take the last one along (wide_takes_last): its operand-ordered weights (or NULL), biases and classes (0: it may not)
    const uint4* wo_last;
    const float* b_last;
    uint32_t n_last;
    // ... and for the last layer's own launch: blocks of the second hidden layer's (0: that one took nothing along) and its K
    uint32_t units_before, k_before;
};

static __device__ __forceinline__ uint16_t f32_to_bf16_bits(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16); // inf / nan: truncate
    u += 0x7FFFu + ((u >> 16) & 1u);                                  // round to nearest even
    return (uint16_t)(u >> 16);
}

static __device__ __forceinline__ uint32_t pack2(uint16_t lo, uint16_t hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }

// 8 consecutive K values [k, k+8) of weight row n (row-major [N][K] bfloat16 bits), zero outside
static __device__ __forceinline__ uint4 weight_chunk(const uint16_t* w, uint32_t N, uint32_t K, uint32_t n, uint32_t k)
{
    if (n >= N || k >= K) return make_uint4(0, 0, 0, 0);
    const uint16_t* p = w + (size_t)n * K + k;
    if (k + 8 <= K && (K & 7u) == 0 && (reinterpret_cast<uintptr_t>(w) & 15u) == 0) return *reinterpret_cast<const uint4*>(p);
    uint16_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = k + q < K ? p[q] : (uint16_t)0;
    return make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
}

// The end of the last layer for 32 rows, a row's classes in lanes l and l ^ 32: sum[j][v] of class 32 j + 8 * (v / 4) + 4 * half + v % 4,
// weights first in the multiplication.  s_bias: shared memory, zeros behind the last class; row: among the logits.
template <int NI>
static __device__ __forceinline__ void last_rows(const LayerArgs& a, const f32x16 (&sum)[NI], const float* s_bias, uint32_t classes, uint32_t half, bool there,
                                                 uint32_t row, uint32_t dst)
{
    // class 0 first, then every class that is strictly larger than all before it (label_start, label_of)
    uint32_t best = 4u * half;
    float bv = 0.f;
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t c0 = j * 32u + 8u * g + 4u * half; // ascending in j and g
            const float4 b = *reinterpret_cast<const float4*>(s_bias + c0);
            const float y[4] = {sum[j][4 * g] + b.x, sum[j][4 * g + 1] + b.y, sum[j][4 * g + 2] + b.z, sum[j][4 * g + 3] + b.w};
            if (j == 0 && g == 0) bv = label_start(half, y[0]);
#pragma unroll
            for (uint32_t e = 0; e < 4u; ++e) {
                const uint32_t c = c0 + e;
                if (c < classes) {
                    if (a.logits && there) a.logits[(size_t)row * classes + c] = y[e];
                    if (y[e] > bv) {
                        bv = y[e];
                        best = c;
                    }
                }
            }
        }
    best = label_of(best, bv);
    if (half == 0 && there && dst < a.n_labels) a.labels[dst] = (uint16_t)best;
}

// How a hidden layer's tiles of 128 rows x 512 columns are dealt out to `units` blocks: a row block with all its n_cb column blocks
// (walk), where that costs no block a tile more than 1 in 16 or the input stays (resident), else tile by tile.
static __device__ __forceinline__ bool wide_walks(uint32_t row_blocks, uint32_t n_cb, uint32_t units, bool resident)
{
    const uint32_t t_walk = (row_blocks + units - 1u) / units * n_cb, t_split = (row_blocks * n_cb + units - 1u) / units; // tiles, longest block
    return n_cb > 1u && row_blocks >= units && (resident || t_walk - t_split <= t_split / 16u);
}
constexpr uint32_t kFewTileRows = 32, kFewTileCols = 256;
// So few rows that tiles of 32 rows x 256 columns (ldh columns in all) give a block at most one: they go that way (wide_few).
static __host__ __device__ __forceinline__ uint64_t wide_few_tiles(uint32_t rows, uint32_t ldh)
{
    return (uint64_t)((rows + kFewTileRows - 1u) / kFewTileRows) * ((ldh + kFewTileCols - 1u) / kFewTileCols);
}
// A block that holds all columns of a row takes the last layer along: two of its eight waves multiply, so it pays where the activations it
// keeps from memory are many (more than one column block, 5 to 15 % of a whole call; more than 256 columns and more than a tile a block, 1 to 3),
// or where its own launch would be one block's latency (up to a tile a block, up to 256 columns, 2 to 4; with more columns 2 % the other way,
// as with fewer columns and more tiles: 41,385 rows through 6-640-192-25 71.2 us along, 67.1 in its own launch).
static __device__ __forceinline__ bool wide_takes_last(uint32_t rows, uint32_t ldh, uint32_t units, bool resident)
{
    const uint32_t n_cb = (ldh + 511u) / 512u;
    const uint32_t row_blocks = (rows + BM - 1u) / BM;
    return wide_few_tiles(rows, ldh) > units && (n_cb == 1u ? (row_blocks <= units) == (ldh <= 256u) : wide_walks(row_blocks, n_cb, units, resident));
}
constexpr uint32_t kWideSlab = 64, kWideSlabs = 3; // K values of a slab, slabs that stay

// the packets of a flow for the raw-bit input: first packet and count, clamped into the packet arrays
static __device__ __forceinline__ void raw_flow_range(const LayerArgs& a, uint32_t flow, uint32_t& b0, uint32_t& n)
{
    uint32_t e0 = a.off[flow + 1];
    b0 = a.off[flow];
    b0 = b0 < a.n_pkts ? b0 : a.n_pkts;
    e0 = e0 < a.n_pkts ? e0 : a.n_pkts;
    n = e0 > b0 ? e0 - b0 : 0;
}

// Header bits as input: feature k = raw_bits * j + b is bit b of packet j, which is bit 7-(b%8) of header byte b/8; zero past
// K and past the flow.  The 8 features from (j, b) on are requested first, as the header words that hold them, and turned into
// bfloat16 0.0 / 1.0 later, when the words have arrived.  Which words these are depends on how the bits lie:
enum RawForm {
    RAW_BYTES, // raw_bits a multiple of 8: the features are the bits of one byte, in one word
    RAW_LONG,  // else from 8 bits a packet: the word with the first feature, the next one if a byte's worth of bits ends there,
               // and the first word of the next packet if this one ends before
    RAW_SHORT, // 3 to 7 bits: the only word of up to four packets (7 bits: two, 4 to 6: three); 1 or 2 bits: of up to eight, so
               // the features themselves as a byte (the one case that waits for its words)
};

// b < raw_bits + 256 bits from the start of packet j on -> the packet they lead to and the bit in it; per = 1 / raw_bits.
// (Exact: b + 0.5 is at least half a bit off a multiple of raw_bits, the product's error below 2^-13 for quotients up to 511.)
static __device__ __forceinline__ void raw_carry(const LayerArgs& a, float per, uint32_t& j, uint32_t& b)
{
    const uint32_t whole = a.raw_bits >= 256u ? (b >= a.raw_bits ? 1u : 0u) : (uint32_t)(((float)b + 0.5f) * per);
    j += whole;
    b -= whole * a.raw_bits;
}

// The words of the features from (j, b) on of a flow whose packets start at b0 (n of them)
template <int FORM>
static __device__ __forceinline__ uint4 raw_words_at(const LayerArgs& a, uint32_t b0, uint32_t n, uint32_t j, uint32_t b)
{
    uint4 r = make_uint4(0, 0, 0, 0);
    const uint32_t end = n < a.raw_pkts ? n : a.raw_pkts;
    if (j >= end) return r;
    const uint32_t* row = a.hdr + (size_t)(b0 + j) * a.hdr_words;
    if (FORM == RAW_BYTES) {
        r.x = row[b >> 5];
    } else if (FORM == RAW_LONG) {
        const uint32_t left = a.raw_bits - b, ahead = 32u - (b & 31u); // features of this packet, of this word
        r.x = row[b >> 5];
        if (ahead < 8u && left > ahead) r.y = row[(b >> 5) + 1u];
        if (left < 8u && j + 1u < end) r.z = row[a.hdr_words];
    } else if (a.raw_bits >= 3u) {
        r.x = row[0];
        if (j + 1u < end) r.y = row[a.hdr_words];
        if (a.raw_bits < 7u && j + 2u < end) r.z = row[2u * a.hdr_words];
        if (a.raw_bits < 4u && j + 3u < end) r.w = row[3u * a.hdr_words];
    } else {
#pragma unroll 4
        for (uint32_t q = 0; q < 8u; ++q) {
            const uint32_t d = (b + q) >> (a.raw_bits - 1u), bit = (b + q) & (a.raw_bits - 1u);
            if (j + d < end) r.x |= ((row[(size_t)d * a.hdr_words] >> (7u - bit)) & 1u) << (7u - q);
        }
    }
    return r;
}

// ... and the features in them
template <int FORM>
static __device__ __forceinline__ uint4 raw_bits_of(const LayerArgs& a, const uint4& r, uint32_t b)
{
    uint32_t byte = r.x; // the features as bits 7..0
    if (FORM == RAW_BYTES) {
        byte = r.x >> (b & 24u);
    } else if (FORM == RAW_LONG) {
        const uint64_t two = (uint64_t)__builtin_bswap32(r.x) << 32 | __builtin_bswap32(r.y); // first bit first
        const uint32_t left = a.raw_bits - b;
        byte = (uint32_t)(two << (b & 31u) >> 56);
        if (left < 8u) byte = (byte & (0xFF00u >> left)) | (r.z & 0xFFu) >> left;
    } else if (a.raw_bits >= 3u) {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
        byte = 0;
        uint32_t end = a.raw_bits - b; // features up to and with packet p
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (p == 2 && a.raw_bits == 7u) break;
            const uint32_t field = (w[p] & 0xFFu) >> (8u - a.raw_bits);
            byte |= end <= 8u ? field << (8u - end) : end < 8u + a.raw_bits ? field >> (end - 8u) : 0u;
            end += a.raw_bits;
        }
    }
    uint32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        v[q] = ((uint32_t)__builtin_amdgcn_sbfe((int)byte, 7 - 2 * q, 1) & 0x3F80u) |
               ((uint32_t)__builtin_amdgcn_sbfe((int)byte, 6 - 2 * q, 1) & 0x3F800000u);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// 8 consecutive K values [k, k+8) of escalated row e as bfloat16, zero past K (bfloat16 activations or feature rows).
template <int AMODE>
static __device__ __forceinline__ uint4 load_a_chunk(const LayerArgs& a, bool row_ok, uint32_t row_in_chunk,
                                              uint32_t flow, uint32_t k)
{
    uint4 out = make_uint4(0, 0, 0, 0);
    if (!row_ok || k >= a.K) return out;
    if (AMODE == A_BF16) {
        const uint16_t* p = a.a_bf16 + (size_t)row_in_chunk * a.lda + k;
        if (k + 8 <= a.K && (a.lda & 7u) == 0) return *reinterpret_cast<const uint4*>(p);
        uint16_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = k + q < a.K ? p[q] : (uint16_t)0;
        return make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
    }
    if (AMODE == A_FEAT) {
        const float* p = a.feat + (size_t)flow * a.feat_ld + k;
        float x[8];
        if (k + 8 <= a.K && (a.feat_ld & 3u) == 0 && (reinterpret_cast<uintptr_t>(a.feat) & 15u) == 0 && (k & 3u) == 0) {
            const float4 x0 = reinterpret_cast<const float4*>(p)[0], x1 = reinterpret_cast<const float4*>(p)[1];
            x[0] = x0.x; x[1] = x0.y; x[2] = x0.z; x[3] = x0.w;
            x[4] = x1.x; x[5] = x1.y; x[6] = x1.z; x[7] = x1.w;
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = k + q < a.K ? p[q] : 0.f;
        }
        uint16_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float z = x[q];
            if (a.mu && k + q < a.K) {
                const float d = z - a.mu[k + q];
                z = d * a.inv_sigma[k + q];
                z = z < -a.clamp ? -a.clamp : z;
                z = z > a.clamp ? a.clamp : z;
            }
            v[q] = k + q < a.K ? f32_to_bf16_bits(z) : (uint16_t)0;
        }
        return make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
    }
}

static __device__ __forceinline__ bf16x8 as_bf16x8(uint4 u)
{
    union {
        uint4 u;
        bf16x8 b;
    } c;
    c.u = u;
    return c.b;
}


} // namespace sfmlp

namespace sf {
// operand-ordered copies of weight matrices (slow_fused.hip): out[(nb*KS + ks)*64 + lane] holds the 8
// values W[nb*32 + lane%32][ks*16 + 8*(lane/32) ..+8), K padded to a multiple of 64, zero outside
struct ReorderSpec {
    const void* w; // [N][K] bfloat16 bits, row-major
    uint32_t N, K;
    void* out;
};
size_t reordered_bytes(uint32_t N, uint32_t K);
int reorder_weights_async(sf_ctx* ctx, const ReorderSpec* specs, int n_specs); // at most 3 per launch
} // namespace sf
