// Step 5, fused form for hidden widths up to 512: the whole 3-layer MLP of a tile of 128
// escalated flows runs in one block without touching HBM between layers (Sections 3.1 and 4.4
// of the paper: only the uncertain flows reach the slow model, and its label replaces the fast
// one).
//
// A block is eight waves; wave w owns output columns [64w, 64w+64) of each hidden layer for
// all 128 rows, i.e. a 4x2 grid of 32x32 MFMA accumulators (128 accumulator registers).  The
// activations of the tile stay in shared memory ([128][520] bfloat16, 16-byte reads of 8
// consecutive rows fall on distinct banks); the weights are re-ordered once per call so that
// the 8 K-values a lane needs for an MFMA B operand are contiguous and a wave's operand is one
// contiguous kilobyte, and are then read straight from the cache into registers.  There is no
// barrier inside a layer's K loop.  The last layer (at most 32 classes) takes a wave per row block, so that a
// logit is one sum in order of K as in the register form, followed by a per-row arg-max in registers and the scatter of the
// label.  (Two waves per row block, halves of K added at the end, were no faster, 64-512-512-10 8,000 rows 15.6 against 15.1 us, 32,768
// rows 23.8 against 23.1, and a row's logits then followed the list's capacity.)
// Long lists of rows with up to 128 values go through the register form instead (slow_rows.hip); the rule is at slow_fused().
// Blocks are persistent.  The rows that exist (the device-side escalation count) are cut into
// row blocks of 32 and dealt out evenly: every block gets a run of consecutive row blocks, the runs
// differ by at most one, and a block walks its run in tiles of four row blocks; what is left at
// the end of a run (one to three row blocks) is a last, lower tile (two row blocks high when that
// is enough), so the blocks finish together and few rows fill the whole device.
#include "slow_few.h"
#include "slow_rows.h"
#include "slow_tiles.h"
#include "small_batch.h"

namespace sf {
bool slow_fused_ok(const sf_mlp* mlp, bool raw_input);
size_t slow_fused_ws_bytes(const sf_mlp* mlp);
int slow_fused(sf_ctx* ctx, void* ws, bool ws_is_ordered, const float* feat, uint32_t feat_ld, uint32_t n_rows,
               const uint32_t* esc_idx, const uint32_t* scatter, const uint32_t* esc_count, uint32_t esc_cap,
               uint32_t n_labels, const sf_mlp* mlp, const uint16_t* pred, const sfsmall::GateRows* gate, float* logits, uint16_t* labels);
bool slow_fused_gates(sf_ctx* ctx, const sf_mlp* mlp, uint32_t n);
int copy_labels_async(sf_ctx* ctx, const uint16_t* pred, uint16_t* labels, uint32_t n); // slow_infer.hip
int order_all(sf_ctx* ctx, const sf_mlp* mlp, void* out);
} // namespace sf

namespace {

using namespace sftiles;

constexpr int kWaves = 8; // waves per block
constexpr uint32_t kRowsLine = 128; // rows a compute unit from which the register form may take a list
// Flows a compute unit whose labels the launch copies.  The blocks that copy read the whole list and, where it fills the units, the last
// tiles wait for them.  Copy in a launch of its own : in this one, us: 5,076 rows of 20,305 flows 11.0 : 8.1, 24,211 of 24,211 16.4 : 16.7,
// 14,317 of 20,454 15.8 : 16.1, the longest loss up to the line 16,045 of 22,922 11.5 : 11.9; past it 28,466 of 31,629 14.7 : 16.6, 45,116 of
// 45,116 22.4 : 24.7 (and short lists would gain, 7,640 of 30,560 13.6 : 9.4; how long a list is only the device knows).
constexpr uint32_t kCopyUnit = 96;
constexpr int kNI = 2;    // 32-column blocks per wave

// W[N][K] (row-major, bfloat16 bits) -> out[(nb * KS + ks) * 64 + lane] = the 8 values
// W[nb*32 + lane%32][ks*16 + 8*(lane/32) .. +8), zero outside; nb < NB, ks < KS.
// One launch re-orders all three layers.
struct ReorderJob {
    const uint16_t* w;
    uint32_t N, K, NB, KS;
    uint32_t first; // index of the job's first 16-byte element in the launch-wide numbering
    uint4* out;
};
struct ReorderArgs {
    ReorderJob job[3];
    uint32_t total;
};

__global__ __launch_bounds__(256) void reorder_weights(ReorderArgs r)
{
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < r.total; e += gridDim.x * blockDim.x) {
        const int ji = e >= r.job[2].first ? 2 : (e >= r.job[1].first ? 1 : 0);
        const ReorderJob& jb = r.job[ji];
        const uint32_t g = e - jb.first;
        const uint32_t lane = g & 63u, t = g >> 6, ks = t % jb.KS, nb = t / jb.KS;
        const uint32_t n = nb * 32u + (lane & 31u), k0 = ks * 16u + 8u * (lane >> 5);
        uint16_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = (n < jb.N && k0 + q < jb.K) ? jb.w[(size_t)n * jb.K + k0 + q] : (uint16_t)0;
        jb.out[g] = make_uint4(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16), v[4] | ((uint32_t)v[5] << 16),
                               v[6] | ((uint32_t)v[7] << 16));
    }
}

__device__ __forceinline__ FusedSmem fused_smem(unsigned char* smem)
{
    FusedSmem m;
    m.H = reinterpret_cast<uint16_t*>(smem);                                    // [128][LDH]; also the input tile
    m.s_flow = reinterpret_cast<uint32_t*>(smem + (size_t)FBM * LDH * 2);       // [2][128]: this tile, next tile
    m.s_b1 = reinterpret_cast<float*>(m.s_flow + 2 * FBM);                      // [HMAX], zero past h1
    m.s_b2 = m.s_b1 + HMAX;                                                     // [HMAX], zero past h2
    m.s_b3 = m.s_b2 + HMAX;                                                     // [32], zero past c
    m.s_mu = m.s_b3 + 32;                                                       // [HMAX] input map (0 / 1 if none)
    m.s_is = m.s_mu + HMAX;                                                     // [HMAX]
    return m;
}

// One row block a block goes through few(row, end of the rows), more through the tiles.  The gate, if there is one, makes the list.
template <class Gate, class Few>
__device__ __forceinline__ void fused_rows(const FusedArgs& a, const FusedSmem& m, uint32_t wave, const Gate& gate, Few few)
{
    // this block's run of row blocks: the runs of the grid differ by at most one row block
    const uint32_t block = blockIdx.x - a.n_copy, blocks = gridDim.x - a.n_copy;
    struct Run {
        uint32_t first, count;
    };
    auto run_of = [&](uint32_t total) {
        const uint32_t all = (total + 31u) / 32u, lo = all / blocks, rem = all % blocks;
        return Run{block * lo + (block < rem ? block : rem), lo + (block < rem ? 1u : 0u)};
    };
    uint32_t total;
    if constexpr (std::is_same<Gate, sfsmall::GateRows>::value) {
        total = sfsmall::gate_rows<kWaves * 64>(gate, m.H, [&](uint32_t n) {
            const Run r = run_of(n);
            return [=](uint32_t p) { return p / 32u - r.first < r.count; };
        });
        if (block == 0 && threadIdx.x == 0) *gate.esc_count = total;
        __syncthreads();
    } else {
        total = *a.esc_count;
        total = total < a.esc_cap ? total : a.esc_cap;
        if (blockIdx.x < a.n_copy) {
            sfsmall::copy_unlisted<kWaves * 64, true>(a.pred, a.labels, a.n_labels, a.esc_idx, total, blockIdx.x * sfsmall::kCopySlice, m.s_flow);
            return;
        }
    }
    const Run run = run_of(total);
    const uint32_t rb_first = run.first, rb_count = run.count;
    if (rb_count == 0) return;
    const uint32_t row_begin = rb_first * 32u;
    uint32_t row_end = (rb_first + rb_count) * 32u;
    row_end = row_end < total ? row_end : total;

    if (rb_count == 1u && few(row_begin, row_end)) return;
    for (uint32_t q = threadIdx.x; q < (uint32_t)HMAX; q += kWaves * 64u) {
        m.s_b1[q] = q < a.h1 ? a.b1[q] : 0.f;
        m.s_b2[q] = q < a.h2 ? a.b2[q] : 0.f;
        if (q < 32u) m.s_b3[q] = q < a.c ? a.b3[q] : 0.f;
        m.s_mu[q] = (a.mu && q < a.n_in) ? a.mu[q] : 0.f;
        m.s_is[q] = (a.mu && q < a.n_in) ? a.inv_sigma[q] : 1.f;
    }
    // full tiles of four row blocks, then what is left: three row blocks run as a (masked) full tile, one or
    // two as a tile of half the height
    const uint32_t rest = rb_count % (uint32_t)kMI;
    const uint32_t n_full = rb_count / (uint32_t)kMI + (rest == 3u ? 1u : 0u);
    if (n_full) run_tiles<kWaves, kNI, kMI>(a, m, wave, row_begin, n_full, row_end);
    if (rest == 1u || rest == 2u) run_tiles<kWaves, kNI, 2>(a, m, wave, row_begin + n_full * FBM, 1u, row_end);
}

__global__ __launch_bounds__(kWaves * 64) void mlp_fused(FusedArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // the wave index is the same in every lane: say so, and everything derived from it (column
    // block, weight pointers) lives in scalar registers
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    fused_rows(a, fused_smem(smem), wave, sfsmall::NoGate{}, [](uint32_t, uint32_t) { return false; });
}

// ... with few rows a block in the form of slow_few.h (a kernel for each of its shapes: code that a short list never runs costs it
// time all the same, 0.7 us with all eight in one kernel)
template <int KS1, int N1, int N2, class Gate>
__global__ __launch_bounds__(kWaves * 64) void mlp_few(FusedArgs a, Gate gate)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const FusedSmem m = fused_smem(smem);
    fused_rows(a, m, wave, gate, [&](uint32_t row0, uint32_t row_end) {
        few_tile<kWaves, KS1, N1, N2>(a, m, wave, row0, row_end);
        return true;
    });
}


constexpr size_t kFusedLds = (size_t)FBM * LDH * 2 + 2 * FBM * 4 + (4 * HMAX + 32) * 4;
static_assert(kFewH <= FBM * LDH, "the few rows' activations in the tile's place");

template <int KS1, int N1, int N2, class Gate>
int launch_few(sf_ctx* ctx, const FusedArgs& a, const Gate& gate, uint32_t grid)
{
    SF_ALLOW_LDS(ctx, sf::kLdsFew + (std::is_same<Gate, sfsmall::NoGate>::value ? 0 : 8) + (KS1 == 8 ? 4 : 0) + (N1 - 1) * 2 + (N2 - 1),
                 (mlp_few<KS1, N1, N2, Gate>));
    mlp_few<KS1, N1, N2, Gate><<<grid, kWaves * 64, kFusedLds, ctx->stream>>>(a, gate);
    SF_LAUNCH_CHECK(ctx, "mlp_few");
    return SF_OK;
}

template <int KS1, class Gate>
int launch_few(sf_ctx* ctx, const FusedArgs& a, const Gate& gate, uint32_t grid)
{
    if (a.h1 > 32u * kWaves) return a.h2 > 32u * kWaves ? launch_few<KS1, 2, 2>(ctx, a, gate, grid) : launch_few<KS1, 2, 1>(ctx, a, gate, grid);
    return a.h2 > 32u * kWaves ? launch_few<KS1, 1, 2>(ctx, a, gate, grid) : launch_few<KS1, 1, 1>(ctx, a, gate, grid);
}

template <class Gate>
int launch_few(sf_ctx* ctx, const FusedArgs& a, const Gate& gate, uint32_t grid)
{
    return a.n_in <= 64u ? launch_few<4>(ctx, a, gate, grid) : launch_few<8>(ctx, a, gate, grid);
}

} // namespace

namespace sf {

bool slow_fused_ok(const sf_mlp* m, bool raw_input)
{
    return m->dtype == SF_BF16 && !raw_input && m->n_in <= HMAX && m->n_h1 <= HMAX && m->n_h2 <= HMAX && m->n_classes <= 32;
}

// the gate goes with the form for few rows a block (a list that the register form may take has the gate's own launches)
bool slow_fused_gates(sf_ctx* ctx, const sf_mlp* m, uint32_t n)
{
    return slow_fused_ok(m, false) && m->n_in <= kFewInput && n <= kRowsLine * (uint32_t)ctx->n_cu;
}

// the kernel reads kRing k-steps past the end of a column block: keep that much padding behind the last one
static size_t sw_bytes(uint32_t N, uint32_t K) { return align_up((size_t)(up(N, 32) / 32) * (up(K, kPadK) / 16) * 64 * 16 + (size_t)kRing * 1024); }

size_t slow_fused_ws_bytes(const sf_mlp* m)
{
    return sw_bytes(m->n_h1, m->n_in) + sw_bytes(m->n_h2, m->n_h1) + sw_bytes(32, m->n_h2) + 3 * kAlign;
}

size_t reordered_bytes(uint32_t N, uint32_t K) { return sw_bytes(N, K); }

int reorder_weights_async(sf_ctx* ctx, const ReorderSpec* specs, int n_specs)
{
    if (n_specs < 1 || n_specs > 3) return fail(ctx, SF_EINVAL, "reorder_weights_async: 1..3 matrices per launch");
    ReorderArgs r;
    r.total = 0;
    for (int q = 0; q < 3; ++q) {
        const ReorderSpec& sp = specs[q < n_specs ? q : n_specs - 1];
        r.job[q].w = (const uint16_t*)sp.w;
        r.job[q].N = sp.N;
        r.job[q].K = sp.K;
        r.job[q].NB = up(sp.N, 32) / 32;
        r.job[q].KS = up(sp.K, kPadK) / 16;
        r.job[q].first = r.total;
        r.job[q].out = (uint4*)sp.out;
        if (q < n_specs) r.total += r.job[q].NB * r.job[q].KS * 64 + (q == n_specs - 1 ? 64 : 0); // (and a fragment of zeros behind the last one)
    }
    // jobs past n_specs start at r.total, so no element maps to them
    uint32_t blocks = (r.total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    reorder_weights<<<blocks, 256, 0, ctx->stream>>>(r);
    SF_LAUNCH_CHECK(ctx, "reorder_weights");
    return SF_OK;
}

// w1 | w2 | w3 in operand order, at the offsets every consumer uses (the last layer padded to 32 columns)
int order_all(sf_ctx* ctx, const sf_mlp* m, void* out)
{
    char* p = (char*)out;
    uint4* w1s = (uint4*)p;
    p += sw_bytes(m->n_h1, m->n_in);
    uint4* w2s = (uint4*)p;
    p += sw_bytes(m->n_h2, m->n_h1);
    uint4* w3s = (uint4*)p;
    const ReorderSpec specs[3] = {{m->w1, m->n_h1, m->n_in, w1s}, {m->w2, m->n_h2, m->n_h1, w2s},
                                  {m->w3, m->n_classes, m->n_h2, w3s}};
    return reorder_weights_async(ctx, specs, 3);
}

int slow_fused(sf_ctx* ctx, void* ws, bool ws_is_ordered, const float* feat, uint32_t feat_ld, uint32_t n_rows,
               const uint32_t* esc_idx, const uint32_t* scatter, const uint32_t* esc_count, uint32_t esc_cap,
               uint32_t n_labels, const sf_mlp* m, const uint16_t* pred, const sfsmall::GateRows* gate, float* logits, uint16_t* labels)
{
    char* p = (char*)ws;
    uint4* w1s = (uint4*)p;
    p += sw_bytes(m->n_h1, m->n_in);
    uint4* w2s = (uint4*)p;
    p += sw_bytes(m->n_h2, m->n_h1);
    uint4* w3s = (uint4*)p;
    if (!ws_is_ordered) {
        const int rc = order_all(ctx, m, ws);
        if (rc != SF_OK) return rc;
    }
    FusedArgs a;
    a.esc_idx = esc_idx;
    a.scatter = scatter;
    a.esc_count = esc_count;
    a.esc_cap = esc_cap;
    a.n_rows = n_rows;
    a.n_labels = n_labels;
    a.feat = feat;
    a.feat_ld = feat_ld;
    a.mu = m->mu;
    a.inv_sigma = m->inv_sigma;
    a.clamp = m->clamp;
    a.n_in = m->n_in;
    a.h1 = m->n_h1;
    a.h2 = m->n_h2;
    a.c = m->n_classes;
    a.w1s = w1s;
    a.w2s = w2s;
    a.w3s = w3s;
    a.b1 = m->b1;
    a.b2 = m->b2;
    a.b3 = m->b3;
    a.logits = logits;
    a.labels = labels;
    a.pred = pred;
    a.n_copy = 0;
    // Register form: lists that may give a compute unit more than 128 rows (192 where the passes have no
    // registers left to run ahead, more than 64 inputs and 384 columns in the first layer, unless their pieces are whole and the second layer
    // small: tiles : this form, 128-455-469-17 33,000 rows 39.3 : 46.6 us, 49,152 38.9 : 47, 60,000 about equal; 128-512-512-10 36.2 : 39.4; but
    // 96-512-100-7 26.8 : 23.4), and models whose second layer is not wide for the first
    // one's depth (a column block's work beside its MFMAs is the same whatever the depth: 300,000 rows 60-40-500-10 106 : 112 us, 64-200-500-10
    // 137 : 130, 24,500 of them 19.1 : 24.4).
    // The capacity decides, since the count is on the device, and a long list may hold few rows.  In us, tiles of eight waves : this
    // form under a capacity of 300,000: 64-512-512-10 8,000 rows 15.2 : 14.5, 16,000 15.1 : 16.2, 32,000 23.1 : 23.3, 60,000 43 : 35;
    // 96-300-200-10 11.3 : 10.4, 11.2 : 12.5, 17.6 : 17.2, 33 : 27; 32-256-256-10 9.7 : 9.9, 9.9 : 10.0, 13.3 : 15.6, 26 : 20.5.  So a line
    // further up would lose more on full lists than it gave on sparse ones.
    const uint32_t nb1 = up(a.h1, 32) / 32u, nb2 = up(a.h2, 32) / 32u;
    const bool tight = a.n_in > 64u && nb1 > 12u && (nb1 < 16u || nb2 > 12u || nb2 % 2u != 0);
    const uint32_t line = tight ? 192u : kRowsLine;
    if (esc_cap > line * (uint32_t)ctx->n_cu && nb2 <= 2u * nb1 && a.n_in <= 128 && (a.n_in & 3u) == 0 && (feat_ld & 3u) == 0 &&
        ((uintptr_t)feat & 15u) == 0) {
        if (pred) {
            const int rc = copy_labels_async(ctx, pred, labels, n_labels);
            if (rc != SF_OK) return rc;
        }
        sfrows::RowsArgs r;
        static_cast<FusedArgs&>(r) = a;
        r.clamp_z = a.mu ? a.clamp : __builtin_inff();
        r.nb1 = nb1;
        r.nb2 = nb2;
        r.ks2 = up(a.h1, kPadK) / 16u;
        r.ks3 = up(a.h2, kPadK) / 16u;
        return sfrows::run(ctx, r);
    }
    const uint32_t rb_cap = (esc_cap + 31u) / 32u;
    uint32_t grid = (uint32_t)ctx->n_cu; // one block per compute unit (its shared memory fills the unit)
    if (grid > rb_cap) grid = rb_cap;
    if (grid == 0) grid = 1;
    if (gate) return launch_few(ctx, a, *gate, grid);
    if (pred && n_labels <= sfsmall::kCopyRows && n_labels <= kCopyUnit * (uint32_t)ctx->n_cu) {
        a.n_copy = (n_labels + sfsmall::kCopySlice - 1u) / sfsmall::kCopySlice;
        grid += a.n_copy;
    } else if (pred) {
        const int rc = copy_labels_async(ctx, pred, labels, n_labels);
        if (rc != SF_OK) return rc;
    }
    if (a.n_in <= kFewInput) return launch_few(ctx, a, sfsmall::NoGate{}, grid);
    SF_ALLOW_LDS(ctx, sf::kLdsFused, mlp_fused);
    mlp_fused<<<grid, kWaves * 64, kFusedLds, ctx->stream>>>(a);
    SF_LAUNCH_CHECK(ctx, "mlp_fused");
    return SF_OK;
}

} // namespace sf
