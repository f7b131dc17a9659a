// kvcomm_anchor_weights: anchor matching.  l2 distance between the segment's base keys and
// each selected anchor's base keys, then the softmax of the negative distance across the
// anchor dimension (Eq. "pred", Eq. "ph_update" and the weight step of Algorithm 1; the
// appendix on long-context anchor matching gives the reduced shape [m,1,1,seq_len,1]).
//
// Deterministic stages, no floating-point atomics:
//   1. dist_partial_kernel streams the key rows once (HBM-bound: (A+1) rows per
//      (layer, head, token)) and leaves, per block, the squared distance of its chunk of
//      (layer, head) pairs: partial[chunk][token][anchor] in double.
//   2. finalize_kernel adds the chunks in a fixed order, takes the square root and the
//      softmax in double, and writes fp32 weights, the nearest anchor and the selection.
// Per-token weights of pools that fit a block's anchor tiles take one launch instead where there are tokens enough to fill the chip
// (token_weights_kernel), and so do per-(layer, head, token) weights (dist_row_softmax_kernel): same sums, another fixed order.
// Squared differences are accumulated in double so that fp32 inputs keep ~1e-7 relative
// accuracy in the weights and the arg-min is decided in the precision the definition uses.
//
// kvcomm_anchor_weights_rule adds the two weighting variants of the appendix on the
// approximation method: "nearest" (same distances, one-hot at the arg-min) and "cosine"
// (cos_partial_kernel leaves <x,y>, |x|^2 and |y|^2 per chunk; the softmax runs over the
// similarities).  Both reuse the two-stage structure and the finalize kernels.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "kvcomm_device.h"

// Partial sums of kvcomm_anchor_weights_static: one array per GPU that has loaded the library, kept
// until the process ends.  In host code this name is only a handle for hipGetSymbolAddress; the
// kernels receive the address that call returns.
static __device__ __align__(256) unsigned char scratch[KVCOMM_STATIC_SCRATCH_BYTES];

namespace {

using namespace kvc;

constexpr int kBlock = 256;
constexpr int kFinalBlock = 512; // threads of a finalize_kernel block
constexpr int kSegBlock = 1024;  // threads of a finalize_segment_kernel block
constexpr int kFinalRun = 16;    // partials of one chunk that stay together in a finalize_kernel block
constexpr int kFinalLanes = 16;  // threads that share the chunks of a (slot, anchor) pair: at most this many, or one per eight chunks
constexpr int kGroupPairs = 32;  // (chunk, token tile) pairs of a group, a multiple of 8
constexpr int kMaxGroups = 32768;  // extent of the grid in z (the hardware takes 65535)
constexpr int kAnchorTile = 16;  // anchors whose accumulators one lane keeps in registers

// Blocks per segment the distance grid aims at.  Fewer blocks = longer runs of (layer, head) pairs = fewer partial sums for the
// second stage: 512 for short segments.  Three blocks per compute unit (768) where runs stay long, kLongRun pairs and more: small
// pools then have enough loads in flight, and the runs of 512 blocks, a power of two of kFarApart bytes and more apart, meet in the
// same memory channels.  Batches whose runs are closer together have blocks enough with 512 per segment.
// us per call, both stages, input sets in no cache, with 512 / 768 / 1024 / 2048 blocks (H = 8, L = 8 ... 32):
//   77 tokens, 12 anchors, cosine, D 64   21 / 27 / 27 / 27      200 tokens, 12 anchors, D 256         40 / 45 / 46 / 46
//   512 tokens, 4 anchors, f32 D 128      40 / 34 / 34 / 33      1024 tokens, 1 anchor, D 256          61 / 50 / 53 / 52
//   8 x 512 tokens, 5 anchors, f32 D 128  301 / 261 / 263 / 253  4 x 512 tokens, 8 anchors, D 128      188 / 193 / 187 / 194
constexpr int kDistBlocks = 512, kDistBlocksLong = 768, kLongRun = 9;
constexpr int64_t kFarApart = (int64_t)4 << 20;

// How a launch is cut into blocks.  Rows of one (layer, head) are LPR lanes wide; a block owns RPB
// consecutive tokens and a run of lh_per_block (layer, head) pairs ("chunk").
struct DistPlan {
    int lpr;            // lanes per row = D / EPV
    int rpb;            // rows (tokens) per block
    int lh_per_block;
    int n_chunks;
};

// seg_lens: the segments of the launch (one for the single-segment entry points).
DistPlan make_plan(const kvcomm_model *m, const int32_t *seg_lens, int n_jobs, int gran)
{
    DistPlan pl;
    const int epv = 16 / elem_size(m->dtype);
    pl.lpr = m->head_dim / epv;
    pl.rpb = kBlock / pl.lpr;
    const int LH = m->n_layers * m->n_kv_heads;
    if (gran == KVCOMM_W_LAYER_HEAD_TOKEN) {
        pl.lh_per_block = 1;
    } else {
        int64_t tiles = 0;
        for (int j = 0; j < n_jobs; ++j) tiles += (seg_lens[j] + pl.rpb - 1) / pl.rpb;
        auto run_of = [&](int64_t blocks) {   // (layer, head) pairs per block
            const int64_t n_chunks = std::max<int64_t>(1, std::min<int64_t>(LH, (blocks * n_jobs + tiles - 1) / tiles));
            return (int)((LH + n_chunks - 1) / n_chunks);
        };
        int64_t longest = 0;
        for (int j = 0; j < n_jobs; ++j) longest = std::max<int64_t>(longest, seg_lens[j]);
        pl.lh_per_block = run_of(kDistBlocksLong);
        const int64_t run_bytes = run_of(kDistBlocks) * longest * m->head_dim * elem_size(m->dtype);
        if (pl.lh_per_block < kLongRun || (n_jobs > 1 && run_bytes < kFarApart)) pl.lh_per_block = run_of(kDistBlocks);
    }
    pl.n_chunks = (LH + pl.lh_per_block - 1) / pl.lh_per_block;
    return pl;
}

struct DistJob {
    const void *seg_k;
    Strides s_seg;
    double *partial;       // [component][n_chunks][S][n_sel]
    int64_t comp_stride;   // elements between components (cosine rule)
    int32_t S, n_token_tiles;
    int16_t a0, n_sel;     // its selected anchors: entries [a0, a0 + n_sel) of anc
    // outputs of the fused form (per-(layer, head, token) weights straight from the distance kernel)
    float *weights;
    int32_t *nearest;
    int32_t *selected_out;
    uint64_t sel_mask;     // bit a = anchor a is selected
    divisor_t by_tiles;    // of n_token_tiles
    int32_t n_anchors;
};

struct DistParams {   // (begins with what every block reads first)
    Strides s_anc;
    int32_t H, LH, lh_per_block, n_jobs;
    int32_t fused, rule;   // fused: a row's distances are complete inside its lanes; write the weights here
    int32_t n_blocks, group_pairs, tile_anchors;   // distance kernel: (chunk, token tile) pairs of all segments and of a group, anchors of a tile
    int32_t tok_shift;     // token_weights_kernel: log2 of the tokens of a block
    int32_t per_segment;   // one weight set per segment: a block also adds up its rows (partial[chunk][tile][anchor])
    double tau;
    divisor_t by_H;
    int32_t block0[KVCOMM_MAX_BATCH];   // first block of a segment
    DistJob job[KVCOMM_MAX_BATCH];
    const void *anc[KVCOMM_MAX_ANCHORS + kAnchorTile];  // selected anchors of all segments (a tile's pointers are read without a look at how many it has)
    uint8_t col[KVCOMM_MAX_ANCHORS];      // original index of a selected anchor
};
static_assert(sizeof(DistParams) <= 4096, "kernel arguments are limited to 4 KB");

__device__ __forceinline__ void await_dist_args(const DistParams &p)
{
    await_args(arg_word(&p), arg_word(&p.rule), arg_word(p.block0), arg_word(&p.job[0]), arg_word(&p.job[0].S), arg_word(p.anc), arg_word(p.anc + 8),
               arg_word(p.col));
}

template <class P>
__device__ __forceinline__ int job_of_block(const P &p, int block)
{
    int ji = 0;
#pragma unroll
    for (int i = 1; i < KVCOMM_MAX_BATCH; ++i)
        if (i < p.n_jobs && block >= p.block0[i]) ji = i;
    return ji;
}

// The grid of the two-stage distance kernels is (pairs of a group, anchor tiles, groups) over the (chunk, token tile) pairs of
// all segments.  With groups of a few pairs the anchor tiles of one pair run at about the same time on the same XCD (hardware
// deals block ids, x fastest, round-robin to the 8 XCDs), so that the segment's rows come from HBM once and from the XCD's L2
// after that.  Where the segments of a launch have different numbers of l2 tiles, one group holds all pairs: between each other
// the tiles that a small pool does not have would leave the same compute units without work (pools of 20, 3 and 3 anchors, 512
// tokens each, D = 256, 16 layers x 8 heads: 191 us in groups, 158 in one).  The cosine rule's narrower tiles gain more from
// the L2 than they lose (the same pools, 32 layers: 309 us in groups, 354 in one).
__device__ __forceinline__ int pair_of_block(const DistParams &p) { return blockIdx.z * p.group_pairs + blockIdx.x; }

// Sum of squared differences of two 16-byte vectors, added to a double accumulator.
template <typename T>
__device__ __forceinline__ void sqdiff_acc(double &acc, const float (&x)[Elem<T>::EPV], const u32x4 raw)
{
    float y[Elem<T>::EPV];
    unpack<T>(raw, y);
#pragma unroll
    for (int e = 0; e < Elem<T>::EPV; ++e) {
        const double d = (double)x[e] - (double)y[e];
        acc = fma(d, d, acc);
    }
}

// Anchor pointers of a tile in scalar registers for the whole kernel.  (Read where they are used, each anchor's load waited
// for a scalar load of its own pointer, in every (layer, head) pair.)  All NA are read in one go, also behind the tile's last
// anchor (never followed): picked one by one they held up the first rows of blocks that walk one pair only (cosine, 1 anchor,
// per-(layer, head, token) weights: 47 against 44 us).
template <typename T, int NA>
struct AnchorPtrs {
    typedef const __attribute__((address_space(1))) u32x4 gvec;
    uint64_t ptr[NA];
    __device__ __forceinline__ AnchorPtrs(const DistParams &p, int first)
    {
#pragma unroll
        for (int j = 0; j < NA; ++j) ptr[j] = reinterpret_cast<uint64_t>(p.anc[first + j]);
#pragma unroll
        for (int j = 0; j < NA; ++j) asm volatile("" : "+s"(ptr[j]));
    }
    __device__ __forceinline__ u32x4 load(int j, int64_t off) const   // off in elements
    {
        return __builtin_nontemporal_load(reinterpret_cast<gvec *>(ptr[j] + (uint64_t)(off * (int64_t)sizeof(T))));
    }
};

// HBM bound.  What keeps loads in flight: all row pieces of a (layer, head) pair are requested before the first is used,
// without a branch between them when the tile is full; tiles of 4 and 8 anchors for small pools hold fewer registers, so
// more wavefronts fit.  The anchors' rows are read once and marked non-temporal; the segment's rows are plain loads: the
// tiles of a large pool share them (fetched by every one of the four tiles of 64 anchors, the distance stage of 1024 tokens
// took 7 % longer), and the update that follows reads the same rows again.  4 x 512 tokens, 8 anchors, inputs that are in
// no cache: 185 us = 6.5 TB/s (191 us before).
template <typename T, int LPR, int NA>   // NA: anchors of a tile (accumulators of a lane)
__global__ __launch_bounds__(kBlock) void dist_partial_kernel(const DistParams p)
{
    constexpr int EPV = Elem<T>::EPV;
    constexpr int RPB = kBlock / LPR;
    await_dist_args(p);
    const int block = pair_of_block(p);
    if (block >= p.n_blocks) return;
    const int ji = job_of_block(p, block);
    const DistJob &jb = p.job[ji];
    if (ji > 0) await_args(arg_word(&jb), arg_word(&jb.sel_mask));
    const int tid = threadIdx.x;
    const int row = tid / LPR, lir = tid % LPR;
    const int bx = block - p.block0[ji];
    const int chunk = div_by(bx, jb.by_tiles);
    const int tile = bx - chunk * jb.n_token_tiles;
    const int a0 = blockIdx.y * p.tile_anchors;
    const int na = min(p.tile_anchors, jb.n_sel - a0);
    // (Fewer registers: 80 and six wavefronts per SIMD instead of 83 and five with 8 anchors.  With 16, bf16, 129 and three; held to 128 and four
    // it measured the same: 1024 tokens, 64 anchors 645 and 647 us, 16 anchors 178 and 178, 33 tokens, 64 anchors 40.0 and 39.5.)
    __builtin_assume(na <= NA);
    if (na <= 0) return;  // the launch's anchor tiles cover the largest pool of the launch
    const int t = tile * RPB + row;
    const bool valid = t < jb.S;
    const int lh0 = chunk * p.lh_per_block;
    const int lh1 = min(lh0 + p.lh_per_block, p.LH);

    double acc[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) acc[j] = 0.0;

    const AnchorPtrs<T, NA> anc(p, jb.a0 + a0);
    const T *seg = static_cast<const T *>(jb.seg_k) + t * jb.s_seg.token + lir * EPV;
    const int64_t arow = t * p.s_anc.token + lir * EPV;
    auto walk = [&](auto full) __attribute__((always_inline)) {   // full: every anchor of the tile exists (no branches)
        for (int lh = lh0; lh < lh1; ++lh) {
            const int l = div_by(lh, p.by_H), h = lh - l * p.H;
            const T *sp = seg + l * jb.s_seg.layer + h * jb.s_seg.head;
            const u32x4 rs = load16(sp);   // plain: see above
            const int64_t aoff = arow + l * p.s_anc.layer + h * p.s_anc.head;
            u32x4 ra[NA];
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (decltype(full)::value || j < na) ra[j] = anc.load(j, aoff);
            float x[EPV];
            unpack<T>(rs, x);
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (decltype(full)::value || j < na) sqdiff_acc<T>(acc[j], x, ra[j]);
        }
    };
    if (valid) {
        if (na == NA)
            walk(std::true_type{});
        else
            walk(std::false_type{});
    }
    // Fixed-shape butterfly over the LPR lanes of a row (all inside one wavefront).
    __shared__ double rows[RPB][NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        if (j < na) {
            double v = acc[j];
#pragma unroll
            for (int off = LPR / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, LPR);
            if (p.per_segment) {
                if (lir == 0) rows[row][j] = valid ? v : 0.0;
            } else if (valid && lir == 0) {
                jb.partial[((int64_t)chunk * jb.S + t) * jb.n_sel + a0 + j] = v;
            }
        }
    }
    if (p.per_segment) {  // the block's rows in a fixed order: one partial per (chunk, token tile, anchor)
        __syncthreads();
        if (tid < na) {
            double v = 0.0;
            for (int r = 0; r < RPB; ++r) v += rows[r][tid];
            jb.partial[((int64_t)chunk * jb.n_token_tiles + tile) * jb.n_sel + a0 + tid] = v;
        }
    }
}

// Reduce-scatter of NA per-lane sums over the LPR lanes of a row (LPR a power of two, lanes of a row are
// consecutive): afterwards lane `lir` holds the row's totals of its own anchors in acc[0 .. max(1, NA /
// LPR)), anchor_of_lane() says which.  Lanes NA and up of a wider row hold copies that anchor_of_lane() maps
// past the tile, so they are ignored.
template <int LPR, int NA>
__device__ __forceinline__ int anchor_of_lane(int lir, int k)
{
    if constexpr (LPR >= NA)
        return lir + k * LPR;              // k == 0: anchor lir (invalid from NA on)
    else
        return (NA / LPR) * lir + k;
}
template <int CNT, int OFF, int LPR, int NA>
__device__ __forceinline__ void reduce_scatter_round(double (&acc)[NA], int lir)
{
    if constexpr (OFF >= 1 && CNT >= 2) {
        const bool up = lir & OFF;
#pragma unroll
        for (int i = 0; i < CNT / 2; ++i) {
            const double keep = up ? acc[i + CNT / 2] : acc[i];
            const double send = up ? acc[i] : acc[i + CNT / 2];
            acc[i] = keep + __shfl_xor(send, OFF, LPR);
        }
        reduce_scatter_round<CNT / 2, OFF / 2, LPR, NA>(acc, lir);
    }
}
template <int LPR, int NA>
__device__ __forceinline__ void row_reduce_scatter(double (&acc)[NA], int lir)
{
    static_assert((NA & (NA - 1)) == 0, "anchor tiles are powers of two");
#pragma unroll
    for (int off = LPR / 2; off >= NA; off >>= 1)
#pragma unroll
        for (int j = 0; j < NA; ++j) acc[j] += __shfl_xor(acc[j], off, LPR);
    constexpr int OFF0 = (LPR < NA ? LPR : NA) / 2;
    reduce_scatter_round<NA, OFF0, LPR, NA>(acc, lir);
}

// One softmax per (layer, head, token), pools of up to kAnchorTile selected anchors: a row's distances are
// complete inside the LPR lanes that read the row, so this kernel finishes the softmax itself and writes the
// weights (no partial sums, no second kernel).
// Lane r of a row takes anchors r, r + LPR, ...; maximum, arg-max (lowest index among equals) and denominator
// are joined by fixed butterflies, so all lanes of a row agree bit for bit.  The exponent is formed in double
// (distances of a few hundred differ by fractions); the exponential and the normalisation are fp32, which is
// what the fp32 weights can resolve.
template <typename T, int LPR, int NA>   // NA >= the largest pool of the launch
__global__ __launch_bounds__(kBlock) void dist_row_softmax_kernel(const DistParams p)
{
    constexpr int EPV = Elem<T>::EPV;
    constexpr int RPB = kBlock / LPR;
    constexpr int NPL = (NA + LPR - 1) / LPR;  // anchors per lane
    await_dist_args(p);
    const int ji = job_of_block(p, blockIdx.x);
    const DistJob &jb = p.job[ji];
    if (ji > 0) await_args(arg_word(&jb), arg_word(&jb.sel_mask));
    const int tid = threadIdx.x;
    const int row = tid / LPR, lir = tid % LPR;
    const int bx = blockIdx.x - p.block0[ji];
    const int chunk = div_by(bx, jb.by_tiles);
    const int tile = bx - chunk * jb.n_token_tiles;
    const int na = jb.n_sel;  // 1 ... NA (checked by the host)
    const int t = tile * RPB + row;
    const bool valid = t < jb.S;
    const int lh0 = chunk * p.lh_per_block;
    const int lh1 = min(lh0 + p.lh_per_block, p.LH);
    if (bx == 0 && jb.selected_out && tid < jb.n_anchors) jb.selected_out[tid] = (int32_t)((jb.sel_mask >> tid) & 1);

    const AnchorPtrs<T, NA> anc(p, jb.a0);
    const T *seg = static_cast<const T *>(jb.seg_k) + t * jb.s_seg.token + lir * EPV;
    const int64_t arow = t * p.s_anc.token + lir * EPV;
    for (int lh = lh0; lh < lh1; ++lh) {
        double acc[NA];
#pragma unroll
        for (int j = 0; j < NA; ++j) acc[j] = 0.0;
        auto add_row = [&](auto full) __attribute__((always_inline)) {   // full: na == NA (no branches)
            const int l = div_by(lh, p.by_H), h = lh - l * p.H;
            const u32x4 rs = load16(seg + l * jb.s_seg.layer + h * jb.s_seg.head);
            const int64_t aoff = arow + l * p.s_anc.layer + h * p.s_anc.head;
            u32x4 ra[NA];
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (decltype(full)::value || j < na) ra[j] = anc.load(j, aoff);
            float x[EPV];
            unpack<T>(rs, x);
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (decltype(full)::value || j < na) sqdiff_acc<T>(acc[j], x, ra[j]);
        };
        if (valid) {
            if (na == NA)
                add_row(std::true_type{});
            else
                add_row(std::false_type{});
        }
        // Sum over the lanes of the row and hand each lane its own anchors in one go: in every round a lane keeps
        // one half of its values and adds the partner's copy of that half (15 exchanges for 16 anchors over 16
        // lanes instead of 64 for a butterfly per anchor).  Rows wider than NA lanes first fold their upper lanes in.
        row_reduce_scatter<LPR, NA>(acc, lir);
        double sc[NPL];
        double smax = -INFINITY;
        int best = NA;
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            const int a = anchor_of_lane<LPR, NA>(lir, k);
            sc[k] = a < na ? -sqrt(acc[k]) : -INFINITY;
            if (sc[k] > smax) {  // ascending a: the lowest index wins among equals
                smax = sc[k];
                best = a;
            }
        }
#pragma unroll
        for (int off = LPR / 2; off >= 1; off >>= 1) {
            const double om = __shfl_xor(smax, off, LPR);
            const int ob = __shfl_xor(best, off, LPR);
            if (om > smax || (om == smax && ob < best)) {
                smax = om;
                best = ob;
            }
        }
        float e[NPL], denom = 0.f;
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            const int a = anchor_of_lane<LPR, NA>(lir, k);
            e[k] = a < na ? (p.rule == KVCOMM_RULE_NEAREST ? (a == best ? 1.f : 0.f)
                                                           : expf((float)((sc[k] - smax) / p.tau)))
                          : 0.f;
            denom += e[k];
        }
#pragma unroll
        for (int off = LPR / 2; off >= 1; off >>= 1) denom += __shfl_xor(denom, off, LPR);
        if (valid) {
            const int64_t slot = (int64_t)lh * jb.S + t;
            float *wrow = jb.weights + slot * jb.n_anchors;
#pragma unroll
            for (int k = 0; k < NPL; ++k) {
                const int a = anchor_of_lane<LPR, NA>(lir, k);
                if (a < na) wrow[p.col[jb.a0 + a]] = e[k] / denom;
            }
            for (int c = lir; c < jb.n_anchors; c += LPR)
                if (!((jb.sel_mask >> c) & 1)) wrow[c] = 0.f;
            // best == NA: no distance is finite; equal distances, so the lowest index, as in the two-stage form
            if (lir == 0 && jb.nearest) jb.nearest[slot] = p.col[jb.a0 + (best < na ? best : 0)];
        }
    }
}

constexpr int kCosTile = 8;  // anchors per lane in the cosine variant (two accumulators each)

// Cosine variant: per chunk, token and selected anchor the three sums <x,y>, |x|^2, |y|^2
// (x = segment key row, y = anchor key row), laid out [component][chunk][token][anchor].
template <typename T, int LPR>
__global__ __launch_bounds__(kBlock) void cos_partial_kernel(const DistParams p)
{
    constexpr int EPV = Elem<T>::EPV;
    constexpr int RPB = kBlock / LPR;
    await_dist_args(p);
    const int block = pair_of_block(p);
    if (block >= p.n_blocks) return;
    const int ji = job_of_block(p, block);
    const DistJob &jb = p.job[ji];
    if (ji > 0) await_args(arg_word(&jb), arg_word(&jb.sel_mask));
    const int tid = threadIdx.x;
    const int row = tid / LPR, lir = tid % LPR;
    const int bx = block - p.block0[ji];
    const int chunk = div_by(bx, jb.by_tiles);
    const int tile = bx - chunk * jb.n_token_tiles;
    const int a0 = blockIdx.y * p.tile_anchors;
    const int na = min(p.tile_anchors, jb.n_sel - a0);
    __builtin_assume(na <= kCosTile);
    if (na <= 0) return;
    const int t = tile * RPB + row;
    const bool valid = t < jb.S;
    const int lh0 = chunk * p.lh_per_block;
    const int lh1 = min(lh0 + p.lh_per_block, p.LH);

    __shared__ double rows[RPB][kCosTile][3];
    double dot[kCosTile], ny[kCosTile], nx = 0.0;
#pragma unroll
    for (int j = 0; j < kCosTile; ++j) dot[j] = ny[j] = 0.0;

    const AnchorPtrs<T, kCosTile> anc(p, jb.a0 + a0);
    if (valid) {
        const T *seg = static_cast<const T *>(jb.seg_k) + t * jb.s_seg.token + lir * EPV;
        const int64_t arow = t * p.s_anc.token + lir * EPV;
        for (int lh = lh0; lh < lh1; ++lh) {
            const int l = div_by(lh, p.by_H), h = lh - l * p.H;
            const u32x4 rs = load16(seg + l * jb.s_seg.layer + h * jb.s_seg.head);
            const int64_t aoff = arow + l * p.s_anc.layer + h * p.s_anc.head;
            u32x4 ra[kCosTile];
#pragma unroll
            for (int j = 0; j < kCosTile; ++j)
                if (j < na) ra[j] = anc.load(j, aoff);
            float x[EPV];
            unpack<T>(rs, x);
#pragma unroll
            for (int e = 0; e < EPV; ++e) nx = fma((double)x[e], (double)x[e], nx);
#pragma unroll
            for (int j = 0; j < kCosTile; ++j)
                if (j < na) {
                    float y[EPV];
                    unpack<T>(ra[j], y);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) {
                        dot[j] = fma((double)x[e], (double)y[e], dot[j]);
                        ny[j] = fma((double)y[e], (double)y[e], ny[j]);
                    }
                }
        }
    }
#pragma unroll
    for (int off = LPR / 2; off >= 1; off >>= 1) nx += __shfl_xor(nx, off, LPR);
#pragma unroll
    for (int j = 0; j < kCosTile; ++j) {
        if (j < na) {
            double u = dot[j], v = ny[j];
#pragma unroll
            for (int off = LPR / 2; off >= 1; off >>= 1) {
                u += __shfl_xor(u, off, LPR);
                v += __shfl_xor(v, off, LPR);
            }
            if (p.per_segment) {
                if (lir == 0) {
                    rows[row][j][0] = valid ? u : 0.0;
                    rows[row][j][1] = valid ? nx : 0.0;
                    rows[row][j][2] = valid ? v : 0.0;
                }
            } else if (valid && lir == 0) {
                const int64_t i = ((int64_t)chunk * jb.S + t) * jb.n_sel + a0 + j;
                jb.partial[i] = u;
                jb.partial[jb.comp_stride + i] = nx;
                jb.partial[2 * jb.comp_stride + i] = v;
            }
        }
    }
    if (p.per_segment) {
        __syncthreads();
        if (tid < 3 * na) {
            const int j = tid / 3, c = tid % 3;
            double v = 0.0;
            for (int r = 0; r < RPB; ++r) v += rows[r][j][c];
            jb.partial[c * jb.comp_stride + ((int64_t)chunk * jb.n_token_tiles + tile) * jb.n_sel + a0 + j] = v;
        }
    }
}

struct FinalJob {
    const double *partial;
    float *weights;
    int32_t *nearest;
    int32_t *selected_out;
    int64_t comp_stride;   // cosine rule: elements between the three partial components
    uint64_t sel_mask;     // bit a = anchor a is selected
    int32_t S, n_slots, n_anchors, chunk_lanes, n_token_tiles;
    int16_t a0, n_sel;     // its selected anchors: entries [a0, a0 + n_sel) of col
};

struct FinalParams {   // (begins with what every block reads first)
    int32_t n_chunks, gran, rule, n_jobs;
    double tau;
    int32_t block0[KVCOMM_MAX_BATCH];  // first block of a segment
    uint64_t pad_;
    FinalJob job[KVCOMM_MAX_BATCH];
    uint8_t col[KVCOMM_MAX_ANCHORS];   // original index of a selected anchor
};

// Score whose softmax across anchors gives the weights: minus the l2 distance, or the cosine
// similarity <x,y> / (|x| |y|) (0 when a norm is 0).
__device__ __forceinline__ double score_of(int rule, double s0, double s1, double s2)
{
    if (rule != KVCOMM_RULE_COSINE_SOFTMAX) return -sqrt(s0);
    const double den = sqrt(s1) * sqrt(s2);
    return den > 0.0 ? s0 / den : 0.0;
}

// Softmax over the selected anchors of one slot: maximum and arg-max from the scores in `sc` (LDS), walked in index order
// by each of the slot's threads, so all agree bit for bit; every thread forms the exponential of its own anchor only and
// the denominator is the sum of the n_sel exponentials in `ex` (LDS) in index order.  `act`: this thread owns anchor
// `a` of `slot`.  Called by whole blocks (it synchronises them once).
template <class Params, class Job>
__device__ __forceinline__ void slot_softmax(const Params &p, const Job &jb, const double *sc, double *ex, int a, int64_t slot,
                                             bool act)
{
    int best = 0;
    double w = 0.0;
    if (act) {
        double smax = sc[0];
        for (int j = 1; j < jb.n_sel; ++j) {
            const double v = sc[j];
            if (v > smax) {
                smax = v;
                best = j;
            }
        }
        w = p.rule == KVCOMM_RULE_NEAREST ? (a == best ? 1.0 : 0.0) : exp((sc[a] - smax) / p.tau);
        ex[a] = w;
    }
    __syncthreads();
    if (!act) return;
    if (p.rule != KVCOMM_RULE_NEAREST) {
        double denom = 0.0;
        for (int j = 0; j < jb.n_sel; ++j) denom += ex[j];
        w /= denom;
    }
    jb.weights[slot * jb.n_anchors + p.col[jb.a0 + a]] = (float)w;
    if (a == 0) {
        if (jb.nearest) jb.nearest[slot] = p.col[jb.a0 + best];
        for (int c = 0; c < jb.n_anchors; ++c)
            if (!((jb.sel_mask >> c) & 1)) jb.weights[slot * jb.n_anchors + c] = 0.f;
    }
}

// Per-token and per-(layer, head, token) granularity.  A (slot, selected anchor) pair is summed by CL threads:
// thread (c, slot, anchor) adds chunks c, c + CL, ... in increasing order (anchor, then slot, vary fastest over the
// threads, so a wavefront reads runs of a chunk's row), the CL sums meet in LDS and are added in increasing c, so the
// result does not depend on timing.
// The kernel is a chain of latencies (chunk loads, LDS sums, a double-precision root and exponential), so the chunks are
// spread over several threads, runs of 16 partials (128 bytes) stay together, and every exponential is formed once.  Up to 16
// threads per pair (or one per eight chunks): with 32 the second chain, of LDS sums, takes longer than what the first one
// saves (cosine, 2 anchors, 64 chunks: 6.4 us with 32, 5.3 with 16; 77 tokens, 5 anchors, l2, both stages: 18.6 and 17.8).
// Against eight threads per pair and n_sel exponentials in each, with the chunk counts of that time: 77 tokens, 5 anchors 14.1 -> 6.0
// us; 4 x 512 tokens, 8 anchors 7.6 -> 5.5; 1024 tokens, 64 anchors 16.6 -> 10.2.
__global__ __launch_bounds__(kFinalBlock) void finalize_kernel(const FinalParams p)
{
    __shared__ double dsh[kFinalBlock], esh[kFinalBlock];
    __shared__ double red[3][kFinalBlock];
    await_args(arg_word(&p), arg_word(&p.job[0]), arg_word(&p.job[0].n_slots), arg_word(p.col));
    const int ji = job_of_block(p, blockIdx.x);
    const FinalJob &jb = p.job[ji];
    if (ji > 0) await_args(arg_word(&jb), arg_word(&jb.n_token_tiles));
    const int bx = blockIdx.x - p.block0[ji];
    const int tid = threadIdx.x;
    if (bx == 0 && jb.selected_out && tid < jb.n_anchors) jb.selected_out[tid] = (int32_t)((jb.sel_mask >> tid) & 1);
    if (jb.n_sel == 0) {  // nothing selected: all weights 0, nearest -1
        const int64_t slot = (int64_t)bx * kFinalBlock + tid;
        if (slot < jb.n_slots) {
            for (int c = 0; c < jb.n_anchors; ++c) jb.weights[slot * jb.n_anchors + c] = 0.f;
            if (jb.nearest) jb.nearest[slot] = -1;
        }
        return;
    }
    const int CL = jb.chunk_lanes;                  // CL * n_sel <= kFinalBlock
    const int spb = kFinalBlock / (CL * jb.n_sel);  // slots per block
    const int per_lane = spb * jb.n_sel;            // (slot, anchor) pairs of a block
    const int a = tid % jb.n_sel, sl = (tid / jb.n_sel) % spb, cl = tid / per_lane;
    const int64_t slot = (int64_t)bx * spb + sl;
    const bool active = cl < CL && slot < jb.n_slots;
    const bool cosine = p.rule == KVCOMM_RULE_COSINE_SOFTMAX;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (active) {
        if (p.gran == KVCOMM_W_TOKEN) {
            const double *src = jb.partial + ((int64_t)cl * jb.S + slot) * jb.n_sel + a;
            const int64_t step = (int64_t)CL * jb.S * jb.n_sel;
#pragma unroll 4
            for (int c = cl; c < p.n_chunks; c += CL, src += step) {
                s0 += src[0];
                if (cosine) {
                    s1 += src[jb.comp_stride];
                    s2 += src[2 * jb.comp_stride];
                }
            }
        } else {  // one chunk per (layer, head): slot = chunk * S + t, CL == 1
            const int64_t i = slot * jb.n_sel + a;
            s0 = jb.partial[i];
            if (cosine) {
                s1 = jb.partial[jb.comp_stride + i];
                s2 = jb.partial[2 * jb.comp_stride + i];
            }
        }
    }
    if (CL > 1) {
        red[0][tid] = s0;
        if (cosine) {
            red[1][tid] = s1;
            red[2][tid] = s2;
        }
        __syncthreads();
        if (active && cl == 0) {
#pragma unroll 4
            for (int c = 1; c < CL; ++c) {
                s0 += red[0][c * per_lane + tid];
                if (cosine) {
                    s1 += red[1][c * per_lane + tid];
                    s2 += red[2][c * per_lane + tid];
                }
            }
        }
    }
    const bool act = active && cl == 0;
    if (act) dsh[tid] = score_of(p.rule, s0, s1, s2);   // tid = sl * n_sel + a
    __syncthreads();
    slot_softmax(p, jb, dsh + sl * jb.n_sel, esh + sl * jb.n_sel, a, slot, act);
}

// Per-segment granularity: one block per segment.  The distance kernel has left one partial per (chunk, token
// tile, anchor), n_rows = n_chunks * n_token_tiles rows of n_sel values (512 ... 768 by make_plan, fewer for small models and
// short segments, which have layers * heads chunks per tile at most).  Thread t adds
// the rows g, g + G, ... of anchor t % n_sel (g = t / n_sel, G = kSegBlock / n_sel groups: consecutive threads read
// consecutive addresses; eight interleaved chains keep as many loads in flight); the groups' sums are added in LDS, 16
// threads per anchor and then one, in a fixed order, so the result does not depend on timing.
// Latency of one block: 1024 threads instead of 256 shorten the chain of loads to a quarter (512 tokens, 8 anchors: 10.4 -> 5.8 us,
// part of it from the shorter list of partials).
__global__ __launch_bounds__(kSegBlock) void finalize_segment_kernel(const FinalParams p)
{
    constexpr int NC = 8, NF = 16;
    __shared__ double red[3][kSegBlock];
    __shared__ double fin[3][NF * KVCOMM_MAX_ANCHORS];
    __shared__ double dsh[KVCOMM_MAX_ANCHORS], esh[KVCOMM_MAX_ANCHORS];
    const FinalJob &jb = p.job[blockIdx.x];
    await_args(arg_word(&p), arg_word(&jb), arg_word(&jb.n_slots), arg_word(p.col));
    const int tid = threadIdx.x;
    if (jb.selected_out && tid < jb.n_anchors) jb.selected_out[tid] = (int32_t)((jb.sel_mask >> tid) & 1);
    if (jb.n_sel == 0) {
        if (tid < jb.n_anchors) jb.weights[tid] = 0.f;
        if (tid == 0 && jb.nearest) jb.nearest[0] = -1;
        return;
    }
    const int n_sel = jb.n_sel, G = kSegBlock / n_sel;
    const int a = tid % n_sel, g = tid / n_sel;
    const int64_t n_rows = (int64_t)p.n_chunks * jb.n_token_tiles;
    const int n_comp = p.rule == KVCOMM_RULE_COSINE_SOFTMAX ? 3 : 1;
    if (g < G) {
        for (int c = 0; c < n_comp; ++c) {
            const double *src = jb.partial + c * jb.comp_stride + a;
            double s[NC] = {};
            int64_t r = g;
            for (; r + (NC - 1) * G < n_rows; r += NC * G) {
#pragma unroll
                for (int u = 0; u < NC; ++u) s[u] += src[(r + u * G) * n_sel];
            }
#pragma unroll
            for (int u = 0; u < NC; ++u)
                if (r + u * G < n_rows) s[u] += src[(r + u * G) * n_sel];
            red[c][tid] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
        }
    }
    __syncthreads();
    if (g < NF) {   // NF * n_sel <= kSegBlock
        for (int c = 0; c < n_comp; ++c) {
            double v = 0.0;
            for (int gg = g; gg < G; gg += NF) v += red[c][gg * n_sel + a];
            fin[c][g * n_sel + a] = v;
        }
    }
    __syncthreads();
    if (tid < n_sel) {
        double tot[3] = {0.0, 0.0, 0.0};
        for (int c = 0; c < n_comp; ++c)
#pragma unroll
            for (int f = 0; f < NF; ++f) tot[c] += fin[c][f * n_sel + tid];
        dsh[tid] = score_of(p.rule, tot[0], tot[1], tot[2]);
    }
    __syncthreads();
    slot_softmax(p, jb, dsh, esh, tid, 0, tid < n_sel);
}

// Per-token granularity in one launch: a block walks ALL (layer, head) pairs of 1, 2, 4 or 8 consecutive tokens, adds up
// its wavefronts in LDS in a fixed order and finishes the softmax itself: no partial sums in memory and no second launch (5 us,
// its gap, and 3 us on the host).  A wavefront reads 64 / LPR rows at a time, the block's tokens of one or more (layer, head)
// pairs, so with 64 / LPR tokens per block every access is 1 KB long; pools of several anchor tiles share the wavefronts out.
// HBM bound where its blocks fill the chip, else bound by what one compute unit can have in flight (35 GB/s): token_shift() weighs
// that against the two-stage kernels.  us per call, two stages -> one, input sets in no cache, D = 128, 32 layers x 8 heads:
//   4 x 512 tokens, 8 anchors 180.9 -> 175.3 (cosine 189.7 -> 176.9); 512 tokens, 8 anchors 54.8 -> 48.2; 200, 12 anchors 38.0 -> 33.3;
//   130, 8 anchors 22.2 -> 18.7; 1024, 4 anchors 56.7 -> 53.4; 2 layers x 4 heads, f32, D = 64, 128 tokens, 4 anchors 12.7 -> 10.2.
// Where the model says otherwise the two stages stay: 77 tokens with 6 anchors (in one launch 15.7 -> 17.4, while 77 with one anchor and 130
// with 8 take it), and pools of many tiles (64 anchors, 1024 tokens: 651 -> 687).  Beside an attention on 160 of the 256 units the
// choice makes no difference (two-stream step of 5 agents 5.49 ms, 5.56 with two stages; on 192 units 5.48 and 5.47).
constexpr int kTokBlock = 512;

template <typename T, int LPR, int NA, bool COS>
__global__ __launch_bounds__(kTokBlock, COS ? 2 : 4) void token_weights_kernel(const DistParams p)
{
    constexpr int EPV = Elem<T>::EPV;
    constexpr int NW = kTokBlock / 64, RPW = 64 / LPR;   // wavefronts, rows that one reads at a time
    constexpr int KEEP = NA > LPR ? NA / LPR : 1;         // anchors of a lane after the sums over a row
    constexpr int NC = COS ? 3 : 1;
    __shared__ double red[NC][NW][RPW][NA];
    __shared__ double sc[RPW * KVCOMM_MAX_ANCHORS], ex[RPW * KVCOMM_MAX_ANCHORS];
    await_dist_args(p);
    const int ji = job_of_block(p, blockIdx.x);
    const DistJob &jb = p.job[ji];
    if (ji > 0) await_args(arg_word(&jb), arg_word(&jb.sel_mask));
    const int tid = threadIdx.x, bx = blockIdx.x - p.block0[ji];
    const int tpb = 1 << p.tok_shift, t0 = bx << p.tok_shift;   // tpb <= RPW
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = (tid & 63) / LPR, lir = tid % LPR;
    if (bx == 0 && jb.selected_out && tid < jb.n_anchors) jb.selected_out[tid] = (int32_t)((jb.sel_mask >> tid) & 1);
    if (jb.n_sel == 0) {   // nothing selected: all weights 0, nearest -1
        if (tid < tpb && t0 + tid < jb.S) {
            for (int c = 0; c < jb.n_anchors; ++c) jb.weights[(int64_t)(t0 + tid) * jb.n_anchors + c] = 0.f;
            if (jb.nearest) jb.nearest[t0 + tid] = -1;
        }
        return;
    }
    const int tiles = (jb.n_sel + NA - 1) / NA, width = (jb.n_sel + tiles - 1) / tiles;   // tiles <= NW
    const int phases = NW / tiles, tile = wave % tiles, phase = wave / tiles;
    const int a0 = tile * width, na = phase < phases ? min(width, jb.n_sel - a0) : 0;
    __builtin_assume(na <= NA);
    const int t = t0 + (rw & (tpb - 1));
    const int lh_step = phases * (RPW >> p.tok_shift);

    double acc[NA], ny[COS ? NA : 1], nx = 0.0;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        acc[j] = 0.0;
        if (COS) ny[j] = 0.0;
    }
    const AnchorPtrs<T, NA> anc(p, jb.a0 + a0);
    const T *seg = static_cast<const T *>(jb.seg_k) + t * jb.s_seg.token + lir * EPV;
    const int64_t arow = t * p.s_anc.token + lir * EPV;
    auto walk = [&](auto full) __attribute__((always_inline)) {   // full: every anchor of the tile exists (no branches)
        for (int lh = phase * (RPW >> p.tok_shift) + (rw >> p.tok_shift); lh < p.LH; lh += lh_step) {
            const int l = div_by(lh, p.by_H), h = lh - l * p.H;
            const u32x4 rs = load16(seg + l * jb.s_seg.layer + h * jb.s_seg.head);
            const int64_t aoff = arow + l * p.s_anc.layer + h * p.s_anc.head;
            u32x4 ra[NA];
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (decltype(full)::value || j < na) ra[j] = anc.load(j, aoff);
            float x[EPV];
            unpack<T>(rs, x);
            if (COS)
#pragma unroll
                for (int e = 0; e < EPV; ++e) nx = fma((double)x[e], (double)x[e], nx);
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (decltype(full)::value || j < na) {
                    if constexpr (COS) {
                        float y[EPV];
                        unpack<T>(ra[j], y);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) {
                            acc[j] = fma((double)x[e], (double)y[e], acc[j]);
                            ny[j] = fma((double)y[e], (double)y[e], ny[j]);
                        }
                    } else {
                        sqdiff_acc<T>(acc[j], x, ra[j]);
                    }
                }
        }
    };
    if (t < jb.S && na > 0) {
        if (na == NA)
            walk(std::true_type{});
        else
            walk(std::false_type{});
    }
    // Sums over the lanes of a row, then over the rows of the same token in the wavefront, then over the wavefronts.
    auto sum_rows = [&](double v) __attribute__((always_inline)) {
        for (int off = LPR << p.tok_shift; off < 64; off <<= 1) v += __shfl_xor(v, off);
        return v;
    };
    row_reduce_scatter<LPR, NA>(acc, lir);
    if constexpr (COS) {
        row_reduce_scatter<LPR, NA>(ny, lir);
#pragma unroll
        for (int off = LPR / 2; off >= 1; off >>= 1) nx += __shfl_xor(nx, off, LPR);
        nx = sum_rows(nx);
    }
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        const int j = anchor_of_lane<LPR, NA>(lir, k);
        const double v = sum_rows(acc[k]);
        double y = 0.0;
        if constexpr (COS) y = sum_rows(ny[k]);
        if (rw < tpb && j < na) {
            red[0][wave][rw][j] = v;
            if constexpr (COS) {
                red[1][wave][rw][j] = nx;
                red[2][wave][rw][j] = y;
            }
        }
    }
    __syncthreads();
    const int tok = tid / jb.n_sel, a = tid % jb.n_sel;   // tpb * n_sel <= kTokBlock
    const bool act = tok < tpb && t0 + tok < jb.S;
    if (act) {
        double s[3] = {0.0, 0.0, 0.0};
        const int at = a / width, aj = a - at * width;
        for (int ph = 0; ph < phases; ++ph)
#pragma unroll
            for (int c = 0; c < NC; ++c) s[c] += red[c][ph * tiles + at][tok][aj];
        sc[tid] = score_of(p.rule, s[0], s[1], s[2]);
    }
    __syncthreads();
    slot_softmax(p, jb, sc + tok * jb.n_sel, ex + tok * jb.n_sel, a, t0 + tok, act);
}

// log2 of the tokens of a token_weights_kernel block, or -1 where the two-stage kernels are taken.  A step of a block (one row of
// every anchor per wavefront and row slot) takes 0.8 us of latency (cosine: 1.7 with its arithmetic), or its bytes at the
// 35 GB/s that a compute unit reaches; two blocks share a unit (cosine: one, by its registers).  The kernel is taken where that, or
// the whole chip's time for the bytes, is at most the chip's time plus the 7 us of partial sums and second launch; of equal sizes the
// larger (longer accesses).  Pools of more than 8 anchors only up to 150 us, where that second launch still weighs: 512 tokens, 16
// anchors, 32 layers x 8 heads 98.8 -> 91.0, but 2048 tokens 343 -> 362 (16 wavefronts of 17 rows each on every unit).
// The modelled line holds to 3 % over 300 shapes: 300 tokens, 8 anchors 36.6 (two stages) and 36.8; 17 tokens, f32, 4 anchors 13.1 and 13.3.
// Two and three anchors of bf16 rows of 256 channels take 15 % more a step where the blocks leave compute units empty (128 tokens, 3 anchors 18.2 in
// two stages and 20.1, 140 tokens 19.6 and 20.4; 170 tokens 21.6 and 20.8; one anchor and four 14.2 and 20.4 either way).
// Heads that lie an odd multiple of 512 KB apart meet in the same memory channels, and the rows that a block has in flight are those of many
// heads: from 128 pairs of layer and head and four anchors on, two stages (2048 tokens, D = 128, 6 anchors: 16 layers 77.5 and 84.9, 24 118.6 and 119.5,
// 32 147 and 161; cosine, 8 anchors, 32 layers 190 and 216; f32, 1024 tokens, 8 anchors 183 and 197; but 12 layers 63.8 and 59.5, and at 32 layers
// 2000 tokens 154 and 145, 1024 77.3 and 72.5); where the pools happen to lie matters too: another run had 16 layers, 8 anchors at 99 both ways.
int token_shift(const kvcomm_model &m, const kvcomm_tensor &anchor_layout, const kvcomm_weights_job *jobs, const DistJob *dist, int n_jobs, int max_sel,
                bool cosine)
{
    if (max_sel > kAnchorTile) return -1;
    const double row = (double)m.head_dim * elem_size(m.dtype);
    const int LH = m.n_layers * m.n_kv_heads, rpw = 1024 / (int)row, nw = kTokBlock / 64;   // rows of a wavefront, wavefronts
    if (max_sel >= 4 && LH >= 128 && anchor_layout.stride_head * elem_size(m.dtype) % (1 << 20) == 1 << 19) return -1;
    const bool few_wide = m.dtype == KVCOMM_BF16 && m.head_dim == 256 && !cosine && (max_sel == 2 || max_sel == 3);
    double bytes = 0.0;
    for (int j = 0; j < n_jobs; ++j) bytes += (double)LH * row * (dist[j].n_sel + 1) * jobs[j].seg_len;
    const double chip_us = bytes / 6.4e6;
    if (max_sel > 8 && chip_us > 150.0) return -1;
    const int tile = cosine ? kCosTile : kAnchorTile;
    const int tiles = std::max(1, (max_sel + tile - 1) / tile), width = (max_sel + tiles - 1) / tiles;
    int best = -1;
    double best_us = chip_us + 7.0;
    for (int shift = 0; 1 << shift <= rpw; ++shift) {
        int64_t blocks = 0;
        for (int j = 0; j < n_jobs; ++j) blocks += ((int64_t)jobs[j].seg_len + (1 << shift) - 1) >> shift;
        if (blocks * kTokBlock >= (int64_t)1 << 32) continue;   // more threads than a launch holds
        const int per_cu = cosine ? 1 : blocks > 256 ? 2 : 1, lh_step = (nw / tiles) * (rpw >> shift);
        const double rounds = (double)((blocks + 256 * per_cu - 1) / (256 * per_cu));
        const double step_us = (few_wide && blocks <= 150 ? 1.15 : 1.0) * std::max(cosine ? 1.7 : 0.8, per_cu * nw * 1024.0 * (width + 1) / 35e3);
        const double us = std::max(chip_us, rounds * (2.0 + step_us * ((LH + lh_step - 1) / lh_step)));
        if (us <= best_us) {
            best_us = us;
            best = shift;
        }
    }
    return best;
}

template <typename T, int LPR>
int launch_tokens(const DistParams &p, int n_blocks, int max_sel, bool cosine, hipStream_t stream)
{
    const dim3 grid(n_blocks), block(kTokBlock);
    if (cosine)
        return launch(token_weights_kernel<T, LPR, kCosTile, true>, grid, block, 0, stream, p);
    return launch(max_sel <= 4 ? token_weights_kernel<T, LPR, 4, false> : max_sel <= 8 ? token_weights_kernel<T, LPR, 8, false>
                                                                           : token_weights_kernel<T, LPR, kAnchorTile, false>,
                  grid, block, 0, stream, p);
}

template <typename T, int LPR>
int launch_dist(const DistParams &p, int n_blocks, int max_sel, int min_sel, bool cosine, hipStream_t stream)
{
    const int na = cosine ? kCosTile : max_sel <= 4 ? 4 : max_sel <= 8 ? 8 : kAnchorTile;
    if (p.fused)
        return launch(na == 4 ? dist_row_softmax_kernel<T, LPR, 4> : na == 8 ? dist_row_softmax_kernel<T, LPR, 8> : dist_row_softmax_kernel<T, LPR, kAnchorTile>,
                      dim3(n_blocks), dim3(kBlock), 0, stream, p);
    DistParams q = p;
    q.n_blocks = n_blocks;
    const int a_tiles = (max_sel + na - 1) / na;
    const bool same_tiles = cosine || (min_sel + na - 1) / na == a_tiles;
    // Tiles of equal width (17 anchors: 9 + 8, not 16 + 1): with a narrow last tile every other block would have next to
    // nothing to do, and so would the compute units they land on (17 anchors, 1024 tokens, per-(layer, head, token) weights,
    // f32 D = 256: 341 -> 234 us; per-token weights, bf16 D = 128, 32 layers: 233 -> 195; 9 anchors, cosine: 285 -> 194).
    q.tile_anchors = same_tiles ? (max_sel + a_tiles - 1) / a_tiles : na;
    q.group_pairs = n_blocks;
    if (same_tiles && a_tiles > 1) {   // at most kMaxGroups groups
        q.group_pairs = kGroupPairs;
        while ((n_blocks - 1) / q.group_pairs >= kMaxGroups) q.group_pairs *= 2;
    }
    const dim3 grid((unsigned)q.group_pairs, (unsigned)a_tiles, (unsigned)((n_blocks + q.group_pairs - 1) / q.group_pairs));
    return launch(cosine ? cos_partial_kernel<T, LPR> : na == 4 ? dist_partial_kernel<T, LPR, 4> : na == 8 ? dist_partial_kernel<T, LPR, 8>
                                                                                              : dist_partial_kernel<T, LPR, kAnchorTile>,
                  grid, dim3(kBlock), 0, stream, q);
}

int check_rule(int rule)
{
    return (rule == KVCOMM_RULE_L2_SOFTMAX || rule == KVCOMM_RULE_NEAREST || rule == KVCOMM_RULE_COSINE_SOFTMAX)
               ? KVCOMM_OK
               : KVCOMM_EINVAL;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Bytes of segment j's partial sums for a plan.
size_t job_partial_bytes(const DistPlan &pl, int32_t seg_len, int32_t n_anchors, int rule)
{
    const size_t n_comp = rule == KVCOMM_RULE_COSINE_SOFTMAX ? 3 : 1;
    return sizeof(double) * n_comp * (size_t)pl.n_chunks * seg_len * n_anchors;
}

}  // namespace

extern "C" size_t kvcomm_weight_slots(const kvcomm_model *model, int32_t seg_len, int32_t gran)
{
    if (check_model(model) || check_gran(gran) || seg_len <= 0) return 0;
    if (gran == KVCOMM_W_TOKEN) return (size_t)seg_len;
    if (gran == KVCOMM_W_SEGMENT) return 1;
    return (size_t)model->n_layers * model->n_kv_heads * seg_len;
}

extern "C" size_t kvcomm_anchor_weights_batch_workspace(const kvcomm_model *model, int32_t gran, int32_t rule,
                                                        const int32_t *seg_lens, const int32_t *n_anchors,
                                                        int32_t n_jobs)
{
    if (check_model(model) || check_gran(gran) || check_rule(rule) || !seg_lens || !n_anchors || n_jobs <= 0 ||
        n_jobs > KVCOMM_MAX_BATCH)
        return 0;
    for (int j = 0; j < n_jobs; ++j)
        if (seg_lens[j] <= 0 || n_anchors[j] <= 0 || n_anchors[j] > KVCOMM_MAX_ANCHORS) return 0;
    const DistPlan pl = make_plan(model, seg_lens, n_jobs, gran);
    size_t total = 0;
    for (int j = 0; j < n_jobs; ++j) total += align256(job_partial_bytes(pl, seg_lens[j], n_anchors[j], rule));
    return total;
}

extern "C" size_t kvcomm_anchor_weights_rule_workspace(const kvcomm_model *model, int32_t seg_len, int32_t n_anchors,
                                                       int32_t gran, int32_t rule)
{
    if (check_model(model) || check_gran(gran) || check_rule(rule) || seg_len <= 0 || n_anchors <= 0 ||
        n_anchors > KVCOMM_MAX_ANCHORS)
        return 0;
    const DistPlan pl = make_plan(model, &seg_len, 1, gran);
    return job_partial_bytes(pl, seg_len, n_anchors, rule);
}

extern "C" size_t kvcomm_anchor_weights_workspace(const kvcomm_model *model, int32_t seg_len, int32_t n_anchors,
                                                  int32_t gran)
{
    return kvcomm_anchor_weights_rule_workspace(model, seg_len, n_anchors, gran, KVCOMM_RULE_L2_SOFTMAX);
}

extern "C" int kvcomm_anchor_weights_batch(const kvcomm_model *model, int32_t gran, int32_t rule, float temperature,
                                           kvcomm_tensor anchor_layout, const kvcomm_weights_job *jobs,
                                           int32_t n_jobs, void *workspace, size_t workspace_bytes, void *stream)
{
    int st = check_model(model);
    if (st) return st;
    if ((st = check_gran(gran)) || (st = check_rule(rule))) return st;
    if (!jobs || n_jobs <= 0) return KVCOMM_EINVAL;
    if (n_jobs > KVCOMM_MAX_BATCH) return KVCOMM_EUNSUPPORTED;
    if (!(temperature > 0.f)) return KVCOMM_EINVAL;  // also rejects NaN
    const int dt = model->dtype;
    if ((st = check_tensor(anchor_layout, dt, false))) return st;
    int32_t seg_lens[KVCOMM_MAX_BATCH];
    for (int j = 0; j < n_jobs; ++j) {
        const kvcomm_weights_job &jd = jobs[j];
        if (jd.seg_len <= 0 || jd.n_anchors <= 0) return KVCOMM_EINVAL;
        if (jd.n_anchors > KVCOMM_MAX_ANCHORS) return KVCOMM_EUNSUPPORTED;
        if ((st = check_tensor(jd.seg_base_k, dt, true))) return st;
        if (!jd.anchor_base_k || !jd.anchor_len || !jd.weights_out) return KVCOMM_EINVAL;
        seg_lens[j] = jd.seg_len;
    }

    const DistPlan pl = make_plan(model, seg_lens, n_jobs, gran);
    const bool cosine = rule == KVCOMM_RULE_COSINE_SOFTMAX;
    DistParams dp{};
    FinalParams fp{};
    int n_sel_total = 0, max_sel = 0, min_sel = KVCOMM_MAX_ANCHORS;
    size_t need = 0;
    for (int j = 0; j < n_jobs; ++j) {
        const kvcomm_weights_job &jd = jobs[j];
        DistJob &dj = dp.job[j];
        FinalJob &fj = fp.job[j];
        dj.a0 = fj.a0 = (int16_t)n_sel_total;
        int n_sel = 0;
        for (int a = 0; a < jd.n_anchors; ++a) {
            if (jd.anchor_len[a] < 0) return KVCOMM_EINVAL;
            if (jd.anchor_len[a] < jd.seg_len) continue;
            if (!jd.anchor_base_k[a] || !aligned16(jd.anchor_base_k[a])) return KVCOMM_EINVAL;
            if (n_sel_total + n_sel >= KVCOMM_MAX_ANCHORS) return KVCOMM_EUNSUPPORTED;  // over all segments of the launch
            fp.col[n_sel_total + n_sel] = dp.col[n_sel_total + n_sel] = (uint8_t)a;
            fj.sel_mask |= (uint64_t)1 << a;
            dp.anc[n_sel_total + n_sel] = jd.anchor_base_k[a];
            ++n_sel;
        }
        dj.n_sel = fj.n_sel = (int16_t)n_sel;
        n_sel_total += n_sel;
        max_sel = n_sel > max_sel ? n_sel : max_sel;
        min_sel = n_sel < min_sel ? n_sel : min_sel;
        need += n_jobs == 1 ? job_partial_bytes(pl, jd.seg_len, jd.n_anchors, rule)
                            : align256(job_partial_bytes(pl, jd.seg_len, jd.n_anchors, rule));
    }
    if (!workspace || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return KVCOMM_EWORKSPACE;

    hipStream_t s = static_cast<hipStream_t>(stream);
    dp.s_anc = strides_of(anchor_layout);
    dp.H = model->n_kv_heads;
    dp.by_H = make_divisor((uint32_t)dp.H);
    dp.LH = model->n_layers * model->n_kv_heads;
    dp.lh_per_block = pl.lh_per_block;
    dp.n_jobs = n_jobs;
    // One softmax per (layer, head, token): a row's distances are complete inside the lanes that read the
    // row, so the distance kernel writes the weights itself (no partial sums, no second kernel) as long as
    // every segment's selected anchors fit one anchor tile.
    const bool fused = gran == KVCOMM_W_LAYER_HEAD_TOKEN && !cosine && min_sel >= 1 && max_sel <= kAnchorTile;
    // (one (layer, head) pair per block, as in the two-stage form: with runs of several pairs per block the
    // softmax of one pair delays the loads of the next, measured 6 % slower)
    dp.fused = fused ? 1 : 0;
    dp.per_segment = gran == KVCOMM_W_SEGMENT ? 1 : 0;
    dp.rule = rule;
    dp.tau = (double)temperature;
    fp.n_chunks = pl.n_chunks;
    fp.gran = gran;
    fp.rule = rule;
    fp.n_jobs = n_jobs;
    fp.tau = (double)temperature;
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    int64_t dist_blocks = 0, final_blocks = 0;
    for (int j = 0; j < n_jobs; ++j) {
        const kvcomm_weights_job &jd = jobs[j];
        DistJob &dj = dp.job[j];
        FinalJob &fj = fp.job[j];
        dj.seg_k = jd.seg_base_k.ptr;
        dj.s_seg = strides_of(jd.seg_base_k);
        dj.partial = reinterpret_cast<double *>(ws);
        ws += align256(job_partial_bytes(pl, jd.seg_len, jd.n_anchors, rule));
        dj.comp_stride = (int64_t)pl.n_chunks * jd.seg_len * dj.n_sel;  // <= a third of the segment's partials
        dj.S = jd.seg_len;
        dj.n_token_tiles = (jd.seg_len + pl.rpb - 1) / pl.rpb;
        dj.by_tiles = make_divisor((uint32_t)dj.n_token_tiles);
        dp.block0[j] = (int32_t)dist_blocks;
        dist_blocks += (int64_t)pl.n_chunks * dj.n_token_tiles;

        dj.weights = jd.weights_out;
        dj.nearest = jd.nearest_out;
        dj.selected_out = jd.selected_out;
        dj.sel_mask = fj.sel_mask;
        dj.n_anchors = jd.n_anchors;
        fj.partial = dj.partial;
        fj.weights = jd.weights_out;
        fj.nearest = jd.nearest_out;
        fj.selected_out = jd.selected_out;
        fj.comp_stride = dj.comp_stride;
        fj.n_token_tiles = dj.n_token_tiles;
        fj.S = jd.seg_len;
        fj.n_slots = (int32_t)kvcomm_weight_slots(model, jd.seg_len, gran);
        fj.n_anchors = jd.n_anchors;
        int cl = 1;
        if (gran == KVCOMM_W_TOKEN && dj.n_sel > 0) {
            const int slots = (kFinalRun + dj.n_sel - 1) / dj.n_sel;   // of a run
            cl = kFinalBlock / (slots * dj.n_sel);
            cl = std::min(cl, std::min(pl.n_chunks, std::max(kFinalLanes, pl.n_chunks / 8)));
        }
        fj.chunk_lanes = cl;
        const int spb = dj.n_sel > 0 ? kFinalBlock / (cl * dj.n_sel) : kFinalBlock;
        fp.block0[j] = (int32_t)final_blocks;
        final_blocks += (fj.n_slots + spb - 1) / spb;
    }
    if (dist_blocks > 0x7fffffff || final_blocks > 0x7fffffff) return KVCOMM_EUNSUPPORTED;

    const int shift = gran == KVCOMM_W_TOKEN ? token_shift(*model, anchor_layout, jobs, dp.job, n_jobs, max_sel, cosine) : -1;
    if (shift >= 0) {
        dp.tok_shift = shift;
        int64_t blocks = 0;
        for (int j = 0; j < n_jobs; ++j) {
            dp.block0[j] = (int32_t)blocks;
            blocks += ((int64_t)jobs[j].seg_len + (1 << shift) - 1) >> shift;
        }
        st = KVCOMM_EUNSUPPORTED;
        const int nb = (int)blocks;
        if (dt == KVCOMM_BF16) {
            switch (pl.lpr) {
                case 8: return launch_tokens<bf16_t, 8>(dp, nb, max_sel, cosine, s);
                case 16: return launch_tokens<bf16_t, 16>(dp, nb, max_sel, cosine, s);
                case 32: return launch_tokens<bf16_t, 32>(dp, nb, max_sel, cosine, s);
            }
        } else {
            switch (pl.lpr) {
                case 16: return launch_tokens<float, 16>(dp, nb, max_sel, cosine, s);
                case 32: return launch_tokens<float, 32>(dp, nb, max_sel, cosine, s);
                case 64: return launch_tokens<float, 64>(dp, nb, max_sel, cosine, s);
            }
        }
        return st;
    }

    if (max_sel > 0) {
        st = KVCOMM_EUNSUPPORTED;
        const int nb = (int)dist_blocks;
        if (dt == KVCOMM_BF16) {
            switch (pl.lpr) {
                case 8: st = launch_dist<bf16_t, 8>(dp, nb, max_sel, min_sel, cosine, s); break;
                case 16: st = launch_dist<bf16_t, 16>(dp, nb, max_sel, min_sel, cosine, s); break;
                case 32: st = launch_dist<bf16_t, 32>(dp, nb, max_sel, min_sel, cosine, s); break;
            }
        } else {
            switch (pl.lpr) {
                case 16: st = launch_dist<float, 16>(dp, nb, max_sel, min_sel, cosine, s); break;
                case 32: st = launch_dist<float, 32>(dp, nb, max_sel, min_sel, cosine, s); break;
                case 64: st = launch_dist<float, 64>(dp, nb, max_sel, min_sel, cosine, s); break;
            }
        }
        if (st) return st;
    }
    if (fused) return KVCOMM_OK;
    if (gran == KVCOMM_W_SEGMENT)
        return launch(finalize_segment_kernel, dim3(n_jobs), dim3(kSegBlock), 0, s, fp);
    return launch(finalize_kernel, dim3((unsigned)final_blocks), dim3(kFinalBlock), 0, s, fp);
}

extern "C" int kvcomm_anchor_weights_rule(const kvcomm_model *model, int32_t gran, int32_t rule, float temperature,
                                          kvcomm_tensor seg_base_k, int32_t seg_len,
                                          const void *const *anchor_base_k, kvcomm_tensor anchor_layout,
                                          const int32_t *anchor_len, int32_t n_anchors, float *weights_out,
                                          int32_t *nearest_out, int32_t *selected_out, void *workspace,
                                          size_t workspace_bytes, void *stream)
{
    kvcomm_weights_job job{};
    job.seg_base_k = seg_base_k;
    job.seg_len = seg_len;
    job.anchor_base_k = anchor_base_k;
    job.anchor_len = anchor_len;
    job.n_anchors = n_anchors;
    job.weights_out = weights_out;
    job.nearest_out = nearest_out;
    job.selected_out = selected_out;
    return kvcomm_anchor_weights_batch(model, gran, rule, temperature, anchor_layout, &job, 1, workspace,
                                       workspace_bytes, stream);
}

extern "C" int kvcomm_anchor_weights(const kvcomm_model *model, int32_t gran, float temperature,
                                     kvcomm_tensor seg_base_k, int32_t seg_len, const void *const *anchor_base_k,
                                     kvcomm_tensor anchor_layout, const int32_t *anchor_len, int32_t n_anchors,
                                     float *weights_out, int32_t *nearest_out, int32_t *selected_out, void *workspace,
                                     size_t workspace_bytes, void *stream)
{
    return kvcomm_anchor_weights_rule(model, gran, KVCOMM_RULE_L2_SOFTMAX, temperature, seg_base_k, seg_len,
                                      anchor_base_k, anchor_layout, anchor_len, n_anchors, weights_out, nearest_out,
                                      selected_out, workspace, workspace_bytes, stream);
}

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, looked up once per GPU

// Address of the current device's copy of `scratch` (every GPU holds its own copy at its own address).
int static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KVCOMM_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return KVCOMM_EHIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return KVCOMM_OK;
}

}  // namespace

extern "C" size_t kvcomm_anchor_weights_static_capacity(void) { return KVCOMM_STATIC_SCRATCH_BYTES; }

extern "C" int kvcomm_anchor_weights_static(const kvcomm_model *model, int32_t gran, float temperature,
                                            kvcomm_tensor seg_base_k, int32_t seg_len,
                                            const void *const *anchor_base_k, kvcomm_tensor anchor_layout,
                                            const int32_t *anchor_len, int32_t n_anchors, float *weights_out,
                                            int32_t *nearest_out, int32_t *selected_out, void *stream)
{
    // Size first: a request that does not fit is refused before anything else is looked at.
    int st = check_model(model);
    if (st) return st;
    if ((st = check_gran(gran))) return st;
    if (seg_len <= 0 || n_anchors <= 0) return KVCOMM_EINVAL;
    if (n_anchors > KVCOMM_MAX_ANCHORS) return KVCOMM_EUNSUPPORTED;
    const size_t need = kvcomm_anchor_weights_workspace(model, seg_len, n_anchors, gran);
    if (need > KVCOMM_STATIC_SCRATCH_BYTES) return KVCOMM_EWORKSPACE;
    void *ws = nullptr;
    if ((st = static_scratch(&ws))) return st;
    // Nothing in the array has to start at zero: the distance kernel writes every partial sum that the
    // finalize kernel reads, whatever an earlier call left behind.
    return kvcomm_anchor_weights(model, gran, temperature, seg_base_k, seg_len, anchor_base_k, anchor_layout,
                                 anchor_len, n_anchors, weights_out, nearest_out, selected_out, ws,
                                 KVCOMM_STATIC_SCRATCH_BYTES, stream);
}
