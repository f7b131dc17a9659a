// kvcomm_align_kv: positional alignment fused with the offset approximation
// (Eq. "ph_update" / Eq. "pf_update" of the paper, keys first rotated to their new
// position as Sec. 3.1 "Positional Alignment" requires).
//
// The kernel is a single streaming pass bounded by HBM bandwidth: per cache row
// (layer, kv head, token) it reads the base K and V rows and one dK and one dV row per
// selected anchor, and writes one K and one V row: 2*(A+2) rows of D elements.
//
// Work split.  A row is covered by LPR = D / (2 * EPV) lanes (EPV = elements per 16-byte
// vector).  Lane r of a row owns channels [r*EPV, r*EPV+EPV) of the first half and the
// same channels of the second half, i.e. both members of each RoPE pair (i, i + D/2), so
// the rotation needs no cross-lane traffic and the kernel may run in place.  A block of
// 256 threads owns a tile of 256/LPR consecutive tokens of one (layer, head) and of ONE of
// the two tensors (blockIdx.y even: keys, odd: values): the two streams are independent, and
// splitting them halves the registers per lane.  Every access to a tensor is a run of whole 128-byte lines; deviations and outputs are marked
// non-temporal (they are not read again soon: 466 us per launch of 4 x 512 tokens with 8 anchors, 500 us with plain
// stores).  The base rows are plain loads: anchor matching has just read the base keys, and a shared segment's base
// cache serves the next agent as well (matching and update of a placeholder of 512 and a prefix segment of 173 tokens,
// 8 anchors: 205 us, 212 us with non-temporal loads; no difference where nothing is in the last-level cache).  Per-token anchor weights and the cos/sin tables load once per block (LDS).
// cos/sin: the angle delta * theta^(-2i/D) is formed in double from a host-computed frequency table (kernel argument), reduced
// to the nearest quarter turn and put through short series in double, and rounded to fp32 (rope_cos_sin()).
#include "align_common.h"

namespace {

using namespace kvc;

constexpr int kBlock = kAlignBlock;
constexpr int kComputeUnits = 256;

struct AlignKvJob : AlignJob {
    uint64_t sel_mask;     // bit a = anchor a of the segment is selected
    divisor_t by_pitch;    // of w_pitch
};

struct AlignParams {
    AlignHead head;
    AlignKvJob job[KVCOMM_MAX_BATCH];
    int32_t tab_delta[kMaxTab];                 // position delta of each rotation table
    const void *anc[2][KVCOMM_MAX_ANCHORS];     // [0] dK, [1] dV of the selected anchors of all segments
    alignas(4) uint8_t tab[KVCOMM_MAX_ANCHORS];            // its rotation table (index among the segment's tables) + 1, 0 = identity
    double inv_freq[kMaxHalf];                  // theta^(-2i/D), i < D/2
};
static_assert(sizeof(AlignParams) <= 4096, "kernel arguments are limited to 4 KB");

// Two anchors' rows (four 16-byte loads per lane) are requested together, the first two under the block's set-up.  What bounds the kernel is
// HBM, and past about 64 KB in flight per compute unit more requests cost: pages are opened and closed out of order.  So the
// launch reserves LDS that keeps the number of blocks per compute unit at what measured best (lds_reserve()).
// SMALL (few_rows()): what bounds the launch is the latency of a block, one group of anchors behind the other.  Four are requested together
// (all segments have as many), the set-up's own inputs before them, and the rows unconditionally (lanes behind the segment re-read its last
// row): only then does the compiler wait for the set-up's loads alone while the rows stay in flight.  (Large launches gain nothing
// from that: their other blocks fill the wait, and it moved them by -5 ... +5 %.)
template <typename T, int LPR, bool SMALL>
__global__ __launch_bounds__(kBlock, SMALL ? 3 : 4) void align_kernel(const AlignParams p)
{
    constexpr int INFLIGHT = SMALL ? 4 : 2;
    constexpr int EPV = Elem<T>::EPV;
    constexpr int HALF = LPR * EPV;  // D / 2
    constexpr int RPB = kBlock / LPR;

    // Block order: (layer, head) chunk, then segment, then token tile, so that the blocks in flight
    // write neighbouring slices of the same cache rows when the segments of a launch are adjacent.
    const int which = blockIdx.y & 1;      // 0 = keys (rotated), 1 = values
    const AlignHead &hd = p.head;
    await_args(arg_word(&hd), arg_word(hd.tile0), arg_word(&p.job[0]), arg_word(&p.job[0].s_base[1]), arg_word(&p.job[0].S), arg_word(p.anc[which]),
               arg_word(p.tab), arg_word(p.tab_delta));
    const int q = div_by(blockIdx.x, hd.by_tiles);
    const int r = blockIdx.x - q * hd.tiles_total;
    const int lh = (blockIdx.y >> 1) * hd.lh_range + q;
    if (lh >= hd.LH) return;   // the whole block: the last range of pairs is not full
    const int ji = job_of_tile(p, r);
    const AlignKvJob &jb = p.job[ji];
    if (ji > 0) await_args(arg_word(&jb), arg_word(&jb.s_base[1]), arg_word(&jb.s_out[1]), arg_word(&jb.S));
    const int n_sel = jb.n_sel, a0 = jb.a0;

    extern __shared__ __align__(16) unsigned char smem_raw[];
    float2 *cs = reinterpret_cast<float2 *>(smem_raw);                          // [n_tab][HALF] (cos, sin)
    float *w_lds = reinterpret_cast<float *>(smem_raw) + 2 * jb.n_tab * HALF;   // [RPB or 1][n_sel]

    const int tid = threadIdx.x;
    const int row = tid / LPR;
    const int lir = tid % LPR;
    const int tile = r - hd.tile0[ji];
    const bool is_k = which == 0;
    const int t = tile * RPB + row;
    const bool valid = t < jb.S;
    const T *bp = static_cast<const T *>(jb.base[which]);
    T *op = static_cast<T *>(jb.out[which]);
    const Strides sb = jb.s_base[which], so = jb.s_out[which];
    const int64_t col0 = (int64_t)lir * EPV;

    // What the block's set-up reads, its weight rows (as they are, unselected anchors included), is requested first, then the rows of
    // its first (layer, head) pair: they arrive under the rotation tables and the barrier.
    const uint64_t sel = jb.sel_mask;
    const int n_w = sel == 0 ? 0 : (hd.gran == KVCOMM_W_SEGMENT ? 1 : min(RPB, jb.S - tile * RPB)) * jb.w_pitch;
    const float *wsrc = jb.weights;
    if (hd.gran != KVCOMM_W_SEGMENT)
        wsrc += ((int64_t)(hd.gran == KVCOMM_W_LAYER_HEAD_TOKEN ? lh : 0) * jb.S + tile * RPB) * jb.w_pitch;
    constexpr int W = !SMALL ? 1 : RPB / 4 < 4 ? RPB / 4 : 4;   // n_w <= RPB * 64 = RPB / 4 weights of every thread
    float w_first[W] = {};
#pragma unroll
    for (int u = 0; u < W; ++u)
        if (tid + u * kBlock < n_w) w_first[u] = wsrc[tid + u * kBlock];
    double freq = 0.0;
    int delta = 0;
    if (SMALL && is_k && tid < jb.n_tab * HALF) {
        freq = p.inv_freq[tid % HALF];
        delta = p.tab_delta[jb.t0 + tid / HALF];
    }
    auto keep_weight = [&](int idx, float w) __attribute__((always_inline)) {
        const int r = div_by(idx, jb.by_pitch), c = idx - r * jb.w_pitch;
        if ((sel >> c) & 1) w_lds[r * n_sel + __popcll(sel & (((uint64_t)1 << c) - 1))] = w;
    };

    const int l = div_by(lh, hd.by_H), h = lh - l * hd.H;
    const int tr = SMALL ? min(t, jb.S - 1) : t;
    const T *xp = bp + l * sb.layer + h * sb.head + tr * sb.token + col0;
    const int64_t aoff = l * hd.s_anc.layer + h * hd.s_anc.head + tr * hd.s_anc.token + col0;
    u32x4 rlo, rhi, rows[INFLIGHT][2];
    auto request_group = [&](int a) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < INFLIGHT; ++u) {
            const T *d = static_cast<const T *>(p.anc[which][a0 + a + u]) + aoff;
            rows[u][0] = load16_stream(d);
            rows[u][1] = load16_stream(d + HALF);
        }
    };
    if (SMALL || valid) {
        rlo = load16(xp);   // plain: see the header
        rhi = load16(xp + HALF);
        if (SMALL || n_sel >= INFLIGHT) request_group(0);
    }

    if (is_k) {
        if (SMALL && tid < jb.n_tab * HALF) {
            asm volatile("" : "+v"(delta));   // (else its conversion, and the wait for it, moves up to its load)
            cs[tid] = rope_cos_sin(delta, freq);
        }
        for (int idx = SMALL ? tid + kBlock : tid; idx < jb.n_tab * HALF; idx += kBlock) {
            const int r = idx / HALF, i = idx % HALF;
            cs[idx] = rope_cos_sin(p.tab_delta[jb.t0 + r], p.inv_freq[i]);
        }
    }
#pragma unroll
    for (int u = 0; u < W; ++u)
        if (tid + u * kBlock < n_w) keep_weight(tid + u * kBlock, w_first[u]);
    for (int idx = tid + W * kBlock; idx < n_w; idx += kBlock) keep_weight(idx, wsrc[idx]);
    __syncthreads();
    if (!valid) return;

    const bool rot_base = is_k && jb.base_tab != 0;
    float bc[EPV], bs[EPV];
    if (rot_base) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float2 v = cs[(jb.base_tab - 1) * HALF + lir * EPV + e];
            bc[e] = v.x;
            bs[e] = v.y;
        }
    }

    const float *wrow = w_lds + (hd.gran == KVCOMM_W_SEGMENT ? 0 : row * n_sel);

    float lo[EPV], hi[EPV];
    unpack<T>(rlo, lo);
    unpack<T>(rhi, hi);
    if (rot_base) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float a = lo[e], b = hi[e];
            lo[e] = a * bc[e] - b * bs[e];
            hi[e] = b * bc[e] + a * bs[e];
        }
    }

    auto accumulate = [&](int a, const u32x4 &rdlo, const u32x4 &rdhi) {
        const float w = wrow[a];
        float dlo[EPV], dhi[EPV];
        unpack<T>(rdlo, dlo);
        unpack<T>(rdhi, dhi);
        const int tb = is_k ? arg_byte(p.tab, a0 + a) : 0;
        if (tb) {
            const float2 *tcs = cs + (tb - 1) * HALF + lir * EPV;
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                const float2 v = tcs[e];
                const float x = dlo[e], y = dhi[e];
                dlo[e] = x * v.x - y * v.y;
                dhi[e] = y * v.x + x * v.y;
            }
        }
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            lo[e] += w * dlo[e];
            hi[e] += w * dhi[e];
        }
    };

    int a = 0;
    while (a + INFLIGHT <= n_sel) {
#pragma unroll
        for (int u = 0; u < INFLIGHT; ++u) accumulate(a + u, rows[u][0], rows[u][1]);
        a += INFLIGHT;
        if (a + INFLIGHT <= n_sel) request_group(a);
    }
    if (SMALL && a + 2 <= n_sel) {
        const T *d0 = static_cast<const T *>(p.anc[which][a0 + a]) + aoff, *d1 = static_cast<const T *>(p.anc[which][a0 + a + 1]) + aoff;
        const u32x4 r[4] = {load16_stream(d0), load16_stream(d0 + HALF), load16_stream(d1), load16_stream(d1 + HALF)};
        accumulate(a, r[0], r[1]);
        accumulate(a + 1, r[2], r[3]);
        a += 2;
    }
    if (a < n_sel) {
        const T *d = static_cast<const T *>(p.anc[which][a0 + a]) + aoff;
        accumulate(a, load16_stream(d), load16_stream(d + HALF));
    }

    T *yp = op + l * so.layer + h * so.head + t * so.token + col0;
    store16_stream(yp, pack<T>(lo));
    store16_stream(yp + HALF, pack<T>(hi));
}

// LDS that a launch asks for beyond its tables, so that two or three blocks share a compute unit instead of the five that the
// registers allow (160 KB: three do not fit at 54 KB, four not at 40.5).  A block moves 8 KB per tensor row set, so `bytes` is the
// whole launch.  us of the update alone with five / three / two blocks per unit, inputs in no cache (32 layers x 8 heads, bf16, D = 128 unless said):
//   up to 0.45 GB the launch is too short to care, and wants every request early: 256 tokens, 8 anchors 54.4 / 58.1 / 58.1; 400, 4 anchors
//     48.6 / 50.0 / 55.3; 600, 3 anchors 58.7 / 63.7 / 74.2.  To 0.75 GB five and three are even (by 2.5 % either way: 512, 8 anchors
//     106.3 / 108.2 / 107.6; 530, 8 anchors 107.9 / 105.3 / 110.2), then three are better: 900, 5 anchors 139.2 / 131.2 / 145.9;
//   two blocks from six anchors and 0.95 GB on where the heads of a pool lie a multiple of 16 KB apart.  Below, three: 685 tokens, 8 anchors
//     (0.90 GB) 138.8 / 134.9 / 143.3; 512 + 173, 8 anchors 139.3 / 138.1 / 143.3; 900, 6 anchors (0.94 GB) 160.2 / 150.9 / 156.7.  Above: 768, 8 anchors
//     168.2 / 163.2 / 158.9; 2 x 512, 8 anchors 239 / 233 / 213; 4 x 512, 6 anchors 388 / 367 / 347, 8: 492 / 465 / 425; f32, 1024, 8 anchors
//     474 / 452 / 419.  Pools of less than six never: 2048, 4 anchors 273 / 260 / 271; 1800, 5 anchors 278 / 257 / 285;
//   heads any other distance apart: two for 16 anchors and more (2 x 1024 871 / 840 / 786, 80 layers, 2048 tokens 2154 / 2054 / 1976), and for eight and more
//     from 1.8 GB on or with rows of 512 bytes and more; else three: 1000 tokens, 7 anchors 200.3 / 189.0 / 199.1; 600, 12 anchors 175.0 / 167.8 /
//     171.6; and three / two: 1000, 9 anchors 232 / 242; 4 x 500, 6 anchors 346 / 353; 3 x 300, 8 anchors 193 / 201; 80 layers of 300, 8 anchors 156 / 164
//     (at worst, of 204 shapes: 1700, 8 anchors, 378 / 356 / 364);
//   bf16 rows of 64 channels (half a line per lane group) hardly gain from two: 2048, 8 anchors 240 / 239 / 257, 1024, 16 anchors 222 / 217 / 216.
// (Four anchors in flight at three blocks, which pools of eight took before, and two at four for smaller ones: 4 x 512 tokens, 8 anchors
// 445, 2 x 1024 tokens, 16 anchors 840, f32 490, 80 layers 2182; 2 anchors 179, now 172.)
// A launch that has only `units` of the chip's compute units (kvcomm_align_kv_batch_beside) must keep as many requests in flight on fewer
// of them.  ms per two-stream step beside an attention of the other units, two / three / four / five blocks per unit (config: 5 agents of 4 x 512
// tokens, 8 anchors, 32 layers; and 4 agents of 4 x 2048 tokens, 16 anchors, 80 layers), one box each:
//   112 units 6.16 / 6.47 / 6.51 / 6.46 and 82.3 / 83.0 / 83.7 / 84.2;  104 units 5.85 / 5.66 / 5.91 / 5.94 and 79.4 / 77.5 / 78.8 / 78.3;
//    96 units 5.86 / 5.54 / 5.95 / 5.94 and 79.1 / 76.1 / 77.0 / 77.1;   88 units 6.39 / 6.13 / 5.93 / 5.83 and 84.1 / 82.7 / 81.7 / 82.0;
//    64 units 6.29 / 6.09 / 5.83 / 5.73 and 82.8 / 79.6 / 80.7 / 80.3.
size_t lds_reserve(const AlignParams &p, int64_t n_blocks, int lpr, int es, int units)
{
    constexpr size_t kThreeBlocks = 81 << 9, kTwoBlocks = 54 << 10;
    double anchors = 0.0;   // of a block, on average
    for (int j = 0; j < p.head.n_jobs; ++j) anchors += (double)p.job[j].n_token_tiles * p.job[j].n_sel / p.head.tiles_total;
    const double bytes = 2.0 * (double)n_blocks * 32 * kBlock * (anchors + 2.0);
    if (bytes < 0.45e9 || units < 92) return 0;
    // heads of the pool a multiple of 16 KB apart; rows of 512 bytes and more
    const bool even = p.head.s_anc.head * es % 16384 == 0, wide = lpr > 8;
    const bool two = lpr > 4 && bytes >= 0.95e9 && anchors >= 6.0 && (even || anchors >= 16.0 || (anchors >= 8.0 && (wide || bytes >= 1.8e9)));
    return units >= 108 && two ? kTwoBlocks : kThreeBlocks;
}

// Four anchors in flight (SMALL): pools of four and more (in every segment) whose rows are at most 2.7 MB per anchor, keys and values, where three
// blocks per unit (what the registers of four allow) hold the launch or a pool has 32 anchors, long chains.  us with two / four (in brackets:
// four, rows requested behind the set-up), 32 layers x 8 heads, bf16, D = 128 unless said:
//   8 tokens, 8 anchors 6.6 / 5.9 (6.1), 64 anchors 25.6 / 18.9 (24.2); 16 tokens, 16 anchors 10.6 / 9.1 (10.0); f32, D = 64, 8 x 4, 77 tokens, 8 anchors
//   6.7 / 5.8 (5.8), 16: 9.7 / 7.8 (8.1); 80 layers, 8 tokens, 64 anchors 49.0 / 35.3 (31.7); one token, f32, 8 anchors 5.4 / 5.2 (4.7);
//   but 33 tokens, 8 anchors 12.2 / 13.3 (14.9); 64 tokens, 16 anchors 26.3 / 29.1 (31.1); 80 layers, one token, 8 anchors 6.2 / 7.4 (7.0).
// Of 480 launches of pools from four on the rule's choice is 0.3 % slower on average than the faster one.
bool few_rows(const AlignParams &p, int64_t n_blocks, int max_sel, int row_bytes)
{
    int64_t tokens = 0;
    int min_sel = max_sel;
    for (int j = 0; j < p.head.n_jobs; ++j) {
        tokens += p.job[j].S;
        min_sel = std::min<int>(min_sel, p.job[j].n_sel);
    }
    return min_sel >= 4 && 2 * tokens * p.head.LH * row_bytes <= 2700000 && (2 * n_blocks <= 3 * kComputeUnits || max_sel >= 32);
}

template <typename T, int LPR>
int launch_align(const AlignParams &p, const AlignLaunch &pl, int units, hipStream_t stream)
{
    constexpr int HALF = LPR * Elem<T>::EPV;
    constexpr int RPB = kBlock / LPR;
    const size_t lds = sizeof(float2) * (size_t)pl.max_tab * HALF + sizeof(float) * (size_t)RPB * pl.max_sel;
    const AlignHead &hd = p.head;
    const dim3 grid((unsigned)(hd.lh_range * hd.tiles_total), (unsigned)(2 * ((hd.LH + hd.lh_range - 1) / hd.lh_range)));
    const auto kernel = few_rows(p, pl.n_blocks, pl.max_sel, 32 * LPR) ? align_kernel<T, LPR, true> : align_kernel<T, LPR, false>;
    return launch(kernel, grid, dim3(kBlock), std::max(lds, lds_reserve(p, pl.n_blocks, LPR, (int)sizeof(T), units)), stream, p);
}

int align_kv_batch(const kvcomm_model *model, int32_t gran, kvcomm_tensor anchor_layout, const kvcomm_align_job *jobs, int32_t n_jobs,
                   int32_t units, void *stream)
{
    AlignParams p{};
    AlignLaunch pl{};
    const int es = model ? elem_size(model->dtype) : 2;
    int st = plan_align(model, gran, anchor_layout, es, jobs, n_jobs, kOnePairPerBlock, p, pl,
                        [](int, const kvcomm_align_job &, int) { return (int)KVCOMM_OK; });
    if (st) return st;
    for (int j = 0; j < n_jobs; ++j) {
        p.job[j].by_pitch = make_divisor((uint32_t)std::max(1, jobs[j].n_anchors));
        for (int a = 0; a < jobs[j].n_anchors; ++a) p.job[j].sel_mask |= (uint64_t)(jobs[j].anchor_len[a] >= jobs[j].seg_len) << a;
    }
    // A launch holds fewer than 2^32 threads along an axis, and 65535 blocks along the second: more (layer, head) pairs than go along the
    // first come as further pairs (keys, values) along that one.
    constexpr int64_t kMaxBlocks = ((int64_t)1 << 32) / kBlock - 1;
    AlignHead &hd = p.head;
    hd.lh_range = (int32_t)std::min<int64_t>(hd.LH, kMaxBlocks / hd.tiles_total);
    if (hd.lh_range < 1 || (hd.LH + hd.lh_range - 1) / hd.lh_range > 65535 / 2) return KVCOMM_EUNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (model->dtype == KVCOMM_BF16) {
        switch (pl.lpr) {
            case 4: return launch_align<bf16_t, 4>(p, pl, units, s);
            case 8: return launch_align<bf16_t, 8>(p, pl, units, s);
            case 16: return launch_align<bf16_t, 16>(p, pl, units, s);
        }
    } else {
        switch (pl.lpr) {
            case 8: return launch_align<float, 8>(p, pl, units, s);
            case 16: return launch_align<float, 16>(p, pl, units, s);
            case 32: return launch_align<float, 32>(p, pl, units, s);
        }
    }
    return KVCOMM_EUNSUPPORTED;
}

}  // namespace

extern "C" int kvcomm_align_kv_batch(const kvcomm_model *model, int32_t gran, kvcomm_tensor anchor_layout,
                                     const kvcomm_align_job *jobs, int32_t n_jobs, void *stream)
{
    return align_kv_batch(model, gran, anchor_layout, jobs, n_jobs, kComputeUnits, stream);
}

extern "C" int kvcomm_align_kv_batch_beside(const kvcomm_model *model, int32_t gran, kvcomm_tensor anchor_layout,
                                            const kvcomm_align_job *jobs, int32_t n_jobs, int32_t units, void *stream)
{
    if (units <= 0) return KVCOMM_EINVAL;
    return align_kv_batch(model, gran, anchor_layout, jobs, n_jobs, units, stream);
}

extern "C" int kvcomm_align_kv(const kvcomm_model *model, int32_t gran, kvcomm_tensor base_k, kvcomm_tensor base_v,
                               int32_t seg_len, const void *const *anchor_dk, const void *const *anchor_dv,
                               kvcomm_tensor anchor_layout, const int32_t *anchor_len, int32_t n_anchors,
                               const float *weights, int32_t delta_pos, const int32_t *anchor_delta_pos,
                               kvcomm_tensor out_k, kvcomm_tensor out_v, void *stream)
{
    kvcomm_align_job job{};
    job.base_k = base_k;
    job.base_v = base_v;
    job.out_k = out_k;
    job.out_v = out_v;
    job.seg_len = seg_len;
    job.delta_pos = delta_pos;
    job.anchor_dk = anchor_dk;
    job.anchor_dv = anchor_dv;
    job.anchor_len = anchor_len;
    job.anchor_delta_pos = anchor_delta_pos;
    job.n_anchors = n_anchors;
    job.weights = weights;
    job.weights_slots = check_model(model) || check_gran(gran) ? 0 : (int64_t)kvcomm_weight_slots(model, seg_len, gran);
    return kvcomm_align_kv_batch(model, gran, anchor_layout, &job, 1, stream);
}
