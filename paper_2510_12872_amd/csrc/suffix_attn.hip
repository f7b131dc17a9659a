// kvcomm_suffix_attn: causal attention of the non-shared suffix queries over the assembled,
// aligned cache (workflow step 4 of the paper; q, k, v as in Sec. 3.1).  Suffix query i sits
// at cache position n_ctx + i and sees keys 0 .. n_ctx + i.
//
// bf16 path (attn_mfma_kernel): flash-style single pass on bf16 MFMA (16x16x32) with fp32
// accumulation and an fp32 online softmax, written for gfx950:
//   * 16x16x32, not 32x32x16: the chip is power-limited under this kernel, and a stream of the small ones sustains
//     1930-1940 TFLOP/s on N(0,1) data where a stream of the large ones sustains 1660-1710.  A wavefront still owns 32 queries,
//     as two halves of 16 that share every K and V^T operand, so LDS reads and registers are what they were.  Twice as
//     many matrix instructions to issue take a part of it back: the pipes are busy in 56 % of the launch's cycles at 1.93 GHz instead of
//     60 % at 1.80, and a launch on 160 of the 256 units, which leaves power to spare where nothing runs beside it, takes 0.85 ms
//     instead of 0.81 (0.86 both on a slower chip; beside the update of another agent the step gains 1 %).  32 layers, Tq 512, 3072 keys: 654 -> 648 us; 64 heads, 8704 keys: 16 layers 1860 -> 1783 us, 80 layers
//     9001 -> 8923 us; one layer, 3072 keys, four runs: 40.8 -> 39.4 us; D = 256, 8 layers, 3072 keys: 423 -> 408 us.
//   * GQA packing: the G query heads that share a kv head are folded into the row axis of one
//     tile (row r = i * G + g), so each K/V tile staged in LDS serves G heads at once.
//   * Both products are computed transposed, S^T = K Q^T and O^T = V^T P^T.  In the 16x16
//     accumulator layout a lane then owns one query column of each half: row max and row sum of the softmax
//     are in-register reductions plus two lane swaps at the end, the rescale of O is a per-lane
//     scalar, and the exponentiated scores are already laid out as the B operand of the second
//     product (the key order inside a 32-key step is a fixed permutation, matched on the V side).
//   * K and V tiles travel global -> LDS with global_load_lds_dwordx4 (no registers, no LDS
//     stores), issued through inline assembly with a scalar row base and a fixed per-lane offset;
//     the XOR swizzle of 16-byte chunks that keeps operand reads bank-conflict free is
//     applied by choosing which global chunk each lane fetches.  K operands are read with
//     ds_read_b128; V^T operands with ds_read_b64_tr_b16, which transposes on the way out of
//     LDS, so V is never transposed by the vector ALU.
//   * Work advances in 32-key sub-steps as a three-stage software pipeline inside each wavefront:
//     in one step the matrix cores compute S(u+2) = K(u+2) Q^T and O += V(u) P(u), pairs of MFMAs
//     alternating, while the vector ALU turns S(u+1) into P(u+1).  The vector work is cut into one
//     piece per MFMA and staggered so that no instruction reads what its own piece produced; every
//     piece is pinned by a scheduling barrier.
//   * The softmax reference is not tracked.  It is set from the first sub-step (key 0 is visible to
//     every query) and a sub-step only checks that the row sum of its exponentials, which is needed
//     anyway, stayed below 2^30; a row that did not is re-referenced to its true maximum (O and
//     the running sum rescaled, the exponentials formed again).  Numerator and denominator share
//     the reference, so the result is that of the usual online softmax.  Row sums are plain fp32
//     additions of the unrounded exponentials.
//   * One barrier per 64 keys; K is kept in a ring of four 32-key halves and V in two 64-key
//     tiles so that loads run 1-2 tiles ahead of their use.
//   * A block is eight wavefronts (two per SIMD, 256 registers each) = 256 rows of the packed
//     (query, head) axis = 64 queries of all four heads for G = 4; one block per CU.
//   * Row tiles are ordered longest-first and the block index is remapped so that the row
//     tiles of one (layer, kv head) run on the same XCD and share its L2.
// fp32 path: attn_f32.hip.
#include <float.h>

#include "attn_common.h"
#include "attn_plan.h"

namespace {

using namespace kvc;

// ------------------------------------------------------------------------------- bf16 MFMA
// PERSIST: the grid is smaller than the number of (layer, kv head, row tile) items and every block walks a
// fixed share of them (the items of its XCD, strided by the XCD's number of blocks), so that the kernel occupies
// gridDim.x CUs only and leaves the rest of the chip to whatever runs beside it.  The arithmetic of an item is
// the same instruction sequence as in the one-item-per-block form.
// SPLIT: an item is one run of key tiles of a row tile.  The block works on the cache as if it began at the run's
// first key (which all its queries see) and leaves unnormalised outputs, references and row sums in the workspace;
// attn_combine_kernel joins them.
template <int D, int NW, int WPE, bool PERSIST, bool SPLIT>
__global__ __launch_bounds__(64 * NW, WPE) void attn_mfma_kernel(const AttnParams p_arg)
{
    // PERSIST reads the parameters through an opaque pointer to the kernel-argument segment, once per item:
    // they are then re-loaded (scalar loads) for every item instead of being held in scalar registers for the
    // whole kernel, which the register budget does not allow.
    using ParamT = std::conditional_t<PERSIST, const __attribute__((address_space(4))) AttnParams, const AttnParams>;
    ParamT *p_ptr;
    if constexpr (PERSIST)
        p_ptr = (ParamT *)__builtin_amdgcn_kernarg_segment_ptr();
    else
        p_ptr = &p_arg;
    ParamT &p0 = *p_ptr;
    constexpr int NF = D / 16;       // K operands of a sub-step (contraction step, key half), V^T operands (16 channels)
    constexpr int BM = 32 * NW;      // query rows per block (32 per wavefront)
    constexpr int RW = 64 / NW;      // key rows of a 64-key group that one wavefront loads
    constexpr int KCH = D / 8;       // 16-byte chunks per K / V row
    constexpr int ROWB = D * 2;      // bytes per K / V row
    constexpr int HALFB = 32 * ROWB; // bytes of a 32-key half tile
    constexpr int TILEB = 64 * ROWB; // bytes of a 64-key tile
    constexpr int RPL = 64 / KCH;    // key rows filled by one wavefront-wide direct load
    constexpr int LPT = RW / RPL;    // direct loads per wavefront, tensor and 64-key group
    // Chunk swizzles: chunk c of key `key` sits at position c ^ swz(key).  16 chunks span the 64 banks (two keys at D = 64).
    // K: sixteen lanes read one chunk of sixteen keys.  V: a transposing read of 32 lanes takes two chunks of eight keys.
    auto k_swz = [](int key) __attribute__((always_inline)) -> int { return D == 64 ? (key >> 1) & 7 : key & 15; };
    auto v_swz = [](int key) __attribute__((always_inline)) -> int {
        return D == 64 ? (2 * (key & 2)) | ((key >> 1) & 2) : 4 * (key & 3) | ((key >> 1) & 2);
    };

    // K: ring of four 32-key halves (half h in slot h & 3); V: two 64-key tiles (tile t in buffer t & 1).
    // Rows are [key][D] with XOR-swizzled 16-byte chunks.
    // After the last tile the same memory stages the output rows (32 rows per wavefront) for coalesced stores;
    // the table of row pointers sits behind it.
    __shared__ __align__(16) unsigned char smem[4 * HALFB + 2 * TILEB + NW * 32 * 8];
    static_assert(NW * 32 * ROWB <= 4 * HALFB + 2 * TILEB, "output staging must fit the K / V buffers");
    lds_byte *kring = (lds_byte *)smem;
    lds_byte *vbuf = kring + 4 * HALFB;

    // XCD-aware item order: hardware deals consecutive block ids round-robin to the 8 XCDs; each XCD gets one
    // contiguous range of the items (the row tiles of a (layer, kv head) then share its L2).  Block b is the
    // (b / 8)-th block of XCD b % 8 and takes that range's items b / 8, b / 8 + (blocks of the XCD), ...
    const int x_id = blockIdx.x & 7;
    const int x_first = x_id * (p0.n_items >> 3) + min(x_id, p0.n_items & 7);
    const int x_count = (p0.n_items >> 3) + (x_id < (p0.n_items & 7) ? 1 : 0);
    const int x_blocks = PERSIST ? ((int)gridDim.x - x_id + 7) >> 3 : x_count;
    int item = blockIdx.x >> 3;
    if (PERSIST && item >= x_count) return;   // the whole block: more blocks than items on this XCD
    do {
    int logical = x_first + item;
    int tid = threadIdx.x;
    ParamT *p_item = p_ptr;
    if constexpr (PERSIST) {
        // opaque per item: nothing derived from the item, the thread id or the parameters is kept in registers
        // across items
        asm volatile("" : "+s"(logical));
        asm volatile("" : "+v"(tid));
        asm volatile("" : "+s"(p_item));
    }
    ParamT &p = *p_item;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, g4 = lane >> 4;
    int split = 0;
    if constexpr (SPLIT) {
        const int rest = div_by(logical, p.by_splits);
        split = logical - rest * p.n_splits;
        logical = rest;
    }
    const int lh = div_by(logical, p.by_row_tiles);
    const int rt = p.n_row_tiles - 1 - (logical - lh * p.n_row_tiles);  // longest rows first
    const int l = div_by(lh, p.by_Hkv), hkv = lh - l * p.Hkv;

    const bf16_t *kb_ = static_cast<const bf16_t *>(p.k) + l * p.s_k.layer + hkv * p.s_k.head;
    const bf16_t *vb_ = static_cast<const bf16_t *>(p.v) + l * p.s_v.layer + hkv * p.s_v.head;

    // Every wavefront of the block walks the same tiles (one barrier per 64-key tile); the causal
    // mask is applied from the first 32-key sub-step that is partly hidden from some query of the block.
    const int wg_imax = min(p.tq - 1, div_by(rt * BM + BM - 1, p.by_G));
    const int wg_imin = min(p.tq - 1, div_by(rt * BM, p.by_G));
    const int all_tiles = (p.n_ctx + wg_imax + 1 + 63) / 64;
    const int first_hidden = (p.n_ctx + wg_imin) / 64 + 1;
    const int tile0 = SPLIT ? split_bound(split, p.n_splits, all_tiles, first_hidden) : 0;
    const int n_tiles = SPLIT ? split_bound(split + 1, p.n_splits, all_tiles, first_hidden) - tile0 : all_tiles;
    if constexpr (SPLIT) {
        if (n_tiles <= 0) {   // the whole block: this run is empty
            if (lane < 32 && div_by(rt * BM + wave * 32 + lane, p.by_G) < p.tq) {
                const int64_t part = ((int64_t)(lh * p.n_row_tiles + rt) * NW + wave) * p.n_splits + split;
                p.part_ml[part * 64 + lane] = -INFINITY;
                p.part_ml[part * 64 + 32 + lane] = 0.f;
            }
            if (!PERSIST) return;
            item += x_blocks;
            continue;
        }
        kb_ += (int64_t)(64 * tile0) * p.s_k.token;
        vb_ += (int64_t)(64 * tile0) * p.s_v.token;
    }
    // Context length and cache length counted from the run's first key (n_ctx_() may be negative; every query of
    // the tile still sees key 0 of the run).
    auto n_ctx_ = [&]() __attribute__((always_inline)) -> int { return SPLIT ? p.n_ctx - 64 * tile0 : p.n_ctx; };
    auto N_ = [&]() __attribute__((always_inline)) -> int { return SPLIT ? p.N - 64 * tile0 : p.N; };
    const int n_sub = 2 * n_tiles;
    const int sub_unmasked = (n_ctx_() + wg_imin + 1) / 32;  // sub-steps [0, sub_unmasked) are visible to all queries

    f32x4 o[2][NF];   // [query half][16 channels]
    constexpr bool kAccO = D == 256;   // O lives in the accumulation registers: the others have no room for it
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int db = 0; db < NF; ++db) o[h][db] = f32x4{0.f, 0.f, 0.f, 0.f};

    // ---- global -> LDS direct loads (global_load_lds_dwordx4): lane i of a wavefront fills the
    // 16-byte LDS chunk (base + i); the swizzle is applied by choosing which global chunk it fetches.
    // One instruction fills RPL consecutive key rows.  Addresses are a wavefront-uniform row pointer
    // plus a per-lane byte offset that does not change from tile to tile.
    // In a 64-key group, wavefront w fills keys [RW*w, RW*w + RW); load `it` fills rows RW*w + it*RPL ...
    auto in_row_k = [&](int it) __attribute__((always_inline)) -> int {  // swizzled source chunk (bytes inside the row), K
        const int key = wave * RW + it * RPL + lane / KCH;   // only the row index modulo 16 matters
        return ((lane % KCH) ^ k_swz(key)) * 16;
    };
    auto in_row_v = [&](int it) __attribute__((always_inline)) -> int {  // same for V
        const int key = wave * RW + it * RPL + lane / KCH;
        return ((lane % KCH) ^ v_swz(key)) * 16;
    };
    uint32_t ld_koff[LPT], ld_voff[LPT];
#pragma unroll
    for (int it = 0; it < LPT; ++it) {
        ld_koff[it] = (uint32_t)((lane / KCH) * p.s_k.token * 2 + in_row_k(it));
        ld_voff[it] = (uint32_t)((lane / KCH) * p.s_v.token * 2 + in_row_v(it));
    }
    const unsigned char *kbytes = reinterpret_cast<const unsigned char *>(kb_);
    const unsigned char *vbytes = reinterpret_cast<const unsigned char *>(vb_);

    // 64 keys starting at key0 (a multiple of 64) -> K ring; its two halves are h0 = key0/32 and h0+1.
    // A half outside [0, n_sub) is skipped.  The lower NW/2 wavefronts fill the first half, the rest the second.
    // General form (prologue and the last tiles): rows past the cache end re-read the last row; such
    // rows are never unmasked.  The row base is clamped on the scalar unit and a lane whose row would
    // still fall behind the end steps its offset back by whole rows.
    const int lq = lane / KCH;  // this lane's row inside a load
    const uint32_t k_row_bytes = (uint32_t)(p.s_k.token * 2), v_row_bytes = (uint32_t)(p.s_v.token * 2);
    auto load_rows = [&](const unsigned char *bytes, int64_t tok_stride, uint32_t row_bytes, int row0, uint32_t voff,
                         const lds_byte *dst) __attribute__((always_inline)) {
        const int row0c = min(row0, N_() - 1);            // wavefront-uniform
        const int excess = max(lq - (N_() - 1 - row0c), 0);  // rows this lane would overshoot by
        dma16_sbase(bytes + (int64_t)row0c * tok_stride * 2, voff - (uint32_t)excess * row_bytes, dst);
    };
    auto load_k64 = [&](int key0) __attribute__((always_inline)) {
        const int h = key0 / 32 + wave / (NW / 2);
        if (h >= n_sub) return;  // wavefront-uniform
        const int rbase = (wave % (NW / 2)) * RW;
#pragma unroll
        for (int it = 0; it < LPT; ++it)
            load_rows(kbytes, p.s_k.token, k_row_bytes, 32 * h + rbase + it * RPL, ld_koff[it],
                      kring + (h & 3) * HALFB + (rbase + it * RPL) * ROWB);
    };
    auto load_v64 = [&](int tile) __attribute__((always_inline)) {
        if (tile >= n_tiles) return;
#pragma unroll
        for (int it = 0; it < LPT; ++it)
            load_rows(vbytes, p.s_v.token, v_row_bytes, 64 * tile + wave * RW + it * RPL, ld_voff[it],
                      vbuf + (tile & 1) * TILEB + (wave * RW + it * RPL) * ROWB);
    };
    // The first tiles are requested before anything else is set up: their latency is the block's start-up time.
    load_k64(0);    // halves 0, 1
    load_k64(64);   // halves 2, 3
    load_v64(0);
    // This lane's two query columns, n and 16 + n of the wavefront's 32: row r = i * G + g of the (layer, kv head) group.
    int qi[2];
    bf16x8 qf[2][NF / 2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r_row = rt * BM + wave * 32 + 16 * h + n;
        const int i_row = div_by(r_row, p.by_G);
        qi[h] = min(i_row, p.tq - 1);
        const int hq = hkv * p.G + r_row - i_row * p.G;
        const bf16_t *qrow = static_cast<const bf16_t *>(p.q) + l * p.s_q.layer + (int64_t)(uint32_t)hq * p.s_q.head + (int64_t)(uint32_t)qi[h] * p.s_q.token;
#pragma unroll
        for (int ks = 0; ks < NF / 2; ++ks) qf[h][ks] = as_bf16x8(load16(qrow + ks * 32 + g4 * 8));
    }

    // Steady state (all rows exist, no half is skipped): the same loads from two running row pointers,
    // so that a load costs one 64-bit scalar add instead of a 64-bit multiply, and with M0 formed from
    // a per-wavefront LDS base plus a literal.  kp / vp point at this wavefront's next row to load:
    // during tile t the K halves 2t+4, 2t+5 (keys 64t+128 ...) and V tile t+1.
    const int64_t k_rpl = (int64_t)RPL * p.s_k.token * 2, v_rpl = (int64_t)RPL * p.s_v.token * 2;
    const int64_t k_adv = (int64_t)(64 - LPT * RPL) * p.s_k.token * 2, v_adv = (int64_t)(64 - LPT * RPL) * p.s_v.token * 2;
    const unsigned char *kp = kbytes + (int64_t)(128 + 32 * (wave / (NW / 2)) + (wave % (NW / 2)) * RW) * p.s_k.token * 2;
    const unsigned char *vp = vbytes + (int64_t)(64 + wave * RW) * p.s_v.token * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)kring;
    const uint32_t k_rows = lds0 + (wave % (NW / 2)) * RW * ROWB;
    // t even: halves 2t+4, 2t+5 live in slots 0, 1; t odd: in slots 2, 3
    const uint32_t kdst_a = __builtin_amdgcn_readfirstlane(k_rows + (0 + wave / (NW / 2)) * HALFB);
    const uint32_t kdst_b = __builtin_amdgcn_readfirstlane(k_rows + (2 + wave / (NW / 2)) * HALFB);
    const uint32_t vdst = __builtin_amdgcn_readfirstlane(lds0 + 4 * HALFB + wave * RW * ROWB);
    auto load_kv_next = [&](uint32_t kdst, auto vb) __attribute__((always_inline)) {
        constexpr int VB = decltype(vb)::value;  // V buffer, a literal
        static_for<0, LPT>([&](auto it) __attribute__((always_inline)) {
            constexpr int I = decltype(it)::value;
            if (I > 0) kp += k_rpl;
            dma16_sbase_at<I * RPL * ROWB>(kp, ld_koff[I], kdst);
        });
        kp += k_rpl + k_adv;
        static_for<0, LPT>([&](auto it) __attribute__((always_inline)) {
            constexpr int I = decltype(it)::value;
            if (I > 0) vp += v_rpl;
            dma16_sbase_at<VB * TILEB + I * RPL * ROWB>(vp, ld_voff[I], vdst);
        });
        vp += v_rpl + v_adv;
    };

    // ---- per-lane LDS read offsets
    // K operand (rows = keys): lane (n, g4) reads chunk 4 * ks + g4 of key n or 16 + n of the half.
    int k_off[NF / 2];
#pragma unroll
    for (int ks = 0; ks < NF / 2; ++ks) k_off[ks] = n * ROWB + (((4 * ks + g4) ^ k_swz(n)) * 16);
    // V^T operand through transposing reads: lane i of a 16-lane group supplies the address of
    // 4 channels [16 * db + 4 * (i % 4), + 4) of key 4 * g4 + i / 4 (second read: + 16 keys).
    int v_off[NF];
    {
        const int row = 4 * g4 + (n >> 2);
#pragma unroll
        for (int db = 0; db < NF; ++db) {
            const int col = 16 * db + 4 * (n & 3);
            v_off[db] = row * ROWB + ((col >> 3) ^ v_swz(row)) * 16 + (col & 7) * 2;
        }
    }
    auto read_k = [&](const lds_byte *kl, int i) __attribute__((always_inline)) -> bf16x8 {  // i = 2 * ks + key half
        return as_bf16x8(*(const __attribute__((address_space(3))) u32x4 *)(kl + (i & 1) * 16 * ROWB + k_off[i >> 1]));
    };
    auto read_v = [&](const lds_byte *vl, int db) __attribute__((always_inline)) -> bf16x8 {
        const lds_byte *va = vl + v_off[db];
        return lds_read_tr_pair(va, va + 16 * ROWB);
    };

    // ---- softmax state of this lane's two queries.
    // m is the REFERENCE the exponentials are taken against (raw score units), mc = m * scale * log2(e).  It is
    // a true maximum when it is set, but it is not tracked: a sub-step only checks that its exponentials stayed
    // in range (their row sums, which are needed anyway, below kOverflow) and re-references the rows when they did
    // not.  Numerator and denominator share the reference, so the result is that of the usual online softmax;
    // exponentials beyond 1 cost no accuracy in floating point.
    float m[2] = {-INFINITY, -INFINITY}, mc[2] = {0.f, 0.f}, lsum[2] = {0.f, 0.f};
    f32x4 sbuf[2][2][2]; // scores of sub-step u live in sbuf[u & 1][key half][query half]
    u32x4 pbuf[2][2];    // packed bf16 probabilities of sub-step u live in pbuf[u & 1][query half]

    // P = exp2(s * scale * log2(e) - mc) for the 16 scores of this lane, as packed bf16 B operands, and their sums.
    // The work is cut into the MFMA slots of a pipeline step and staggered so that no instruction reads
    // what its own slot produced: element j is scaled in slot b-2, exponentiated in slot b-1 and
    // summed / packed in slot b = j * NS / 16 (slots -2 and -1 precede the first MFMA).  A wavefront issues in
    // order, so a dependent chain inside one slot would hold back the next MFMA for its whole latency.
    // Element j is key row 16 * kh + 4 * g4 + r of the sub-step for query half j / 8, kh = j / 4 % 2, r = j % 4; `limit`
    // plus the query's index is its last visible key.
    // Row sums are plain fp32 additions of the unrounded exponentials: v_dot2 on the rounded pairs
    // would agree with the numerator to the last bit, but it shares a pipeline with the MFMAs and costs four
    // times as much next to them; the difference is a relative 2^-9 / sqrt(keys) of the denominator.
    struct ExpState {
        float x[16], e[16], rs[2];
    };
    typedef f32x4 Scores[2][2];
    auto score = [&](const Scores &s, int j, int limit, bool masked) __attribute__((always_inline)) -> float {
        const int h = j >> 3, kh = (j >> 2) & 1, r = j & 3;
        return masked && 16 * kh + 4 * g4 + r > limit + qi[h] ? -INFINITY : s[kh][h][r];
    };
    auto exp_slot = [&](const Scores &s, u32x4 (&pk)[2], ExpState &st, int limit, bool masked, int t, int NS)
                        __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int b = j * NS / 16, h = j >> 3;
            if (b - 2 == t) st.x[j] = __builtin_fmaf(score(s, j, limit, masked), p.scale_log2, -mc[h]);
            if (b - 1 == t) st.e[j] = __builtin_amdgcn_exp2f(st.x[j]);
            if (b == t) {
                if (j & 1) {
                    uint32_t pr = pack_bf16x2(st.e[j - 1], st.e[j]);
                    asm volatile("" : "+v"(pr));  // keeps the conversion in this slot (it would sink to its use, a step later)
                    pk[h][(j & 7) >> 1] = pr;
                }
                st.rs[h] = (j & 7) == 0 ? st.e[j] : st.rs[h] + st.e[j];
            }
        }
    };
    // A row whose exponentials left the safe range (or the first sub-step, whose reference is still -inf): take
    // the true maximum of the sub-step as the new reference if it is larger, rescale what has been accumulated,
    // and form the exponentials again.  Rare: the reference only ever moves by more than log2(kOverflow).
    auto rereference = [&](const Scores &s, u32x4 (&pk)[2], ExpState &st, int limit, bool masked) __attribute__((always_inline)) {
        if (kAccO || !masked) mfma_settle<kAccO>(o);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float mx = -INFINITY;
#pragma unroll
            for (int j = 8 * h; j < 8 * h + 8; ++j) mx = fmaxf(mx, score(s, j, limit, masked));
            const float m_new = fmaxf(m[h], query_max(mx));
            // m == -inf: nothing but exponentials of 0 so far (the first sub-step, or scores of -inf only)
            const float corr = m[h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m[h] - m_new) * p.scale_log2);
            m[h] = m_new;
            // No score above -inf yet (key 0 of the block's keys is visible to every query, but its score may be -inf): a
            // reference so low that scores of -inf still give 0 and the first finite one overflows, which brings it here.
            mc[h] = fmaxf(m_new * p.scale_log2, -FLT_MAX);
            lsum[h] *= corr;
#pragma unroll
            for (int db = 0; db < NF; ++db) o[h][db] *= corr;
        }
#pragma unroll
        for (int t = -2; t < 16; ++t) exp_slot(s, pk, st, limit, masked, t, 16);
    };
    constexpr float kOverflow = 1073741824.f;  // 2^30

    // One pipeline step for sub-step u (U4 = u & 3, a literal at every call site, fixes every ring slot and buffer):
    //   matrix cores:  S(u+2) = K(u+2) Q^T  and  O += V(u) P(u), pairs of MFMAs that share the K or V^T operand alternating;
    //   vector ALU:    P(u+1) = exp2(S(u+1) - reference), spread evenly over the MFMAs.
    // DO_QK / DO_EXP are false only in the last two sub-steps.  LDS operands are fetched two pairs of their own
    // product ahead; every MFMA + vector chunk is pinned by a scheduling barrier.
    auto step = [&](int u, auto u4c, auto do_qk_c, auto do_exp_c, auto masked_c) __attribute__((always_inline)) {
        constexpr int U4 = decltype(u4c)::value;
        constexpr bool DO_QK = decltype(do_qk_c)::value, DO_EXP = decltype(do_exp_c)::value, MASKED = decltype(masked_c)::value;
        constexpr int NS = 4 * NF;   // slots: the MFMAs of both products
        // The compiler copies operands right before the MFMAs of masked sub-steps, and moves scores of D = 256 between register files.
        constexpr Mfma HOW_S = !MASKED && !kAccO ? Mfma::kInPlace : Mfma::kBuiltin;
        constexpr Mfma HOW_O = !MASKED ? Mfma::kInPlace : kAccO ? Mfma::kGuarded : Mfma::kBuiltin;
        Scores &s_acc = sbuf[U4 & 1];
        const Scores &s_exp = sbuf[(U4 + 1) & 1];
        const lds_byte *kl = kring + ((U4 + 2) & 3) * HALFB;
        const lds_byte *vl = vbuf + ((U4 >> 1) & 1) * TILEB + (U4 & 1) * HALFB;
        const int limit = n_ctx_() - 32 * (u + 1);  // last key of S(u+1), relative to its sub-step, that query 0 sees
        bf16x8 ka[NF], va[NF], pf[2];
        pf[0] = as_bf16x8(pbuf[U4 & 1][0]);
        pf[1] = as_bf16x8(pbuf[U4 & 1][1]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (DO_QK) ka[i] = read_k(kl, i);
            va[i] = read_v(vl, i);
        }
        ExpState st;
        auto vec = [&](int t) __attribute__((always_inline)) {
            if (DO_EXP) exp_slot(s_exp, pbuf[(U4 + 1) & 1], st, limit, MASKED, t, NS);
        };
        vec(-2);
        vec(-1);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (DO_QK) {
                    if (i < 2)
                        mfma_first<HOW_S>(s_acc[i & 1][h], ka[i], qf[h][i >> 1]);
                    else
                        mfma_next<HOW_S>(s_acc[i & 1][h], ka[i], qf[h][i >> 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (h == 0 && i + 2 < NF) {
                    if (DO_QK) ka[i + 2] = read_k(kl, i + 2);
                    va[i + 2] = read_v(vl, i + 2);
                }
                vec(4 * i + h);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                mfma_next<HOW_O, kAccO>(o[h][i], va[i], pf[h]);
                __builtin_amdgcn_sched_barrier(0);
                vec(4 * i + 2 + h);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (DO_EXP) {
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(st.rs[0] + st.rs[1] < kOverflow)) != 0, 0))
                rereference(s_exp, pbuf[(U4 + 1) & 1], st, limit, MASKED);
            lsum[0] += st.rs[0];
            lsum[1] += st.rs[1];
        }
    };
    const auto tile_barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wavefront's direct loads have landed in LDS
        __syncthreads();                     // ... and everybody else's; what was read in this tile is free
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    template_int<0> u0; template_int<1> u1; template_int<2> u2; template_int<3> u3;

    // ---- pipeline over tiles.  During tile t the sub-steps 2t and 2t+1 read K halves 2t+2 and 2t+3 and V tile t;
    // the loads issued at its start (K halves 2t+4, 2t+5 into the slots of halves 2t and 2t+1, V tile t+1 into the
    // buffer of tile t-1) only overwrite what tile t-1 finished reading.
    tile_barrier();

    // Prologue: S(0) and S(1); the reference of every query from S(0) (key 0 is visible to all); P(0).
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const lds_byte *kl = kring + h * HALFB;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const bf16x8 ka = read_k(kl, i);
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    sbuf[h][i & 1][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qf[c][i >> 1], i < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : sbuf[h][i & 1][c], 0, 0, 0);
            }
        }
        ExpState st;
        rereference(sbuf[0], pbuf[0], st, n_ctx_(), true);
        lsum[0] = st.rs[0];
        lsum[1] = st.rs[1];
    }
    // Halves 0 and 1 have no tile before them: every wavefront must have read them before the loads of the
    // first tile (halves 4 and 5 share their slots) are issued.
    __syncthreads();

    if (kAccO) mfma_settle<kAccO>(o);   // (the zeros)
    const int t_last = n_tiles - 1;
    // Leading tiles whose exponentials need no mask and whose look-ahead loads stay inside the cache: a tile pair
    // starting at t forms the exponentials of sub-steps up to 2t+4 and loads keys up to 64t + 255.
    const int t_safe = N_() >= 256 ? (N_() - 128) / 64 : 0;
    const int t_plain = max(0, min(min((sub_unmasked - 1) >> 1, t_last), t_safe));
    // Two tiles (four sub-steps) per trip so that ring slots and buffers are compile-time constants.
    auto tile_pair = [&](int t, auto plain) __attribute__((always_inline)) {
        constexpr bool PLAIN = decltype(plain)::value;
        using M_ = std::integral_constant<bool, !PLAIN>;
        if (PLAIN) {
            load_kv_next(kdst_a, template_int<1>{});  // K halves 2t+4, 2t+5, V tile t+1
        } else {
            load_k64(64 * t + 128);
            load_v64(t + 1);
        }
        step(2 * t, u0, T_{}, T_{}, M_{});
        step(2 * t + 1, u1, T_{}, T_{}, M_{});
        tile_barrier();
        if (PLAIN) {
            load_kv_next(kdst_b, template_int<0>{});  // K halves 2t+6, 2t+7, V tile t+2
        } else {
            load_k64(64 * t + 192);
            load_v64(t + 2);
        }
        step(2 * t + 2, u2, T_{}, T_{}, M_{});
        step(2 * t + 3, u3, T_{}, T_{}, M_{});
        tile_barrier();
    };
    int t = 0;
    for (; t + 2 <= t_plain; t += 2) tile_pair(t, T_{});
    mfma_settle<kAccO>(o);
    for (; t + 2 <= t_last; t += 2) tile_pair(t, F_{});
    if (t < t_last) {  // two tiles left (t is even): a whole one, then the last
        load_k64(64 * t + 128);
        load_v64(t + 1);
        step(2 * t, u0, T_{}, T_{}, T_{});
        step(2 * t + 1, u1, T_{}, T_{}, T_{});
        tile_barrier();
        ++t;
        step(2 * t, u2, F_{}, T_{}, T_{});      // S(2t+1) exists already; nothing further to multiply
        step(2 * t + 1, u3, F_{}, F_{}, T_{});  // the last sub-step only adds its V P
    } else {
        step(2 * t, u0, F_{}, T_{}, T_{});
        step(2 * t + 1, u1, F_{}, F_{}, T_{});
    }

    if (kAccO) mfma_settle<kAccO>(o);
    if constexpr (SPLIT) {
        // ---- epilogue of a split: accumulators as they are (256-byte runs per store), reference and row sum.
        const int64_t part = ((int64_t)(lh * p.n_row_tiles + rt) * NW + wave) * p.n_splits + split;
        const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int n_e = lane_e & 15, g_e = lane_e >> 4;
        f32x4 *po = reinterpret_cast<f32x4 *>(p.part_o + part * (32 * D));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float ltot = query_sum(lsum[h]);
            const int row = 16 * h + n_e;
            if (div_by(rt * BM + wave * 32 + row, p.by_G) < p.tq) {
#pragma unroll
                for (int db = 0; db < NF; ++db) po[part_slot(4 * db + g_e, row)] = o[h][db];
                if (g_e < 2) p.part_ml[part * 64 + 32 * g_e + row] = g_e ? ltot : m[h];
            }
        }
        if (!PERSIST) return;
        __syncthreads();   // every wavefront has read its last tiles: the buffers become those of the next item
        item += x_blocks;
        continue;
    }
    // ---- epilogue: normalise and store; lane (n, g4) holds channels 16 * db + 4 * g4 ... + 3 of query rows n and 16 + n.
    // Stored straight from these registers a store instruction would scatter 8-byte pieces over 16 rows (16 K
    // partial-line writes per block, several microseconds of back-pressure).  Instead each wavefront passes its
    // 32 rows through LDS (8-byte slots XOR-swizzled with the row number so that neither side conflicts much) and
    // writes them out as whole rows, 16 bytes per lane.
    {
        // Row coordinates again, from a freshly read lane id: the compiler then keeps none of the
        // prologue's address terms alive across the tile loops.
        const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int n_e = lane_e & 15, g_e = lane_e >> 4;
        constexpr int SLOTS = 2 * KCH;                       // 8-byte slots per row
        constexpr int FM = (SLOTS < 32 ? SLOTS : 32) - 1;    // swizzle mask
        __syncthreads();  // every wavefront has finished reading K and V (and no direct load is outstanding)
        unsigned char *stage = smem + wave * (32 * ROWB);
        uint64_t *ptab = reinterpret_cast<uint64_t *>(smem + 4 * HALFB + 2 * TILEB) + wave * 32;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = 16 * h + n_e, r_row = rt * BM + wave * 32 + row;
            const uint32_t qi_e = (uint32_t)div_by(r_row, p.by_G), hq_e = (uint32_t)(hkv * p.G + r_row) - qi_e * (uint32_t)p.G;
            const bool valid = qi_e < (uint32_t)p.tq;
            bf16_t *orow = static_cast<bf16_t *>(p.out) + l * p.s_o.layer + (int64_t)hq_e * p.s_o.head + (int64_t)qi_e * p.s_o.token;
            const float ltot = query_sum(lsum[h]);
            if (g_e == 0) ptab[row] = valid ? (uint64_t)(uintptr_t)orow : 0;
            const float inv = 1.f / ltot;
#pragma unroll
            for (int db = 0; db < NF; ++db) {
                u32x2 w;
                w[0] = pack_bf16x2(o[h][db][0] * inv, o[h][db][1] * inv);
                w[1] = pack_bf16x2(o[h][db][2] * inv, o[h][db][3] * inv);
                *reinterpret_cast<u32x2 *>(stage + row * ROWB + ((4 * db + g_e) ^ (row & FM)) * 8) = w;
            }
            if (p.lse && g_e == 0 && valid)
                p.lse[((int64_t)l * p.Hkv * p.G + hq_e) * p.tq + qi_e] = m[h] * p.scale + logf(ltot);
        }
        // the reads below touch what other lanes of this wavefront wrote: LDS operations of a wavefront complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int RPS = 64 / KCH;   // rows per store instruction
        const int c = lane_e % KCH;
#pragma unroll
        for (int it = 0; it < 32 / RPS; ++it) {
            const int row = it * RPS + lane_e / KCH;
            const int f = row & FM;
            const u32x2 lo = *reinterpret_cast<const u32x2 *>(stage + row * ROWB + ((2 * c) ^ f) * 8);
            const u32x2 hi = *reinterpret_cast<const u32x2 *>(stage + row * ROWB + ((2 * c + 1) ^ f) * 8);
            bf16_t *dst = reinterpret_cast<bf16_t *>((uintptr_t)ptab[row]);
            if (dst) {
                const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
                *reinterpret_cast<u32x4 *>(dst + c * 8) = v;
            }
        }
    }
    if (!PERSIST) break;
    __syncthreads();   // the staging area becomes the K / V buffers of the next item
    item += x_blocks;
    } while (item < x_count);
}

}  // namespace

extern "C" size_t kvcomm_suffix_attn_workspace(const kvcomm_model *model, int32_t n_ctx, int32_t tq)
{
    if (check_model(model) || tq <= 0 || n_ctx < 0 || model->dtype != KVCOMM_BF16) return 0;
    return attn_workspace(*model, attn_plan(*model, n_ctx, tq, true));
}

namespace {

template <int D, int NW, int WPE>
int launch_mfma(const AttnParams &p, unsigned n_blocks, bool persist, hipStream_t s)
{
    const dim3 grid(n_blocks), block(64 * NW);
    if (p.n_splits > 1)
        return persist ? launch(attn_mfma_kernel<D, NW, WPE, true, true>, grid, block, 0, s, p)
                       : launch(attn_mfma_kernel<D, NW, WPE, false, true>, grid, block, 0, s, p);
    return persist ? launch(attn_mfma_kernel<D, NW, WPE, true, false>, grid, block, 0, s, p)
                   : launch(attn_mfma_kernel<D, NW, WPE, false, false>, grid, block, 0, s, p);
}

// max_blocks > 0: at most that many thread blocks (the kernels' persistent form when there are more items; the fp32 kernel of
// short caches is small-block and ignores it).
// A workspace of at least kvcomm_suffix_attn_workspace() bytes lets a small launch split the key axis; without one
// (or with one that is too small or not 16-byte aligned) the keys of a row tile stay in one block.
int suffix_attn(const kvcomm_model *model, kvcomm_tensor q, kvcomm_tensor cache_k, kvcomm_tensor cache_v, int32_t n_ctx,
                int32_t tq, float softmax_scale, kvcomm_tensor out, float *lse_out, int32_t max_blocks, void *workspace,
                size_t workspace_bytes, void *stream)
{
    int st = check_model(model);
    if (st) return st;
    if (tq <= 0 || n_ctx < 0) return KVCOMM_EINVAL;
    const int dt = model->dtype;
    if ((st = check_tensor(q, dt, true)) || (st = check_tensor(cache_k, dt, true)) ||
        (st = check_tensor(cache_v, dt, true)) || (st = check_tensor(out, dt, true)))
        return st;

    AttnParams p{};
    p.q = q.ptr;
    p.k = cache_k.ptr;
    p.v = cache_v.ptr;
    p.out = out.ptr;
    p.lse = lse_out;
    p.s_q = strides_of(q);
    p.s_k = strides_of(cache_k);
    p.s_v = strides_of(cache_v);
    p.s_o = strides_of(out);
    p.L = model->n_layers;
    p.Hkv = model->n_kv_heads;
    p.G = model->n_q_heads / model->n_kv_heads;
    p.n_ctx = n_ctx;
    p.tq = tq;
    p.N = n_ctx + tq;
    p.scale = softmax_scale > 0.f ? softmax_scale : (float)(1.0 / sqrt((double)model->head_dim));
    p.scale_log2 = (float)((double)p.scale * 1.4426950408889634);
    p.n_splits = 1;
    p.groups_per_tile = 1;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int D = model->head_dim;

    if (dt == KVCOMM_F32) {
        p.groups_per_tile = attn_f32_groups(*model, tq, max_blocks);
        const int rows = 16 * p.groups_per_tile;
        p.n_row_tiles = (int32_t)(((int64_t)p.G * tq + rows - 1) / rows);
        const int64_t n_items = (int64_t)p.L * p.Hkv * p.n_row_tiles;
        if (n_items > 0x7fffffff) return KVCOMM_EUNSUPPORTED;
        p.n_items = (int32_t)n_items;
        set_divisors(p);
        return launch_attn_f32(p, D, (unsigned)(max_blocks > 0 ? std::min(max_blocks, p.n_items) : p.n_items), s);
    }

    // The direct loads address a row group as a 64-bit scalar base plus an unsigned 32-bit per-lane byte
    // offset that spans up to 64 * 8 / D rows: the token stride has to leave that offset below 2^32.
    const int64_t rows_per_load = 64 * 8 / D;
    const int64_t max_tok = ((int64_t)1 << 31) / (2 * rows_per_load);
    if (cache_k.stride_token >= max_tok || cache_v.stride_token >= max_tok) return KVCOMM_EUNSUPPORTED;

    AttnPlan plan = attn_plan(*model, n_ctx, tq, true);
    size_t need = attn_workspace(*model, plan);
    if (plan.n_splits > 1 && (!workspace || workspace_bytes < need || !aligned16(workspace))) {
        plan = attn_plan(*model, n_ctx, tq, false);
        need = 0;
    }
    p.n_row_tiles = plan.n_row_tiles;
    p.n_splits = plan.n_splits;
    p.groups_per_tile = plan.tile_rows / plan.group_rows;
    p.n_items = p.L * p.Hkv * p.n_row_tiles * p.n_splits;
    if (p.n_splits > 1) {
        p.part_o = static_cast<float *>(workspace);
        p.part_ml = p.part_o + attn_parts(*model, plan) * (size_t)(plan.group_rows * D);
    }
    set_divisors(p);
    const bool persist = max_blocks > 0 && max_blocks < p.n_items;
    const unsigned n_blocks = persist ? (unsigned)max_blocks : (unsigned)p.n_items;
    if (plan.rows_kernel) {
        st = launch_attn_rows(p, D, plan.tile_rows, n_blocks, s);
    } else {
        switch (D) {
            case 64: st = launch_mfma<64, kAttnWaves, 2>(p, n_blocks, persist, s); break;
            case 128: st = launch_mfma<128, kAttnWaves, 2>(p, n_blocks, persist, s); break;
            default: st = launch_mfma<256, 4, 1>(p, n_blocks, persist, s); break;
        }
    }
    if (st || p.n_splits == 1) return st;
    return launch_attn_combine(p, D, plan.group_rows, s);
}

}  // namespace

extern "C" int kvcomm_suffix_attn(const kvcomm_model *model, kvcomm_tensor q, kvcomm_tensor cache_k,
                                  kvcomm_tensor cache_v, int32_t n_ctx, int32_t tq, float softmax_scale,
                                  kvcomm_tensor out, float *lse_out, void *workspace, size_t workspace_bytes, void *stream)
{
    return suffix_attn(model, q, cache_k, cache_v, n_ctx, tq, softmax_scale, out, lse_out, 0, workspace, workspace_bytes,
                       stream);
}

extern "C" int kvcomm_suffix_attn_confined(const kvcomm_model *model, kvcomm_tensor q, kvcomm_tensor cache_k,
                                           kvcomm_tensor cache_v, int32_t n_ctx, int32_t tq, float softmax_scale,
                                           kvcomm_tensor out, float *lse_out, int32_t max_blocks, void *stream)
{
    return kvcomm_suffix_attn_confined_ws(model, q, cache_k, cache_v, n_ctx, tq, softmax_scale, out, lse_out, max_blocks,
                                          nullptr, 0, stream);
}

extern "C" int kvcomm_suffix_attn_confined_ws(const kvcomm_model *model, kvcomm_tensor q, kvcomm_tensor cache_k,
                                              kvcomm_tensor cache_v, int32_t n_ctx, int32_t tq, float softmax_scale,
                                              kvcomm_tensor out, float *lse_out, int32_t max_blocks, void *workspace,
                                              size_t workspace_bytes, void *stream)
{
    if (max_blocks < 8) return KVCOMM_EINVAL;   // at least one block on each of the 8 XCDs
    return suffix_attn(model, q, cache_k, cache_v, n_ctx, tq, softmax_scale, out, lse_out, max_blocks, workspace,
                       workspace_bytes, stream);
}
