// bf16 suffix attention for few query rows (decoded tokens, very short suffixes), and the kernel that joins the
// partial results of a launch that splits the key axis.
#include "attn_plan.h"

namespace {

using namespace kvc;

template <int N>
__device__ __forceinline__ void wait_loads()   // at most N of this wavefront's vector-memory operations stay outstanding
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

// Direct loads of 32 rows from key0 on into a wavefront's buffer, chunk c of row `key` at position c ^ swz(key): a wavefront-uniform row
// pointer plus per-lane offsets that do not change from one sub-step to the next (lane_offsets(); the pattern repeats after
// NIN loads).  Rows past the cache end (last sub-step only) re-read the last row; they are always masked.
template <int D, int NIN, class Swz>
__device__ __forceinline__ void lane_offsets(uint32_t (&in)[NIN], int lane, int64_t tok, Swz swz)
{
    constexpr int KCH = D / 8, RPL = 64 / KCH;
    const int lq = lane / KCH;
#pragma unroll
    for (int i = 0; i < NIN; ++i) in[i] = (uint32_t)lq * (uint32_t)(tok * 2) + (uint32_t)(((lane % KCH) ^ swz(i * RPL + lq)) * 16);
}
template <int D, bool NT, int NIN, class Swz>
__device__ __forceinline__ void load_half(const unsigned char *bytes, int64_t tok, int key0, int n_keys, const uint32_t (&in)[NIN], int lane, Swz swz,
                                          lds_byte *dst)
{
    constexpr int KCH = D / 8, ROWB = D * 2, RPL = 64 / KCH, LPT = 32 / RPL;   // chunks and bytes of a row, rows of a load, loads
    if (key0 + 32 <= n_keys) {   // wavefront-uniform
        const unsigned char *row = bytes + (int64_t)key0 * tok * 2;
#pragma unroll
        for (int it = 0; it < LPT; ++it, row += (int64_t)RPL * tok * 2) dma16_sbase<NT>(row, in[it % NIN], dst + it * RPL * ROWB);
    } else {
        const int lq = lane / KCH;
#pragma unroll 1
        for (int it = 0; it < LPT; ++it) {
            const int row0 = min(key0 + it * RPL, n_keys - 1);
            const int row = min(lq, n_keys - 1 - row0);   // steps back by whole rows where the cache ends
            dma16_sbase<NT>(bytes + (int64_t)row0 * tok * 2,
                            (uint32_t)row * (uint32_t)(tok * 2) + (uint32_t)(((lane % KCH) ^ swz(it * RPL + lq)) * 16), dst + it * RPL * ROWB);
        }
    }
}

// attn_rows_kernel: 32 packed (query, head) rows per block (GQA packing and transposed products as in
// attn_mfma_kernel), which the wavefronts SHARE: each takes every NW-th 32-key sub-step of the block's key
// run with its own softmax state, and the states are joined through LDS at the end.  The 256-row kernel would leave
// seven of eight wavefronts without rows and walk the keys one 64-key tile after the other (one layer, one token,
// 3100 keys: 62 us; here 20 us in one block per kv head, 8.4 + 4.3 us with the keys cut into runs, and less with 16 rows, see below).
// What bounds it is the latency of the K / V stream, and HBM where every layer is in one launch (32 layers: 64 us =
// 6.4 TB/s): K and V of a sub-step go global -> LDS into the wavefront's own buffers (no block barrier in the loop),
// K of the next sub-step is requested as soon as its operands are in registers and V likewise, so a wavefront
// always has 8 ... 16 KB in flight (D = 128).  Eight wavefronts measured 10 % better than two blocks of four.
template <int D, bool NT, bool PERSIST>
__global__ __launch_bounds__(64 * rows_waves(D), D == 256 ? 1 : 2) void attn_rows_kernel(const AttnParams p)
{
    constexpr int NW = rows_waves(D);
    constexpr int NKS = D / 16, NDB = D / 32, KCH = D / 8, ROWB = D * 2, HALFB = 32 * ROWB;
    constexpr int RPL = 64 / KCH;    // key rows filled by one wavefront-wide direct load
    constexpr int LPT = 32 / RPL;    // direct loads of a 32-key half
    constexpr int KSWZ = (KCH < 16 ? KCH : 16) - 1, VSWZ = KCH - 1;
    constexpr int KD = (KSWZ + 1) / RPL > 1 ? (KSWZ + 1) / RPL : 1;  // loads after which the swizzle pattern of the rows repeats
    constexpr int VD = 4 / RPL > 1 ? 4 / RPL : 1;
    constexpr int JW = 2 * HALFB / 16;               // 16-byte slots of a wavefront's buffers: all its outputs at the end
    static_assert(NDB * 256 == JW, "a wavefront's outputs fill its own buffers");
    // Chunk c of key `key` sits at position c ^ swz(key).
    auto k_swz = [](int key) __attribute__((always_inline)) -> int { return key & KSWZ; };
    auto v_swz = [](int key) __attribute__((always_inline)) -> int { return (4 * (key & 3)) & VSWZ; };
    __shared__ __align__(16) unsigned char smem[NW * 2 * HALFB];
    __shared__ float ml[2][NW][32];

    await_attn_args(p);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 31, hg = lane >> 5;
    lds_byte *kbuf = (lds_byte *)smem + wave * 2 * HALFB;
    lds_byte *vbuf = kbuf + HALFB;

    const int x_id = blockIdx.x & 7;
    const int x_first = x_id * (p.n_items >> 3) + min(x_id, p.n_items & 7);
    const int x_count = (p.n_items >> 3) + (x_id < (p.n_items & 7) ? 1 : 0);
    const int x_blocks = PERSIST ? ((int)gridDim.x - x_id + 7) >> 3 : x_count;
    int item = blockIdx.x >> 3;
    if (PERSIST && item >= x_count) return;   // the whole block: more blocks than items on this XCD
    do {
        const int logical = x_first + item;
        const int run = div_by(logical, p.by_row_tiles);
        const int rt = logical - run * p.n_row_tiles;   // the row tiles of a key run are neighbours: they share its L2 lines
        const int lh = div_by(run, p.by_splits), split = run - lh * p.n_splits;
        const int l = div_by(lh, p.by_Hkv), hkv = lh - l * p.Hkv;

        const int r_row = rt * 32 + n, i_row = div_by(r_row, p.by_G);
        const bool valid = i_row < p.tq;
        const int qi = min(i_row, p.tq - 1);
        const int hq = hkv * p.G + r_row - i_row * p.G;
        const int imax = min(p.tq - 1, div_by(rt * 32 + 31, p.by_G)), imin = min(p.tq - 1, div_by(rt * 32, p.by_G));
        const int units = (p.n_ctx + imax + 32) / 32;   // sub-steps that some query of the tile sees
        // split_bound() without a causal edge: s * units / n_splits (<= 2^30: see there)
        const int u0 = div_by(split * units, p.by_splits), u1 = div_by((split + 1) * units, p.by_splits);

        const unsigned char *kbytes = reinterpret_cast<const unsigned char *>(static_cast<const bf16_t *>(p.k) + l * p.s_k.layer + hkv * p.s_k.head);
        const unsigned char *vbytes = reinterpret_cast<const unsigned char *>(static_cast<const bf16_t *>(p.v) + l * p.s_v.layer + hkv * p.s_v.head);
        uint32_t k_in[KD], v_in[VD];
        lane_offsets<D>(k_in, lane, p.s_k.token, k_swz);
        lane_offsets<D>(v_in, lane, p.s_v.token, v_swz);
        auto load_k = [&](int u) __attribute__((always_inline)) { load_half<D, NT>(kbytes, p.s_k.token, 32 * u, p.N, k_in, lane, k_swz, kbuf); };
        auto load_v = [&](int u) __attribute__((always_inline)) { load_half<D, NT>(vbytes, p.s_v.token, 32 * u, p.N, v_in, lane, v_swz, vbuf); };
        int u = u0 + wave;
        bf16x8 qf[NKS];
        const bf16_t *qrow = static_cast<const bf16_t *>(p.q) + l * p.s_q.layer + (int64_t)hq * p.s_q.head + (int64_t)qi * p.s_q.token;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[ks] = as_bf16x8(load16(qrow + ks * 16 + hg * 8));
        if (u < u1) {
            load_k(u);
            load_v(u);
        }

        int k_off[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) k_off[ks] = n * ROWB + (((2 * ks + hg) ^ k_swz(n)) * 16);
        int v_off[NDB];
        {
            const int i16 = lane & 15, gi = (lane >> 4) & 1, row = 4 * hg + (i16 >> 2);
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                const int col = 32 * db + 16 * gi + 4 * (i16 & 3);
                v_off[db] = row * ROWB + ((col >> 3) ^ v_swz(row)) * 16 + (col & 7) * 2;
            }
        }

        f32x16 o[NDB];
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
        float m = -INFINITY, mc = 0.f, lsum = 0.f;   // lsum: this lane's half of the row sum
        __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0), seen by the compiler: it puts no wait for the queries into the loop

        for (; u < u1; u += NW) {
            const bool more = u + NW < u1;   // wavefront-uniform
            wait_loads<LPT>();               // K(u) has landed (V(u) may be outstanding)
            f32x16 s;
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j] = 0.f;
            bf16x8 ka[NKS];                  // all operand reads in flight at once
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) ka[ks] = as_bf16x8(*(const __attribute__((address_space(3))) u32x4 *)(kbuf + k_off[ks]));
            wait_lds();                      // K(u) has been read: its buffer is free
            if (more) load_k(u + NW);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[ks], s, 0, 0, 0);

            if (32 * u + 31 > p.n_ctx + imin) {   // some key is hidden from some query
                const int limit = p.n_ctx + qi - 32 * u;
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (8 * (j >> 2) + 4 * hg + (j & 3) > limit) s[j] = -INFINITY;
            }
            float mx = s[0];
#pragma unroll
            for (int j = 1; j < 16; ++j) mx = fmaxf(mx, s[j]);
            {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            }
            if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
                const float m_new = fmaxf(m, mx);
                const float corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_new) * p.scale_log2);
                lsum *= corr;
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) o[db][j] *= corr;
                m = m_new;
                mc = m == -INFINITY ? 0.f : m * p.scale_log2;   // a row that sees no key of this run yet: exponentials 0
            }
            bf16x8 pf[2];
            float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 pk;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * h + 2 * j], p.scale_log2, -mc));
                    const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * h + 2 * j + 1], p.scale_log2, -mc));
                    rs0 += e0;
                    rs1 += e1;
                    pk[j] = pack_bf16x2(e0, e1);
                }
                pf[h] = as_bf16x8(pk);
            }
            lsum += rs0 + rs1;

            if (more)
                wait_loads<LPT>();   // V(u) has landed (K of the next sub-step may be outstanding)
            else
                wait_loads<0>();
            bf16x8 va[2 * NDB];
#pragma unroll
            for (int i = 0; i < 2 * NDB; ++i) {
                const lds_byte *vl = vbuf + (i / NDB) * 16 * ROWB + v_off[i % NDB];
                va[i] = lds_read_tr_pair(vl, vl + 8 * ROWB);
            }
            wait_lds();                      // V(u) has been read
            if (more) load_v(u + NW);
#pragma unroll
            for (int i = 0; i < 2 * NDB; ++i) o[i % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], pf[i / NDB], o[i % NDB], 0, 0, 0);
        }

        // ---- join the wavefronts' states: outputs as they are go over the wavefront's own K / V buffers (no other wavefront
        // reads those), so one barrier does; a thread then owns whole slots (its own n and hg) and sums them over
        // the wavefronts with their factors against the common maximum.
        {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(lsum), __float_as_uint(lsum), false, false);
            lsum = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
        if (hg == 0) {
            ml[0][wave][n] = m;
            ml[1][wave][n] = lsum;
        }
        f32x4 *join = reinterpret_cast<f32x4 *>(smem);
        if (valid) {
#pragma unroll
            for (int d = 0; d < NDB; ++d)
#pragma unroll
                for (int j4 = 0; j4 < 4; ++j4)
                    join[wave * JW + part_slot(8 * d + 2 * j4 + hg, n)] = f32x4{o[d][4 * j4], o[d][4 * j4 + 1], o[d][4 * j4 + 2], o[d][4 * j4 + 3]};
        }
        __syncthreads();
        float M = ml[0][0][n];
#pragma unroll
        for (int w = 1; w < NW; ++w) M = fmaxf(M, ml[0][w][n]);
        float f[NW], ltot = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = ml[0][w][n], lw = ml[1][w][n];
            f[w] = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mw - M) * p.scale_log2);
            ltot += mw == -INFINITY ? lw : lw * f[w];   // reference -inf: no key seen and sum 0, or nothing but NaN scores and a sum that says so
        }
        const int64_t part = (int64_t)(lh * p.n_row_tiles + rt) * p.n_splits + split;
        if (valid) {
            const float inv = 1.f / ltot;
#pragma unroll
            for (int i = 0; i < NDB * 256; i += 64 * NW) {
                f32x4 a = join[i + tid] * f[0];
#pragma unroll
                for (int w = 1; w < NW; ++w) a += join[w * JW + i + tid] * f[w];
                if (p.n_splits > 1) {
                    reinterpret_cast<f32x4 *>(p.part_o + part * (32 * D))[i + tid] = a;
                } else {
                    bf16_t *orow = static_cast<bf16_t *>(p.out) + l * p.s_o.layer + (int64_t)hq * p.s_o.head + (int64_t)qi * p.s_o.token;
                    const u32x2 w2 = {pack_bf16x2(a[0] * inv, a[1] * inv), pack_bf16x2(a[2] * inv, a[3] * inv)};
                    *reinterpret_cast<u32x2 *>(orow + i / 8 + 8 * wave + 4 * hg) = w2;
                }
            }
        }
        if (wave == 0 && hg == 0 && valid) {
            if (p.n_splits > 1) {
                p.part_ml[part * 64 + n] = M;
                p.part_ml[part * 64 + 32 + n] = ltot;
            } else if (p.lse) {
                p.lse[((int64_t)l * p.Hkv * p.G + hq) * p.tq + qi] = M * p.scale + logf(ltot);
            }
        }
        if (!PERSIST) break;
        __syncthreads();   // the joined states have been read: LDS becomes the next item's buffers
        item += x_blocks;
    } while (item < x_count);
}

// attn_rows_kernel16: the same split of the keys for 16 packed rows per block, on 16x16x32 MFMAs in the operand layout of attn_mfma_kernel.  What
// bounds a small launch is the number of instructions on a wavefront's way (a lone one issues one per 8 cycles), and with half the rows
// every part of it is half as long: products, exponentials, rescaling, join.  Taken where its blocks all run at once (attn_plan()).
// us per launch (HIP graph, with the combine launch where keys are cut), 32 rows -> 16: one layer, 8 kv heads, G = 4, one token: 1 key 6.3 -> 4.8,
// 701 keys 10.2 -> 8.2, 3101 keys 12.1 -> 8.4 (D = 64 9.7 -> 7.0, G = 2, D = 256 15.9 -> 11.3; 9.6, 8.0 and 13.3 with the combine kernel of 32 rows);
// 4 layers x 8 heads, Tq 16, 516 keys 9.4 -> 7.5; 32 layers, one token, 3101 keys 73.2 -> 70.8.
// RH = 2: two neighbouring tiles per block, which share every K and V operand; every row's sums are those of RH = 1, bit for bit (the runs of
// the two tiles may begin a sub-step apart).  For confined launches of more tiles than blocks.  us on 160 / 64 / 8 blocks one by one, two at a time (and as tiles
// of 32 rows on 32x32x16 MFMAs, whose sums are others): 2 layers x 8 heads, G = 4, Tq 64, 364 keys 10.8 / 19.5 / 136, 8.8 / 15.3 / 103 (8.1 / 13.9 / 95);
// D = 64, one layer, Tq 128, 2128 keys 16.1 / 29.2 / 220, 12.7 / 22.7 / 165 (11.2 / 19.6 / 139); 4 layers, Tq 16, 516 keys on 64 / 8 12.5 / 82, 9.7 / 63 (8.8 / 57).
template <int D, bool NT, bool PERSIST, int RH>
__global__ __launch_bounds__(64 * rows_waves(D), D == 256 ? 1 : 2) void attn_rows_kernel16(const AttnParams p)
{
    constexpr int NW = rows_waves(D), ROWS = 16;   // rows of a tile
    constexpr int NF = D / 16, KCH = D / 8, ROWB = D * 2, HALFB = 32 * ROWB;
    constexpr int RPL = 64 / KCH;                    // key rows filled by one wavefront-wide direct load
    constexpr int LPT = 32 / RPL;                    // direct loads of a 32-key half
    constexpr int KD = 16 / RPL, VD = RPL < 8 ? 8 / RPL : 1;   // loads after which the swizzle pattern of the rows repeats
    constexpr int JW = D * ROWS / 4;                 // 16-byte slots of a wavefront's outputs
    constexpr int JP = 2 * HALFB / 16;               // 16-byte slots of its buffers
    static_assert(RH * JW <= JP, "a wavefront's outputs fit its own buffers");
    // Chunk c of key `key` sits at position c ^ swz(key), as in attn_mfma_kernel.
    auto k_swz = [](int key) __attribute__((always_inline)) -> int { return D == 64 ? (key >> 1) & 7 : key & 15; };
    auto v_swz = [](int key) __attribute__((always_inline)) -> int {
        return D == 64 ? (2 * (key & 2)) | ((key >> 1) & 2) : 4 * (key & 3) | ((key >> 1) & 2);
    };
    __shared__ __align__(16) unsigned char smem[NW * 2 * HALFB];
    __shared__ float ml[2][NW][RH * ROWS];

    await_attn_args(p);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    lds_byte *kbuf = (lds_byte *)smem + wave * 2 * HALFB;
    lds_byte *vbuf = kbuf + HALFB;

    const int x_id = blockIdx.x & 7;
    const int x_first = x_id * (p.n_items >> 3) + min(x_id, p.n_items & 7);
    const int x_count = (p.n_items >> 3) + (x_id < (p.n_items & 7) ? 1 : 0);
    const int x_blocks = PERSIST ? ((int)gridDim.x - x_id + 7) >> 3 : x_count;
    int item = blockIdx.x >> 3;
    if (PERSIST && item >= x_count) return;   // the whole block: more blocks than items on this XCD
    do {
        const int logical = x_first + item;
        const int run = div_by(logical, p.by_row_tiles);
        const int rt0 = (logical - run * p.n_row_tiles) * RH;   // the row tiles of a key run are neighbours: they share its L2 lines
        const int lh = div_by(run, p.by_splits), split = run - lh * p.n_splits;
        const int l = div_by(lh, p.by_Hkv), hkv = lh - l * p.Hkv;
        const int n_tiles = RH == 1 ? p.n_row_tiles : (p.G * p.tq + ROWS - 1) / ROWS;   // of a (layer, kv head)

        int qi[RH], hq[RH], imin[RH], u0[RH], u1[RH];
        bool valid[RH];
#pragma unroll
        for (int h = 0; h < RH; ++h) {
            const int r_row = (rt0 + h) * ROWS + n, i_row = div_by(r_row, p.by_G);   // (also the row that this thread joins: tid % ROWS == n)
            valid[h] = i_row < p.tq;
            qi[h] = min(i_row, p.tq - 1);
            hq[h] = hkv * p.G + r_row - i_row * p.G;
            const int imax = min(p.tq - 1, div_by((rt0 + h) * ROWS + ROWS - 1, p.by_G));
            imin[h] = min(p.tq - 1, div_by((rt0 + h) * ROWS, p.by_G));
            const int units = (p.n_ctx + imax + 32) / 32;   // sub-steps that some query of the tile sees
            // split_bound() without a causal edge: s * units / n_splits (<= 2^30: see there)
            u0[h] = div_by(split * units, p.by_splits), u1[h] = div_by((split + 1) * units, p.by_splits);
        }
        if (RH == 2 && rt0 + 1 == n_tiles) u0[RH - 1] = u1[RH - 1] = u0[0];   // there is no second tile
        const int u_end = RH == 2 ? max(u1[0], u1[RH - 1]) : u1[0];
        // 0 or 1, and so the ends: the tiles' last queries are at most 16 keys apart.  1: a wavefront's sub-steps belong to one tile and the other in turn.
        const int apart = u0[RH - 1] - u0[0];
        const int u_end0 = apart ? u1[0] : u_end;   // of turn 0 (that of turn 1 is u_end)

        const unsigned char *kbytes = reinterpret_cast<const unsigned char *>(static_cast<const bf16_t *>(p.k) + l * p.s_k.layer + hkv * p.s_k.head);
        const unsigned char *vbytes = reinterpret_cast<const unsigned char *>(static_cast<const bf16_t *>(p.v) + l * p.s_v.layer + hkv * p.s_v.head);
        uint32_t k_in[KD], v_in[VD];
        lane_offsets<D>(k_in, lane, p.s_k.token, k_swz);
        lane_offsets<D>(v_in, lane, p.s_v.token, v_swz);
        auto load_k = [&](int u) __attribute__((always_inline)) { load_half<D, NT>(kbytes, p.s_k.token, 32 * u, p.N, k_in, lane, k_swz, kbuf); };
        auto load_v = [&](int u) __attribute__((always_inline)) { load_half<D, NT>(vbytes, p.s_v.token, 32 * u, p.N, v_in, lane, v_swz, vbuf); };
        int u = u0[0] + wave, turn = 0;
        bf16x8 qf[RH][NF / 2];
#pragma unroll
        for (int h = 0; h < RH; ++h) {
            const bf16_t *qrow = static_cast<const bf16_t *>(p.q) + l * p.s_q.layer + (int64_t)hq[h] * p.s_q.head + (int64_t)qi[h] * p.s_q.token;
#pragma unroll
            for (int ks = 0; ks < NF / 2; ++ks) qf[h][ks] = as_bf16x8(load16(qrow + ks * 32 + g * 8));
        }
        if (u < u_end0) {
            load_k(u);
            load_v(u);
        }

        // Operand addresses: K chunk 4 * ks + g of key n (and 16 + n); V^T is transposed on the way out of LDS.
        int k_off[NF / 2], v_off[NF];
#pragma unroll
        for (int ks = 0; ks < NF / 2; ++ks) k_off[ks] = n * ROWB + (((4 * ks + g) ^ k_swz(n)) * 16);
        {
            const int row = 4 * g + (n >> 2);
#pragma unroll
            for (int db = 0; db < NF; ++db) {
                const int col = 16 * db + 4 * (n & 3);
                v_off[db] = row * ROWB + ((col >> 3) ^ v_swz(row)) * 16 + (col & 7) * 2;
            }
        }

        f32x4 o[RH][NF];
        float m[RH], mc[RH], lsum[RH];   // lsum: this lane's quarter of the row sum
#pragma unroll
        for (int h = 0; h < RH; ++h) {
#pragma unroll
            for (int db = 0; db < NF; ++db) o[h][db] = f32x4{0.f, 0.f, 0.f, 0.f};
            m[h] = -INFINITY, mc[h] = 0.f, lsum[h] = 0.f;
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0), seen by the compiler: it puts no wait for the queries into the loop

        // The sub-step u for the tiles [H0, H1), which take it in step: their chains of instructions run beside each other.
        auto sub_step = [&](auto h0_c, auto h1_c, int next, bool more) __attribute__((always_inline)) {   // (u, next, more: wavefront-uniform)
            constexpr int H0 = decltype(h0_c)::value, H1 = decltype(h1_c)::value;
            wait_loads<LPT>();               // K(u) has landed (V(u) may be outstanding)
            bf16x8 ka[NF];                   // all operand reads in flight at once: ks = i / 2, keys 16 * (i & 1) ...
#pragma unroll
            for (int i = 0; i < NF; ++i)
                ka[i] = as_bf16x8(*(const __attribute__((address_space(3))) u32x4 *)(kbuf + (i & 1) * 16 * ROWB + k_off[i >> 1]));
            wait_lds();                      // K(u) has been read: its buffer is free
            if (more) load_k(next);
            f32x4 s[RH][2];                  // score j of this lane: key 16 * (j / 4) + 4 * g + j % 4
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int h = H0; h < H1; ++h)
                    s[h][i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[i], qf[h][i >> 1], i < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[h][i & 1], 0, 0, 0);

            if (32 * u + 31 > p.n_ctx + imin[H0]) {   // some key is hidden from some query (imin grows from tile to tile)
#pragma unroll
                for (int h = H0; h < H1; ++h) {
                    const int limit = p.n_ctx + qi[h] - 32 * u - 4 * g;
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (16 * (j >> 2) + (j & 3) > limit) s[h][j >> 2][j & 3] = -INFINITY;
                }
            }
            float mx[RH];
            bool grows = false;
#pragma unroll
            for (int h = H0; h < H1; ++h) {
                mx[h] = s[h][0][0];
#pragma unroll
                for (int j = 1; j < 8; ++j) mx[h] = fmaxf(mx[h], s[h][j >> 2][j & 3]);
                mx[h] = query_max(mx[h]);
                grows |= mx[h] > m[h];
            }
            if (__builtin_amdgcn_ballot_w64(grows) != 0) {
#pragma unroll
                for (int h = H0; h < H1; ++h) {   // (a row whose reference stays is multiplied by 1)
                    const float m_new = fmaxf(m[h], mx[h]);
                    const float corr = m[h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m[h] - m_new) * p.scale_log2);
                    lsum[h] *= corr;
#pragma unroll
                    for (int db = 0; db < NF; ++db) o[h][db] *= corr;
                    m[h] = m_new;
                    mc[h] = m[h] == -INFINITY ? 0.f : m[h] * p.scale_log2;   // a row that sees no key of this run yet: exponentials 0
                }
            }
            bf16x8 pf[RH];
#pragma unroll
            for (int h = H0; h < H1; ++h) {
                u32x4 pk;
                float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h][j >> 1][2 * (j & 1)], p.scale_log2, -mc[h]));
                    const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h][j >> 1][2 * (j & 1) + 1], p.scale_log2, -mc[h]));
                    rs0 += e0;
                    rs1 += e1;
                    pk[j] = pack_bf16x2(e0, e1);
                }
                pf[h] = as_bf16x8(pk);
                lsum[h] += rs0 + rs1;
            }

            if (more)
                wait_loads<LPT>();   // V(u) has landed (K of the next sub-step may be outstanding)
            else
                wait_loads<0>();
            bf16x8 va[NF];
#pragma unroll
            for (int db = 0; db < NF; ++db) va[db] = lds_read_tr_pair(vbuf + v_off[db], vbuf + v_off[db] + 16 * ROWB);
            wait_lds();                      // V(u) has been read
            if (more) load_v(next);
#pragma unroll
            for (int db = 0; db < NF; ++db)
#pragma unroll
                for (int h = H0; h < H1; ++h) o[h][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[db], pf[h], o[h][db], 0, 0, 0);
        };
        if constexpr (RH == 1) {
            for (; u < u_end; u += NW) sub_step(template_int<0>{}, template_int<1>{}, u + NW, u + NW < u_end);
        } else {
            if (apart == 0)
                for (; u < min(u1[0], u1[RH - 1]); u += NW) sub_step(template_int<0>{}, template_int<2>{}, u + NW, u + NW < u_end);
            while (u < (turn == 0 ? u_end0 : u_end)) {   // the tiles are apart, or one of them ends before the other
                const int next = apart == 0 ? u + NW : turn == 0 ? u + apart : u + NW - apart;
                const int next_turn = apart == 0 ? 0 : turn ^ 1;
                const bool more = next < (next_turn == 0 ? u_end0 : u_end);
                if (turn == 0 && u < u1[0])
                    sub_step(template_int<0>{}, template_int<1>{}, next, more);
                else
                    sub_step(template_int<1>{}, template_int<2>{}, next, more);
                u = next;
                turn = next_turn;
            }
        }

        // ---- join the wavefronts' states as in attn_rows_kernel.  Lane (n, g) holds channels 16 * db + 4 * g ... + 3 of row n: slot
        // (4 * db + g, n).
        f32x4 *join = reinterpret_cast<f32x4 *>(smem);
#pragma unroll
        for (int h = 0; h < RH; ++h) {
            lsum[h] = query_sum(lsum[h]);
            if (g == 0) {
                ml[0][wave][ROWS * h + n] = m[h];
                ml[1][wave][ROWS * h + n] = lsum[h];
            }
            if (valid[h]) {
#pragma unroll
                for (int db = 0; db < NF; ++db) join[wave * JP + JW * h + 64 * db + lane] = o[h][db];
            }
        }
        __syncthreads();
        // A wavefront joins rows of one tile: RH = 2 the even ones of the first, the odd ones of the second.
        const int jh = RH == 1 ? 0 : wave & 1, jw = RH == 1 ? wave : wave >> 1;
        const int jrow = ROWS * jh + n, jqi = jh ? qi[RH - 1] : qi[0], jhq = jh ? hq[RH - 1] : hq[0];
        float M = ml[0][0][jrow];
#pragma unroll
        for (int w = 1; w < NW; ++w) M = fmaxf(M, ml[0][w][jrow]);
        float f[NW], ltot = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = ml[0][w][jrow], lw = ml[1][w][jrow];
            f[w] = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mw - M) * p.scale_log2);
            ltot += mw == -INFINITY ? lw : lw * f[w];   // reference -inf: no key seen and sum 0, or nothing but NaN scores and a sum that says so
        }
        const int64_t part = (int64_t)(lh * n_tiles + rt0 + jh) * p.n_splits + split;
        if (jh ? valid[RH - 1] : valid[0]) {
            const float inv = 1.f / ltot;
#pragma unroll
            for (int i = 0; i < JW; i += 64 * NW / RH) {
                const int slot = i + 64 * jw + lane;
                if (JW % (64 * NW / RH) && slot >= JW) break;
                const f32x4 *own = join + JW * jh + slot;
                f32x4 a = own[0] * f[0];
#pragma unroll
                for (int w = 1; w < NW; ++w) a += own[w * JP] * f[w];
                if (p.n_splits > 1) {
                    reinterpret_cast<f32x4 *>(p.part_o + part * (ROWS * D))[slot] = a;
                } else {
                    bf16_t *orow = static_cast<bf16_t *>(p.out) + l * p.s_o.layer + (int64_t)jhq * p.s_o.head + (int64_t)jqi * p.s_o.token;
                    const u32x2 w2 = {pack_bf16x2(a[0] * inv, a[1] * inv), pack_bf16x2(a[2] * inv, a[3] * inv)};
                    *reinterpret_cast<u32x2 *>(orow + slot / ROWS * 4) = w2;
                }
            }
            if (jw == 0 && g == 0) {
                if (p.n_splits > 1) {
                    p.part_ml[part * 2 * ROWS + n] = M;
                    p.part_ml[part * 2 * ROWS + ROWS + n] = ltot;
                } else if (p.lse) {
                    p.lse[((int64_t)l * p.Hkv * p.G + jhq) * p.tq + jqi] = M * p.scale + logf(ltot);
                }
            }
        }
        if (!PERSIST) break;
        __syncthreads();   // the joined states have been read: LDS becomes the next item's buffers
        item += x_blocks;
    } while (item < x_count);
}

// attn_combine_kernel, groups of 32 rows: one block per (group, 32 channels).  out = sum_s f_s O_s / sum_s f_s l_s with
// f_s = exp2((m_s - max m) * scale * log2 e), splits in increasing order.  All loads of the U >= n_splits partial results are in
// flight at once (the launch is a few microseconds of latency); rows leave as 64-byte pieces through LDS.
template <int D, int U>
__device__ __forceinline__ void combine32(const AttnParams &p)
{
    __shared__ __align__(16) u32x2 stage[32][9];   // 8 pieces of 4 channels a row (+1: bank spread)
    const int tid = threadIdx.x;
    const int n = tid & 31, hg = (tid >> 5) & 1, j4 = tid >> 6;
    // XCD x takes one contiguous range of the (row tile, group, channels) triples, in the order of attn_mfma_kernel's items
    const int x_id = blockIdx.x & 7, n_blocks = gridDim.x;
    const int logical = x_id * (n_blocks >> 3) + min(x_id, n_blocks & 7) + (blockIdx.x >> 3);
    const int db = logical % (D / 32), item = logical / (D / 32);
    const int row_tile = div_by(item, p.by_groups), w = item - row_tile * p.groups_per_tile;
    const int lh = div_by(row_tile, p.by_row_tiles), rt = p.n_row_tiles - 1 - (row_tile - lh * p.n_row_tiles);
    const int group = (lh * p.n_row_tiles + rt) * p.groups_per_tile + w;
    const int l = div_by(lh, p.by_Hkv), hkv = lh - l * p.Hkv;
    const int bm = 32 * p.groups_per_tile;
    auto row_of = [&](int nn, bool &ok, int64_t &q_i, int64_t &h_q) {
        const int r = rt * bm + w * 32 + nn;
        q_i = div_by(r, p.by_G);
        ok = q_i < p.tq;
        h_q = hkv * p.G + r - q_i * p.G;
    };
    bool valid;
    int64_t qi, hq;
    row_of(n, valid, qi, hq);

    if (valid) {
        const int64_t part0 = (int64_t)group * p.n_splits;
        const f32x4 *po = reinterpret_cast<const f32x4 *>(p.part_o) + part0 * (8 * D) + db * 256 + tid;
        const float *pm = p.part_ml + part0 * 64 + n;
        float ms[U], ls[U];
        f32x4 os[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int s = min(i, p.n_splits - 1);
            ms[i] = pm[s * 64];
            ls[i] = pm[s * 64 + 32];
            os[i] = po[(int64_t)s * (8 * D)];   // not used, and possibly never written, where m_s is -inf and the sum 0
        }
#pragma unroll
        for (int i = 1; i < U; ++i) {
            ms[i] = i < p.n_splits ? ms[i] : -INFINITY;
            ls[i] = i < p.n_splits ? ls[i] : 0.f;
        }
        float M = ms[0], L = 0.f;
#pragma unroll
        for (int i = 1; i < U; ++i) M = fmaxf(M, ms[i]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (ms[i] != -INFINITY || ls[i] != 0.f) {   // a run of NaN scores has reference -inf and sum NaN
                const float f = __builtin_amdgcn_exp2f((ms[i] - M) * p.scale_log2);
                L = fmaf(f, ls[i], L);
                acc += f * os[i];
            }
        }
        const float inv = 1.f / L;
        stage[n][2 * j4 + hg] = u32x2{pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv)};
        if (p.lse && db == 0 && tid < 32) p.lse[((int64_t)l * p.Hkv * p.G + hq) * p.tq + qi] = M * p.scale + logf(L);
    }
    __syncthreads();
    if (tid < 128) {
        const int row = tid >> 2, c = tid & 3;
        row_of(row, valid, qi, hq);
        if (valid) {
            const u32x2 lo = stage[row][2 * c], hi = stage[row][2 * c + 1];
            bf16_t *dst = static_cast<bf16_t *>(p.out) + l * p.s_o.layer + hq * p.s_o.head + qi * p.s_o.token + 32 * db + 8 * c;
            *reinterpret_cast<u32x4 *>(dst) = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    }
}

// Groups of 16 rows (attn_rows_kernel16): one block per (group, 16 channels); the four wavefronts share the runs (wavefront w takes
// w, w + 4, ...) and their states are joined through LDS, in a fixed order.  With few rows the launch is the chain of one wavefront's
// instructions: one token, 13 runs, both launches 9.6 us with all runs in every thread, 8.4 so.
template <int D, int U>
__device__ __forceinline__ void combine16(const AttnParams &p)
{
    constexpr int ROWS = 16, UW = U / 4;
    __shared__ f32x4 accs[4][64];
    __shared__ float ml[2][4][ROWS];
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, c4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x_id = blockIdx.x & 7, n_blocks = gridDim.x;   // (the order of combine32())
    const int logical = x_id * (n_blocks >> 3) + min(x_id, n_blocks & 7) + (blockIdx.x >> 3);
    const int db = logical % (D / 16), item = logical / (D / 16);
    const int lh = div_by(item, p.by_row_tiles), rt = p.n_row_tiles - 1 - (item - lh * p.n_row_tiles);
    const int l = div_by(lh, p.by_Hkv), hkv = lh - l * p.Hkv;
    const int r = rt * ROWS + n, qi = div_by(r, p.by_G), hq = hkv * p.G + r - qi * p.G;
    const bool valid = qi < p.tq;

    if (valid) {
        const int64_t part0 = (int64_t)(lh * p.n_row_tiles + rt) * p.n_splits;
        const f32x4 *po = reinterpret_cast<const f32x4 *>(p.part_o) + part0 * (ROWS * D / 4) + db * 64 + lane;
        const float *pm = p.part_ml + part0 * 2 * ROWS + n;
        float ms[UW], ls[UW];
        f32x4 os[UW];
#pragma unroll
        for (int i = 0; i < UW; ++i) {
            const int s = min(wave + 4 * i, p.n_splits - 1);
            ms[i] = pm[s * 2 * ROWS];
            ls[i] = pm[s * 2 * ROWS + ROWS];
            os[i] = po[(int64_t)s * (ROWS * D / 4)];   // not used, and possibly never written, where m_s is -inf and the sum 0
        }
        float M = -INFINITY, L = 0.f;
#pragma unroll
        for (int i = 0; i < UW; ++i) {
            ms[i] = wave + 4 * i < p.n_splits ? ms[i] : -INFINITY;
            ls[i] = wave + 4 * i < p.n_splits ? ls[i] : 0.f;
            M = fmaxf(M, ms[i]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < UW; ++i) {
            if (ms[i] != -INFINITY || ls[i] != 0.f) {   // a run of NaN scores has reference -inf and sum NaN
                const float f = __builtin_amdgcn_exp2f((ms[i] - M) * p.scale_log2);
                L = fmaf(f, ls[i], L);
                acc += f * os[i];
            }
        }
        accs[wave][lane] = acc;
        if (c4 == 0) {
            ml[0][wave][n] = M;
            ml[1][wave][n] = L;
        }
    }
    __syncthreads();
    if (wave == 0 && valid) {
        float ms[4], M = -INFINITY, L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            ms[w] = ml[0][w][n];
            M = fmaxf(M, ms[w]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float lw = ml[1][w][n];
            if (ms[w] != -INFINITY || lw != 0.f) {
                const float f = __builtin_amdgcn_exp2f((ms[w] - M) * p.scale_log2);
                L = fmaf(f, lw, L);
                acc += f * accs[w][lane];
            }
        }
        const float inv = 1.f / L;
        bf16_t *dst = static_cast<bf16_t *>(p.out) + l * p.s_o.layer + (int64_t)hq * p.s_o.head + (int64_t)qi * p.s_o.token + 16 * db + 4 * c4;
        *reinterpret_cast<u32x2 *>(dst) = u32x2{pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv)};
        if (p.lse && db == 0 && c4 == 0) p.lse[((int64_t)l * p.Hkv * p.G + hq) * p.tq + qi] = M * p.scale + logf(L);
    }
}

template <int D, int U, int ROWS>
__global__ __launch_bounds__(256) void attn_combine_kernel(const AttnParams p)
{
    await_attn_args(p);
    if constexpr (ROWS == 16)
        combine16<D, U>(p);
    else
        combine32<D, U>(p);
}

template <int D>
int launch_combine(const AttnParams &p, int rows, hipStream_t stream)
{
    static_assert(kRowsMaxSplits <= 16 && kTileMaxSplits <= 16, "the combine kernels take all partial results of a row at once");
    const int64_t groups = (int64_t)p.L * p.Hkv * p.n_row_tiles * p.groups_per_tile;
    const dim3 grid((unsigned)(groups * (rows == 16 ? D / 16 : D / 32))), block(256);
    const auto of16 = p.n_splits <= 4 ? attn_combine_kernel<D, 4, 16> : p.n_splits <= 8 ? attn_combine_kernel<D, 8, 16> : attn_combine_kernel<D, 16, 16>;
    const auto of32 = p.n_splits <= 4 ? attn_combine_kernel<D, 4, 32> : p.n_splits <= 8 ? attn_combine_kernel<D, 8, 32> : attn_combine_kernel<D, 16, 32>;
    return launch(rows == 16 ? of16 : of32, grid, block, 0, stream, p);
}

template <int D>
int launch_rows(const AttnParams &p, int rows, bool nt, bool persist, unsigned n_blocks, hipStream_t stream)
{
    const dim3 block(64 * rows_waves(D));
    if (rows == 16 && persist && p.n_row_tiles > 1) {   // more tiles than blocks: two of a (layer, kv head) at a time
        AttnParams pairs = p;
        pairs.n_row_tiles = (p.n_row_tiles + 1) / 2;
        pairs.by_row_tiles = make_divisor((uint32_t)pairs.n_row_tiles);
        pairs.n_items = p.n_items / p.n_row_tiles * pairs.n_row_tiles;
        return launch(attn_rows_kernel16<D, false, true, 2>, dim3(std::min(n_blocks, (unsigned)pairs.n_items)), block, 0, stream, pairs);
    }
    const dim3 grid(n_blocks);
    const auto rows16 = persist ? (nt ? attn_rows_kernel16<D, true, true, 1> : attn_rows_kernel16<D, false, true, 1>)
                                : (nt ? attn_rows_kernel16<D, true, false, 1> : attn_rows_kernel16<D, false, false, 1>);
    const auto rows32 = persist ? (nt ? attn_rows_kernel<D, true, true> : attn_rows_kernel<D, false, true>)
                                : (nt ? attn_rows_kernel<D, true, false> : attn_rows_kernel<D, false, false>);
    return launch(rows == 16 ? rows16 : rows32, grid, block, 0, stream, p);
}

}  // namespace

namespace kvc {

int launch_attn_rows(const AttnParams &p, int D, int rows, unsigned n_blocks, hipStream_t stream)
{
    // Non-temporal K / V only where they cannot stay in the last-level cache and no other block reads them: 32 layers
    // of 3100 keys (407 MB) take 64 us with it and 72 us without, 4 layers (51 MB, read again for the next token) 33 and 26.
    const bool nt = p.n_row_tiles == 1 && (int64_t)p.L * p.Hkv * p.N * D * 4 > kLastLevelCache;
    const bool persist = n_blocks < (unsigned)p.n_items;
    switch (D) {
        case 64: return launch_rows<64>(p, rows, nt, persist, n_blocks, stream);
        case 128: return launch_rows<128>(p, rows, nt, persist, n_blocks, stream);
        case 256: return launch_rows<256>(p, rows, nt, persist, n_blocks, stream);
        default: return KVCOMM_EUNSUPPORTED;
    }
}

int launch_attn_combine(const AttnParams &p, int D, int rows, hipStream_t stream)
{
    switch (D) {
        case 64: return launch_combine<64>(p, rows, stream);
        case 128: return launch_combine<128>(p, rows, stream);
        case 256: return launch_combine<256>(p, rows, stream);
        default: return KVCOMM_EUNSUPPORTED;
    }
}

}  // namespace kvc
