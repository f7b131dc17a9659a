// fp32 suffix attention: fp32 MFMA (exact fp32 products and sums) with expf and an online softmax, fp32 throughout.
#include "attn_plan.h"

namespace {

using namespace kvc;

constexpr int kF32Waves = 8;

// Caches of up to f32_row_keys() tokens: one wavefront per query row, one key per lane, dot products on the vector ALU.  Its time grows with
// the keys, that of the kernel below starts higher.  4 layers x 8 heads, G = 4, us here / there: one key 4.0 / 4.5 (D = 64), 4.8 / 5.8 (128),
// 6.4 / 8.0 (256); 6 keys 4.5 / 4.6, 5.3 / 5.8, 6.9 / 8.0; 12 keys 5.1 / 4.6, 6.0 / 5.9, 7.7 / 8.6; 20 keys 6.0 / 4.7, 7.2 / 6.1, 9.1 / 8.3; 64 keys
// 11.2 / 5.1, 13.4 / 6.4, 17.3 / 8.7.
constexpr int f32_row_keys(int D) { return D == 256 ? 16 : 8; }

template <int D>
__global__ __launch_bounds__(256) void attn_f32_row_kernel(const AttnParams p)
{
    static_assert(f32_row_keys(D) <= 64, "every key has its lane");
    constexpr int CPL = D / 64;  // output channels per lane
    __shared__ float q_lds[4][D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + wave;  // over (l, hq, i)
    const int Hq = p.Hkv * p.G;
    if (row >= (int64_t)p.L * Hq * p.tq) return;
    const int i = (int)(row % p.tq);
    const int hq = (int)((row / p.tq) % Hq);
    const int l = (int)(row / ((int64_t)p.tq * Hq));
    const int hkv = hq / p.G;
    const float *q = static_cast<const float *>(p.q) + l * p.s_q.layer + (int64_t)hq * p.s_q.head + i * p.s_q.token;
    const float *k = static_cast<const float *>(p.k) + l * p.s_k.layer + (int64_t)hkv * p.s_k.head;
    const float *v = static_cast<const float *>(p.v) + l * p.s_v.layer + (int64_t)hkv * p.s_v.head;
    for (int c = lane; c < D; c += 64) q_lds[wave][c] = q[c];
    // only this wavefront reads q_lds[wave]; its writes are ordered before the reads below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    const int last = p.n_ctx + i;   // < f32_row_keys(D)
    float sc = -INFINITY;
    if (lane <= last) {
        const float *kr = k + (int64_t)lane * p.s_k.token;
        float dot = 0.f;
#pragma unroll 4
        for (int c = 0; c < D; c += 4) {
            const f32x4 kv = *reinterpret_cast<const f32x4 *>(kr + c);
            dot = fmaf(q_lds[wave][c], kv[0], dot);
            dot = fmaf(q_lds[wave][c + 1], kv[1], dot);
            dot = fmaf(q_lds[wave][c + 2], kv[2], dot);
            dot = fmaf(q_lds[wave][c + 3], kv[3], dot);
        }
        sc = dot * p.scale;
    }
    float m = sc;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    const float pj = lane <= last ? expf(sc - m) : 0.f;
    float lsum = pj;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off);
    float acc[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c] = 0.f;
    for (int j = 0; j <= last; ++j) {
        const float pv = __shfl(pj, j);
        const float *vr = v + (int64_t)j * p.s_v.token;
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = fmaf(pv, vr[lane + 64 * c], acc[c]);
    }
    float *o = static_cast<float *>(p.out) + l * p.s_o.layer + (int64_t)hq * p.s_o.head + i * p.s_o.token;
    const float inv = 1.f / lsum;
#pragma unroll
    for (int c = 0; c < CPL; ++c) o[lane + 64 * c] = acc[c] * inv;
    if (p.lse && lane == 0) p.lse[row] = m + logf(lsum);
}

// attn_f32_kernel: 16 * RH packed (query, head) rows per block (GQA packing as in attn_mfma_kernel) on 16x16x4 MFMAs; the wavefronts share
// the rows and each takes every NW-th 16-key sub-step with its own softmax state, joined through LDS at the end.  Both products
// are transposed, so a lane owns one query column of each 16 rows, and every operand comes straight from global memory in the layout the
// instruction wants: of K and Q 16-byte pieces (the contraction order is free as long as both agree: piece j of lane (n, g) holds channels
// 16 * j + 4 * g ... + 3), of V four consecutive channels of one key (row m of accumulator (t, c) stands for channel 64 * t + 4 * m + c),
// P from the score registers.
// What bounds it: at large sizes matrix cores (fp32 MFMA, 1/16 of the bf16 rate), at small ones the length of a wavefront's chain.  So 16 rows
// up to a block per compute unit (attn_f32_groups()): half the products of a sub-step and twice the blocks; else two groups of 16 that share every
// K and V operand.  us before (32 rows and 32 keys on 32x32x2 MFMAs, K loads of 64 lines) and now: 2 layers x 4 heads x 64 rows, 224
// keys, D = 64 10.3 -> 7.7; 4 x 8, G = 8, one token, 1025 keys, D = 128 54.8 -> 29.6, 256 96 -> 58; 4 x 8, G = 4, Tq 128, 1152 keys, D = 64 60.5 -> 55.5,
// 128 118 -> 105, 256 195 -> 193; one layer, Tq 512, 3072 keys, D = 128 272 -> 243 (97 TFLOP/s; back to back, as all of these).
template <int D, int RH>
__device__ __forceinline__ void attn_f32_item(const AttnParams &p, int item)   // item: one row tile of a (layer, kv head)
{
    constexpr int NW = kF32Waves;
    constexpr int NJ = D / 16, NT = D / 64;                 // 16-byte pieces of a K row in a lane, loads of a V row
    constexpr int NP = D == 256 ? 2 : 1, PJ = NJ / NP;         // parts of a K row (32 registers at most), pieces of a part
    constexpr int HOLD = RH == 2 ? 1 : NP;                   // parts in registers at a time
    constexpr int VR = D == 256 ? 2 : 4;                   // V rows of a lane's four keys in registers at a time
    constexpr bool kQInRegs = D == 64 && RH == 1;
    __shared__ __align__(16) f32x4 smem[NW * NT * 256];      // the wavefronts' outputs of 16 rows, before them Q
    static_assert(RH * NJ * 64 <= NW * NT * 256, "Q must fit");
    __shared__ __align__(16) float ms[RH * 16][NW], ls[RH * 16][NW];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    const int lh = div_by(item, p.by_row_tiles), rt = item - lh * p.n_row_tiles;
    const int l = div_by(lh, p.by_Hkv), hkv = lh - l * p.Hkv;
    const int row0 = rt * 16 * RH;
    const int imax = min(p.tq - 1, div_by(row0 + 16 * RH - 1, p.by_G)), imin = min(p.tq - 1, div_by(row0, p.by_G));
    const int units = (p.n_ctx + imax + 16) / 16;   // sub-steps that some query of the tile sees

    const float *kb = static_cast<const float *>(p.k) + l * p.s_k.layer + hkv * p.s_k.head;
    const float *vb = static_cast<const float *>(p.v) + l * p.s_v.layer + hkv * p.s_v.head;
    int qi[RH];
    const float *qrow[RH];
#pragma unroll
    for (int h = 0; h < RH; ++h) {
        const int r_row = row0 + 16 * h + n, i_row = div_by(r_row, p.by_G), head = hkv * p.G + r_row - i_row * p.G;
        qi[h] = min(i_row, p.tq - 1);
        qrow[h] = static_cast<const float *>(p.q) + l * p.s_q.layer + (int64_t)head * p.s_q.head + (int64_t)qi[h] * p.s_q.token;
    }
    f32x4 k[HOLD][PJ], v[VR][NT];
    // Rows past the cache end re-read the last one; they are always masked.
    auto load_k = [&](int u, int part) __attribute__((always_inline)) {
        const float *kr = kb + (int64_t)min(16 * u + n, p.N - 1) * p.s_k.token + 16 * PJ * part + 4 * g;
#pragma unroll
        for (int j = 0; j < PJ; ++j) k[part % HOLD][j] = *reinterpret_cast<const f32x4 *>(kr + 16 * j);
    };
    auto load_v = [&](int u, int r0) __attribute__((always_inline)) {   // score r of this lane is key 4 * g + r
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            const float *vr = vb + (int64_t)min(16 * u + 4 * g + r0 + r, p.N - 1) * p.s_v.token + 4 * n;
#pragma unroll
            for (int t = 0; t < NT; ++t) v[r][t] = *reinterpret_cast<const f32x4 *>(vr + 64 * t);
        }
    };
    f32x4 qf[RH][kQInRegs ? NJ : 1];
    if constexpr (kQInRegs) {
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
            for (int j = 0; j < NJ; ++j) qf[h][j] = *reinterpret_cast<const f32x4 *>(qrow[h] + 16 * j + 4 * g);
    } else {
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
            for (int i = 0; i < (NJ + NW - 1) / NW; ++i) {
                const int j = wave + i * NW;
                if (NJ >= NW || j < NJ) smem[(h * NJ + j) * 64 + lane] = *reinterpret_cast<const f32x4 *>(qrow[h] + 16 * j + 4 * g);
            }
    }
    if (wave < units) {
#pragma unroll
        for (int part = 0; part < HOLD; ++part) load_k(wave, part);
        load_v(wave, 0);
    } else {
#pragma unroll
        for (int part = 0; part < HOLD; ++part)
#pragma unroll
            for (int j = 0; j < PJ; ++j) k[part][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < VR; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) v[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if constexpr (!kQInRegs) __syncthreads();

    f32x4 o[RH][NT][4];
    float m[RH], lsum[RH];   // lsum: this lane's quarter of the row sum
    bool odd = false;        // left out a value that is not finite
#pragma unroll
    for (int h = 0; h < RH; ++h) {
        m[h] = -INFINITY;
        lsum[h] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[h][t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    auto sub_step = [&](int u, auto edge_c) __attribute__((always_inline)) {   // edge: some key is hidden from some query
        constexpr bool EDGE = decltype(edge_c)::value;
        const bool more = u + NW < units;
        f32x4 s[RH];
#pragma unroll
        for (int h = 0; h < RH; ++h) s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int part = 0; part < NP; ++part) {
#pragma unroll
            for (int j = 0; j < PJ; ++j) {
                f32x4 q[RH];
#pragma unroll
                for (int h = 0; h < RH; ++h) q[h] = kQInRegs ? qf[h][kQInRegs ? j : 0] : smem[(h * NJ + part * PJ + j) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int h = 0; h < RH; ++h) s[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[part % HOLD][j][e], q[h][e], s[h], 0, 0, 0);
                if (D == 256 || !kQInRegs) __builtin_amdgcn_sched_barrier(0);   // (all of Q would be read first, into registers that do not exist)
            }
            if (HOLD < NP && part + 1 < NP) load_k(u, part + 1);
        }
        if (more) {
#pragma unroll
            for (int part = 0; part < HOLD; ++part) load_k(u + NW, part);
        }
#pragma unroll
        for (int h = 0; h < RH; ++h) {
            const int limit = p.n_ctx + qi[h] - 16 * u - 4 * g;     // last visible one of this lane's keys
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[h][r] *= p.scale;
                if (EDGE && r > limit) s[h][r] = -INFINITY;
                mx = fmaxf(mx, s[h][r]);
            }
            mx = query_max(mx);
            if (__builtin_amdgcn_ballot_w64(mx > m[h]) != 0) {
                const float m_new = fmaxf(m[h], mx);
                const float corr = m[h] == -INFINITY ? 0.f : expf(m[h] - m_new);
                lsum[h] *= corr;
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c) o[h][t][c] *= corr;
                m[h] = m_new;
            }
            const float mref = m[h] == -INFINITY ? 0.f : m[h];   // a row that sees no key yet: exponentials 0
            float rs = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[h][r] = expf(s[h][r] - mref);
                rs += s[h][r];
            }
            lsum[h] += rs;
        }

        // A hidden key must not reach the result, not even as 0 * inf: at the causal edge values that are not finite are
        // left out here and added behind the loop to the queries that do see them.
#pragma unroll
        for (int r0 = 0; r0 < 4; r0 += VR) {
            if (r0) {
                __builtin_amdgcn_sched_barrier(0);
                load_v(u, r0);
            }
#pragma unroll
            for (int r = 0; r < VR; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float x = v[r][t][c];
                        if (EDGE) {
                            const bool fin = fabsf(x) < INFINITY;
                            odd |= !fin;
                            x = fin ? x : 0.f;
                        }
#pragma unroll
                        for (int h = 0; h < RH; ++h)
                            o[h][t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, s[h][r0 + r], o[h][t][c], 0, 0, 0);
                    }
        }
        if (more) load_v(u + NW, 0);
    };
    // Two loops: with a branch inside one, V selected in place, the compiler gave other values the registers of rows that were still to
    // be multiplied.
    const int u_edge = (p.n_ctx + imin + 1) / 16;   // first sub-step with a hidden key
    int u = wave;
    for (; u < min(u_edge, units); u += NW) sub_step(u, std::false_type{});
    for (; u < units; u += NW) sub_step(u, std::true_type{});

    // ---- join the wavefronts' states and store.  Lane (n, g) holds channels 64 * t + 16 * g + 4 * r + c of query rows n (and 16 + n).
#pragma unroll
    for (int h = 0; h < RH; ++h) {
        lsum[h] = query_sum(lsum[h]);
        if (g == 0) ms[16 * h + n][wave] = m[h];
    }
    __syncthreads();   // also: every wavefront has read Q for the last time
#pragma unroll
    for (int h = 0; h < RH; ++h) {
        float M = ms[16 * h + n][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) M = fmaxf(M, ms[16 * h + n][w]);
        const float f = m[h] == -INFINITY ? 0.f : expf(m[h] - M);
        if (g == 0) ls[16 * h + n][wave] = m[h] == -INFINITY ? lsum[h] : lsum[h] * f;   // reference -inf: sum 0, or NaN from NaN scores
        if (h) __syncthreads();   // the rows before have been read
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                smem[(wave * NT + t) * 256 + r * 64 + lane] = f32x4{o[h][t][0][r], o[h][t][1][r], o[h][t][2][r], o[h][t][3][r]} * f;
        __syncthreads();
        float ltot = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) ltot += ls[16 * h + n][w];
        const float inv = 1.f / ltot;
        const int r_row = row0 + 16 * h + n, i_row = div_by(r_row, p.by_G), head = hkv * p.G + r_row - i_row * p.G;
        float *orow = static_cast<float *>(p.out) + l * p.s_o.layer + (int64_t)head * p.s_o.head + (int64_t)i_row * p.s_o.token;
        if (i_row < p.tq) {
#pragma unroll
            for (int i = 0; i < (4 * NT + NW - 1) / NW; ++i) {
                const int slot = wave + NW * i;   // 4 * t + r
                if (slot < 4 * NT) {
                    f32x4 a = smem[slot * 64 + lane];
#pragma unroll
                    for (int w = 1; w < NW; ++w) a += smem[w * NT * 256 + slot * 64 + lane];
                    *reinterpret_cast<f32x4 *>(orow + 64 * (slot >> 2) + 16 * g + 4 * (slot & 3)) = a * inv;
                }
            }
        }
        if (p.lse && wave == 0 && g == 0 && i_row < p.tq) p.lse[((int64_t)l * p.Hkv * p.G + head) * p.tq + i_row] = M + logf(ltot);
    }

    // Rare: values left out at the causal edge, for the queries that see them (thread: one query, every 4 * NW-th channel).
    if (__syncthreads_or(odd)) {
#pragma unroll 1
        for (int h = 0; h < RH; ++h) {   // (all of it formed again: nothing is kept for this across the loop)
            const int r_row = row0 + 16 * h + n, i_row = div_by(r_row, p.by_G);
            if (i_row >= p.tq) continue;
            const int head = hkv * p.G + r_row - i_row * p.G;
            const float *qr = static_cast<const float *>(p.q) + l * p.s_q.layer + (int64_t)head * p.s_q.head + (int64_t)i_row * p.s_q.token;
            float *orow = static_cast<float *>(p.out) + l * p.s_o.layer + (int64_t)head * p.s_o.head + (int64_t)i_row * p.s_o.token;
            float M = ms[16 * h + n][0], ltot = 0.f;
            for (int w = 1; w < NW; ++w) M = fmaxf(M, ms[16 * h + n][w]);
            for (int w = 0; w < NW; ++w) ltot += ls[16 * h + n][w];
            for (int key = (p.n_ctx + imin + 1) & ~15; key <= p.n_ctx + i_row; ++key) {
                const float *vr = vb + (int64_t)key * p.s_v.token;
                float pk = -1.f;
                for (int c = 4 * wave + g; c < D; c += 4 * NW) {
                    const float x = vr[c];
                    if (fabsf(x) < INFINITY) continue;
                    if (pk < 0.f) {
                        const float *kr = kb + (int64_t)key * p.s_k.token;
                        float dot = 0.f;
                        for (int i = 0; i < D; ++i) dot = fmaf(qr[i], kr[i], dot);
                        pk = expf(dot * p.scale - M) / ltot;
                    }
                    orow[c] += pk * x;
                }
            }
        }
    }
}

// PERSIST: a grid of fewer blocks than items, each walking every gridDim.x-th one.  Two blocks of D = 64 fit a compute unit.  (One group at D = 128 held to
// two as well spilled up to 24 registers: one token, 1025 keys, 4 layers x 8 heads, G = 8 on 16 blocks 60.7 us instead of 54.9; in one round the same 28.6.)
template <int D, int RH, bool PERSIST>
__global__ __launch_bounds__(64 * kF32Waves, D == 64 ? 4 : 2) void attn_f32_kernel(const AttnParams p)
{
    await_attn_args(p);
    if constexpr (!PERSIST) {
        attn_f32_item<D, RH>(p, blockIdx.x);
    } else {
        for (int item = blockIdx.x; item < p.n_items; item += gridDim.x) {
            attn_f32_item<D, RH>(p, item);
            __syncthreads();   // the joined states have been read: LDS becomes the next item's
        }
    }
}

template <int D>
int launch_f32(const AttnParams &p, bool persist, unsigned n_blocks, hipStream_t stream)
{
    const auto one = persist ? attn_f32_kernel<D, 1, true> : attn_f32_kernel<D, 1, false>;
    const auto two = persist ? attn_f32_kernel<D, 2, true> : attn_f32_kernel<D, 2, false>;
    return launch(p.groups_per_tile == 1 ? one : two, dim3(n_blocks), dim3(64 * kF32Waves), 0, stream, p);
}

}  // namespace

namespace kvc {

int launch_attn_f32(const AttnParams &p, int D, unsigned n_blocks, hipStream_t stream)
{
    if (p.N <= f32_row_keys(D)) {
        const dim3 grid((unsigned)(((int64_t)p.L * p.Hkv * p.G * p.tq + 3) / 4)), block(256);
        switch (D) {
            case 64: return launch(attn_f32_row_kernel<64>, grid, block, 0, stream, p);
            case 128: return launch(attn_f32_row_kernel<128>, grid, block, 0, stream, p);
            case 256: return launch(attn_f32_row_kernel<256>, grid, block, 0, stream, p);
            default: return KVCOMM_EUNSUPPORTED;
        }
    }
    n_blocks = std::min<unsigned>(n_blocks, (1u << 23) - 1);   // a launch holds fewer than 2^32 threads
    const bool persist = n_blocks < (unsigned)p.n_items;
    switch (D) {
        case 64: return launch_f32<64>(p, persist, n_blocks, stream);
        case 128: return launch_f32<128>(p, persist, n_blocks, stream);
        case 256: return launch_f32<256>(p, persist, n_blocks, stream);
        default: return KVCOMM_EUNSUPPORTED;
    }
}

}  // namespace kvc
