// Host-side choice of the bf16 attention kernel and of the cut of the key axis, and the launches that
// suffix_attn.hip takes from attn_rows.hip.
#pragma once

#include "attn_common.h"

namespace kvc {

constexpr int kAttnWaves = 8;   // wavefronts of a 256-row block; measured: 2 % faster than two blocks of 4 per CU (every K/V tile enters LDS once per CU)
constexpr int rows_waves(int D) { return D == 256 ? 4 : 8; }   // wavefronts of a rows-kernel block: what LDS holds
constexpr int kChipCUs = 256;
constexpr int kRowsMaxSplits = 16;  // attn_combine_kernel takes 4 us up to here, 6 us at 25, 11 us at 64
constexpr int kTileMaxSplits = 8;
constexpr int kMinRunTiles = 5;     // 64-key tiles of a run on average; 1200 keys, Tq 500, 64 row tiles: 35 us in four runs, 31.5 in two or uncut
constexpr int kMinSplitKeys = KVCOMM_ATTN_MIN_SPLIT_KEYS;
constexpr int64_t kLastLevelCache = (int64_t)256 << 20;

struct AttnPlan {
    bool rows_kernel;
    int tile_rows;      // packed (query, head) rows of a row tile
    int n_row_tiles;
    int n_splits;
    int group_rows;     // rows whose partial results lie together
};

// Rounds that `x` chips full of blocks take (a last round that is not full costs less than a whole one).
static inline double attn_rounds(double x) { return x <= 1.0 ? 1.0 : x + 0.3 * (ceil(x) - x); }

// Microseconds of a launch of the rows kernel (32 rows per block, the keys shared out over its wavefronts) with `items`
// (row tile, layer, kv head) triples: 6 us plus 1.1 us per iteration (32 keys of every wavefront) when few CUs are
// busy, 1.5 us when all are.  8 kv heads, G = 4, D = 128, 3100 keys (13 iterations): 22 / 24 / 26 / 50 us in 64 / 128 /
// 256 / 512 blocks.
static inline double attn_rows_us(const kvcomm_model &m, int64_t items, int64_t its)
{
    const double x = (double)items / kChipCUs, scale = m.head_dim == 64 ? 0.65 : m.head_dim == 128 ? 1.0 : 2.0;
    return attn_rounds(x) * (6.0 + scale * (1.1 + 0.4 * std::min(1.0, x)) * (double)its);
}

// Microseconds of a launch of the 256-row kernel (a block fills a CU) with the keys cut into `ns` runs: a block is 9 us
// of set-up and epilogue plus 1.15 us per 64-key tile when few CUs are busy and 1.7 us when all are; the partial
// results are written and read at about 8 TB/s, plus 3.5 us for the combine launch.  One layer, Tq 512, 3072 keys, 64
// row tiles: 66 us unsplit, 50 / 42 / 42 / 49 us in 2 / 3 / 4 / 5 runs; 320 row tiles: 141 us unsplit, 139 us in two runs.
static inline double attn_tiles_us(const kvcomm_model &m, int64_t items, int tile_rows, int64_t tiles, int ns)
{
    const double x = (double)items * ns / kChipCUs, scale = m.head_dim == 64 ? 0.65 : m.head_dim == 128 ? 1.0 : 1.45;
    const double part_bytes = (double)items * tile_rows * m.head_dim * 8;
    return attn_rounds(x) * (9.0 + scale * (1.15 + 0.55 * std::min(1.0, x)) * (double)((tiles + ns - 1) / ns)) +
           (ns > 1 ? 3.5 + part_bytes * ns / 8e6 : 0.0);
}

// Which kernel, and into how many runs the keys of a row tile are cut (one if the caller has no workspace).
// Both kernels with their best cut (and its combine launch) are compared by the modelled times.  The rows kernel is kept up to
// 1.2 times the other's time where its blocks all fit the chip at once (what the model is off, and fewer partial results), and
// taken for larger launches where it is clearly faster (few rows, so that most of a 256-row tile would be empty).
// Measured, one layer, 8 kv heads, G = 4, us: rows kernel (with its cut) / 256-row kernel (128 rows at D = 256) uncut / cut
//   D 128  Tq 256: 2000 keys 20 / 44 / 29, 3100 25 / 63 / 33, 9000 58 / 165 / 47, 20000 115 / 356 / 83;
//          Tq 512: 3100 keys 45 / 64 / 41;  Tq 200, 40000 keys: 186 / 701 / 146
//   D 64   Tq 256: 3100 keys 18 / 47 / 24, 40000 135 / 523 / 98;  Tq 512: 3100 keys 30 / 47 / 31, 5000 42 / 72 / 38
//   D 256  Tq 256: 3100 keys 65 / 90 / 46, 9000 147 / 241 / 91;  Tq 512: 3100 keys 119 / 94 / 70;  Tq 700, G = 1, 9000 keys: 149 / 241 / 74
// Cuts of the rows kernel pay when they take off more than the combine launch (4 us, its gap and its launch on the
// host), and only up to one round of blocks.  One decoded token, 3100 keys, in one run / 13: D 64 15.4 / 12.3 us, D 128 20 / 13,
// D 256 55 / 19.
static inline AttnPlan attn_plan(const kvcomm_model &m, int n_ctx, int tq, bool may_split)
{
    const int G = m.n_q_heads / m.n_kv_heads, D = m.head_dim;
    const int64_t rows = (int64_t)G * tq, LH = (int64_t)m.n_layers * m.n_kv_heads, N = (int64_t)n_ctx + tq;

    const int tile_rows = D == 256 ? 128 : 32 * kAttnWaves;
    const int64_t tile_items = LH * ((rows + tile_rows - 1) / tile_rows), tiles = (N + 63) / 64;
    may_split = may_split && N >= kMinSplitKeys;
    int tile_ns = 1;
    const double one_run_us = attn_tiles_us(m, tile_items, tile_rows, tiles, 1);
    double tile_us = one_run_us;
    for (int ns = 2; may_split && tile_items <= 2 * kChipCUs && ns <= kTileMaxSplits && ns * kMinRunTiles <= tiles; ++ns) {
        const double t = attn_tiles_us(m, tile_items, tile_rows, tiles, ns);
        // The model is 8 ... 10 % (rms) off: near the line a cut has to promise more than that.  8 layers, Tq 64, 1000 keys, D = 64:
        // 20.5 us uncut, 24.8 in four runs (modelled 0.94); 9000 keys, Tq 700, D = 256: 249 us uncut, 266 in two (0.94).
        if (t < 0.95 * tile_us && t < (ns == 2 && D <= 128 ? 0.95 : 0.93) * one_run_us) {
            tile_us = t;
            tile_ns = ns;
        }
    }

    const int64_t rows_items = LH * ((rows + 31) / 32);
    const int64_t its = (N + 32 * rows_waves(D) - 1) / (32 * rows_waves(D));
    const double rows_one_run_us = attn_rows_us(m, rows_items, its);
    double rows_us = rows_one_run_us;
    int rows_ns = 1;
    if (may_split && rows_items <= kChipCUs / 2) {
        int64_t ns = std::min<int64_t>(std::min<int64_t>(kRowsMaxSplits, kChipCUs / rows_items), its);
        const int64_t split_its = (its + ns - 1) / ns;
        ns = (its + split_its - 1) / split_its;   // the fewest runs of that many iterations
        const double t = attn_rows_us(m, rows_items * ns, split_its);
        if (ns > 1 && rows_one_run_us - t > 8.0) {
            rows_us = t + 4.0;
            rows_ns = (int)ns;
        }
    }
    AttnPlan pl{};
    pl.rows_kernel = (rows_items <= kChipCUs && rows_us < 1.2 * tile_us) || rows_one_run_us < 0.7 * tile_us;
    // 16 rows per block where a tile has no more, and where those blocks, in the runs found for 32, all run at once.  Of 304 launches of 17 to 340
    // rows those of up to one round took 0.67 ... 0.94 of the time with 16 rows (one layer, 2064 keys, Tq 64 16.4 -> 13.4 us; 2 layers, 364 keys,
    // Tq 64 8.6 -> 6.9), all others 0.99 ... 1.65 (one layer, 3116 keys, Tq 16 11.5 and 13.4).
    const int64_t items16 = LH * ((rows + 15) / 16);
    const bool half = rows <= 16 || items16 * rows_ns <= kChipCUs;
    if (pl.rows_kernel && half && rows_ns == 1 && may_split && items16 <= kChipCUs / 4) {
        // Their cuts pay earlier: an iteration takes 0.9 us (D = 64: 0.6), the combine launch 3.3.  8 blocks, G = 4, D = 128, one run / the cut: 520
        // keys (3 iterations) 7.3 / 7.7 us, 1000 (4) 8.7 / 7.5 (1 block 8.3 / 7.8, 32 9.0 / 7.7, 64 9.5 / 9.0; 780 keys 7.1 / 7.7, 7.5 / 7.3, 7.7 / 7.6,
        // 7.8 / 7.9), 2000 (8) 12.8 / 8.2; 64 blocks, 1250 keys (5, in runs of two) 12.6 / 13.6, 2000 (in
        // runs of two) 16.9 / 16.2; D = 64, 8 blocks, 1000 keys 6.7 / 6.7, 1250 7.2 / 6.7; 64 blocks, 1250 keys 7.4 / 7.7, 1500 7.9 / 7.8.  More blocks
        // have the memory's rate already: 128 blocks, G = 2, 2000 keys, D = 128 22.0 / 26.0, D = 64 13.0 / 15.6.
        int64_t ns = std::min<int64_t>(std::min<int64_t>(kRowsMaxSplits, kChipCUs / items16), its);
        const int64_t split_its = (its + ns - 1) / ns;
        ns = (its + split_its - 1) / split_its;
        if (its - split_its >= (D == 128 && split_its == 1 ? 3 : 4)) rows_ns = (int)ns;   // iterations saved
    }
    pl.tile_rows = !pl.rows_kernel ? tile_rows : half ? 16 : 32;
    pl.group_rows = std::min(pl.tile_rows, 32);
    pl.n_row_tiles = (int)((rows + pl.tile_rows - 1) / pl.tile_rows);
    pl.n_splits = pl.rows_kernel ? rows_ns : tile_ns;
    return pl;
}

// (row group, split) pairs of a launch.
static inline size_t attn_parts(const kvcomm_model &m, const AttnPlan &pl)
{
    return (size_t)m.n_layers * m.n_kv_heads * pl.n_row_tiles * (pl.tile_rows / pl.group_rows) * pl.n_splits;
}

static inline size_t attn_workspace(const kvcomm_model &m, const AttnPlan &pl)
{
    return pl.n_splits > 1 ? attn_parts(m, pl) * sizeof(float) * (size_t)pl.group_rows * ((size_t)m.head_dim + 2) : 0;
}

// Groups of 16 packed rows of an fp32 block: one up to a block per compute unit, two above (they share what they load; the line is where the
// measured times cross, also at D = 64, where two blocks fit a unit).  us with
// one / two, 4 layers x 8 heads, G = 4: D = 128, 1056 keys, Tq 32 (256 blocks of one group) 44.5 / 49.8, 1088 keys, Tq 64 (512) 58.6 / 55.6; one
// layer, 1152 keys, Tq 128 (256) 34.8 / 52.5; 2 layers, 400 keys, Tq 100 (400) 26.0 / 25.4; D = 64, 540 keys, Tq 40 (320) 21.0 / 18.7; D = 256,
// 1056 keys, Tq 32 (256) 84 / 90, 1088 keys, Tq 64 (512) 118 / 97; but 128 keys, Tq 128, 4 layers x 4 heads, G = 8 (1024) 23.2 / 24.3.
// A row's sums do not depend on it, so a confined launch takes two where it has more groups than blocks (max_blocks; 0: not confined): one layer, D = 128,
// 1152 keys, Tq 128 (256 groups) on 160 / 64 / 8 blocks one by one 66.9 / 125 / 950, two at a time 51.2 / 98.8 / 743.
static inline int attn_f32_groups(const kvcomm_model &m, int tq, int max_blocks)
{
    const int64_t rows = (int64_t)(m.n_q_heads / m.n_kv_heads) * tq;
    const int64_t at_once = max_blocks > 0 && rows > 16 ? std::min(max_blocks, kChipCUs) : kChipCUs;
    return (int64_t)m.n_layers * m.n_kv_heads * ((rows + 15) / 16) <= at_once ? 1 : 2;
}

int launch_attn_rows(const AttnParams &p, int D, int rows, unsigned n_blocks, hipStream_t stream);
int launch_attn_f32(const AttnParams &p, int D, unsigned n_blocks, hipStream_t stream);
int launch_attn_combine(const AttnParams &p, int D, int rows, hipStream_t stream);   // rows: of a group of partial results

}  // namespace kvc
