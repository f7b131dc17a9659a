"""What the attention calls launch (CPU only, see launches.py)."""
import pytest

from launches import BF16, F32, align_launches, attention_launches


@pytest.mark.parametrize("dtype,kernel", [(F32, "attn_f32_kernel"), (BF16, "attn_mfma_kernel"), (BF16, "attn_rows_kernel")])
@pytest.mark.parametrize("D", [64, 128, 256])
def test_confined_launches_keep_to_their_blocks(tmp_path, dtype, kernel, D):
    """Every kernel whose blocks fill a compute unit: at most max_blocks of them, and the plain launch has more."""
    shape = (1, 8, 4, D, dtype, 40, 64) if kernel != "attn_mfma_kernel" else (4, 8, 4, D, dtype, 100, 512)
    plain, *conf = attention_launches(tmp_path, [shape + (0, True)] + [shape + (n, True) for n in (8, 13, 60, 100000)])
    for n, r in zip((8, 13, 60, 100000), conf):
        (name, grid), (plain_name, plain_grid) = r["launches"][0], plain["launches"][0]
        assert r["status"] == 0 and kernel in name and kernel in plain_name
        assert grid == [min(n, plain_grid[0]), 1, 1] and plain_grid[0] > 60


def test_keys_are_cut_where_that_clearly_pays(tmp_path):
    """One layer of a long prompt is cut into runs; launches that would win a few percent by the model, which measured slower,
    are not: one launch, and no scratch asked for."""
    cut = [(1, 8, 4, 128, BF16, 2560, 512), (1, 8, 4, 128, BF16, 1500, 330), (1, 8, 4, 128, BF16, 3100, 1)]
    whole = [(8, 8, 4, 64, BF16, 936, 64), (1, 8, 4, 64, BF16, 488, 512), (1, 16, 2, 64, BF16, 530, 470),
             (1, 16, 2, 256, BF16, 8300, 700), (16, 8, 4, 256, BF16, 1168, 32)]
    for shape, r in zip(cut + whole, attention_launches(tmp_path, [s + (0, True) for s in cut + whole])):
        names = [n for n, _ in r["launches"]]
        assert r["status"] == 0 and len(names) == (2 if shape in cut else 1), (shape, names)
        assert (r["workspace"] > 0) == (shape in cut)
        assert ("attn_combine_kernel" in names[-1]) == (shape in cut)
    # runs of five 64-key tiles at least: 64 row tiles over 1200 keys make 128 blocks, not 256
    short, = attention_launches(tmp_path, [(1, 8, 4, 128, BF16, 688, 512, 0, True)])
    assert short["launches"][0][1] == [128, 1, 1]


# (L, Hkv, G, D, n_ctx, tq), kernel with scratch, kernel without, measured us of both (the other kernel's with its best cut)
KERNELS = [((1, 8, 4, 256, 2844, 256), "mfma", "rows"),     # 46 against 65
           ((1, 8, 4, 256, 8744, 256), "mfma", "rows"),     # 91 against 147
           ((1, 8, 1, 256, 8300, 700), "mfma", "rows"),     # 74 against 149
           ((1, 8, 4, 128, 19744, 256), "mfma", "rows"),    # 83 against 115
           ((1, 8, 4, 128, 39800, 200), "mfma", "rows"),    # 146 against 186
           ((1, 8, 4, 128, 2844, 256), "rows", "rows"),     # 25 against 33
           ((1, 8, 4, 64, 2844, 256), "rows", "rows"),      # 18 against 24
           ((1, 8, 4, 128, 3099, 1), "rows", "rows"),
           ((32, 8, 4, 128, 3099, 1), "rows", "rows"),
           ((1, 8, 4, 128, 2560, 512), "mfma", "rows"),
           ((32, 8, 4, 128, 2560, 512), "mfma", "mfma"),
           ((1, 2, 4, 128, 10, 2), "rows", "rows")]


def test_the_faster_kernel_is_taken(tmp_path):
    res = attention_launches(tmp_path, [k[0][:4] + (BF16,) + k[0][4:] + (0, ws) for k in KERNELS for ws in (True, False)])
    for (shape, *want), with_ws, without in zip(KERNELS, res[::2], res[1::2]):
        for r, kernel in zip((with_ws, without), want):
            assert r["status"] == 0 and f"attn_{kernel}_kernel" in r["launches"][0][0], (shape, kernel, r)
        assert len(without["launches"]) == 1


def test_the_shapes_of_the_gpu_tests_reach_what_they_name(tmp_path):
    from test_gpu_attn_kernels import TILES
    from test_gpu_attn_split import SHAPES
    rows = attention_launches(tmp_path, [s[:4] + (BF16,) + s[4:6] + (0, True) for s in SHAPES])
    for s, r in zip(SHAPES, rows):
        kernel = "attn_mfma_kernel" if "-row tiles" in s[6] else "attn_rows_kernel"
        assert kernel in r["launches"][0][0], (s, r)
    for s, r in zip(TILES, attention_launches(tmp_path, [s[:4] + (BF16,) + s[4:] + (0, True) for s in TILES])):
        assert "attn_mfma_kernel" in r["launches"][0][0], (s, r)
    for s, nt in (((32, 8, 4, 128, 3100, 1), True), ((1, 8, 4, 128, 3100, 1), False)):
        r, = attention_launches(tmp_path, [s[:4] + (BF16,) + s[4:] + (0, True)])
        assert ("ELb1E" in r["launches"][0][0]) == nt and "attn_rows_kernel" in r["launches"][0][0]


@pytest.mark.parametrize("L,H,D,dtype,lens,pools,rows", [(32, 8, 128, BF16, [512] * 4, [8] * 4, 32), (1, 1, 64, F32, [1], [0], 32),
                                                         (80, 8, 128, BF16, [1 << 20], [1], 32), (257, 8, 256, F32, [300000], [1], 8),
                                                         (4000, 8, 64, BF16, [1 << 17, 5], [1, 1], 64)])
def test_updates_of_any_size_stay_within_a_launch(tmp_path, L, H, D, dtype, lens, pools, rows):
    """A launch holds fewer than 2^32 threads along each axis.  Every (layer, head, token tile, tensor) has its block."""
    r, = align_launches(tmp_path, [(L, H, D, dtype, lens, pools, None)])
    assert r["status"] == 0 and len(r["launches"]) == 1
    (x, y, z), (threads, _, _) = r["launches"][0]["grid"], r["launches"][0]["block"]
    assert threads == 256 and x * threads < 1 << 32 and y <= 65535 and z == 1
    tiles = sum(-(-S // rows) for S in lens)
    pairs, left = divmod(x, tiles)
    assert left == 0 and pairs * (y // 2 - 1) < L * H <= pairs * (y // 2) and y % 2 == 0


def test_blocks_per_unit_of_an_update(tmp_path):
    """The LDS that a launch reserves bounds its blocks per compute unit (160 KB): two for large launches of large pools, three for
    others from 0.45 GB on, no bound below; beside other work, on a part of the units, more of them, until the bound goes."""
    big, few, mid, small, narrow = ((32, 8, 128, BF16, [512] * 4, [8] * 4), (32, 8, 128, BF16, [512] * 4, [4] * 4), (32, 8, 128, BF16, [512], [8]),
                                    (32, 8, 128, BF16, [77], [6]), (32, 8, 64, BF16, [512] * 8, [8] * 8))
    want = [(big, None, 2), (few, None, 3), (mid, None, 3), (small, None, 0), (narrow, None, 3), (big, 256, 2), (big, 112, 2), (big, 96, 3),
            (mid, 96, 3), (big, 88, 0), (big, 1, 0), (small, 96, 0)]
    for (shape, units, blocks), r in zip(want, align_launches(tmp_path, [s + (u,) for s, u, _ in want])):
        lds = r["launches"][0]["lds"]
        assert r["status"] == 0 and (lds < 32768 if blocks == 0 else 163840 // lds == blocks), (shape, units, lds)
    assert [r["status"] for r in align_launches(tmp_path, [small + (u,) for u in (0, -3)])] == [-1, -1]


def test_anchors_in_flight_of_an_update(tmp_path):
    """Four where few rows are moved (by one round of blocks, or for pools of 32 and more) and every segment has four, two elsewhere."""
    want = [((2, 3, 64, BF16, [70], [9]), True), ((2, 3, 64, BF16, [70], [3]), False), ((2, 3, 64, BF16, [70, 20], [9, 3]), False),
            ((32, 8, 128, BF16, [8], [4]), True), ((32, 8, 128, BF16, [33], [8]), False), ((80, 8, 128, BF16, [3], [8]), False),
            ((80, 8, 128, BF16, [3], [48]), True), ((80, 8, 128, BF16, [20], [48]), False), ((32, 8, 128, BF16, [512] * 4, [8] * 4), False)]
    for (shape, four), r in zip(want, align_launches(tmp_path, [s + (None,) for s, _ in want])):
        assert r["status"] == 0 and ("ELb1E" in r["launches"][0]["name"]) == four, (shape, r)
