"""What the attention calls launch (CPU only, see launches.py)."""
import pytest

from launches import attention_launches

F32, BF16 = 0, 1


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
