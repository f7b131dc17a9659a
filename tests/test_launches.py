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
