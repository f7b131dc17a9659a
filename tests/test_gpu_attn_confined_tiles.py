"""Confined attention of launches whose plain form has tiles of 16 rows: with more tiles than blocks two of a (layer, kv head) go together, so
that the blocks walk no more rounds than tiles of 32 rows would take; bit for bit the plain launch's results, with and without cut keys, also where the
runs of the two tiles begin at different keys, and where the last tile has no partner."""
import pytest
import torch

import paper_2510_12872_amd as kv

from launches import BF16, F32, attention_launches

DEV = "cuda"
# dtype, L, Hkv, G, D, n_ctx, tq; runs
SHAPES = [(BF16, (2, 8, 4, 128, 300, 64), 1), (BF16, (1, 8, 4, 64, 333, 100), 1), (BF16, (1, 3, 1, 256, 450, 49), 1), (BF16, (1, 5, 1, 64, 1480, 37), 6),
          (BF16, (1, 2, 1, 128, 1480, 40), 6), (BF16, (1, 2, 2, 128, 1495, 20), 6), (BF16, (1, 2, 1, 256, 6120, 33), 13), (BF16, (1, 8, 4, 128, 0, 20), 1),
          (F32, (2, 8, 4, 64, 130, 60), 1), (F32, (1, 3, 1, 128, 250, 49), 1), (F32, (1, 2, 3, 256, 7, 40), 1), (F32, (1, 8, 4, 128, 0, 21), 1)]


def _tiles(shape, rows):
    L, hkv, G, _, _, tq = shape
    return L * hkv * -(-G * tq // rows)


def test_rounds_of_confined_launches(tmp_path):
    for dtype, s, runs in SHAPES:
        blocks = sorted({8, 9, 13, 64, 160, _tiles(s, 16) * runs - 1, _tiles(s, 16) * runs, _tiles(s, 16) * runs + 1} - set(range(8)))
        plain, *conf = attention_launches(tmp_path, [s[:4] + (dtype,) + s[4:] + (n, True) for n in [0] + blocks])
        assert plain["status"] == 0 and len(plain["launches"]) == (1 if runs == 1 else 2), (s, plain)
        assert plain["launches"][0][1] == [_tiles(s, 16) * runs, 1, 1], (s, plain)
        for n, r in zip(blocks, conf):
            name, grid = r["launches"][0]
            pairs = n < _tiles(s, 16) * runs
            if dtype == BF16:
                assert f"attn_rows_kernel16ILi{s[3]}ELb0ELb{int(pairs)}ELi{1 + pairs}E" in name, (s, n, name)
            else:
                assert f"attn_f32_kernelILi{s[3]}ELi{1 + pairs}E" in name, (s, n, name)
            assert grid == [min(n, _tiles(s, 32 if pairs else 16) * runs), 1, 1], (s, n, grid)
            assert r["launches"][1:] == plain["launches"][1:]
    # one tile of a (layer, kv head) has no partner
    for dtype, name in ((BF16, "attn_rows_kernel16ILi128ELb0ELb1ELi1E"), (F32, "attn_f32_kernelILi128ELi1ELb1E")):
        r, = attention_launches(tmp_path, [(4, 8, 4, 128, dtype, 100, 4, 13, True)])
        assert name in r["launches"][0][0] and r["launches"][0][1] == [13, 1, 1], r


def test_runs_that_begin_at_different_keys():
    """(SHAPES holds pairs of tiles with a cut between the begins of their runs: s * units / runs.)"""
    apart = 0
    for dtype, (L, hkv, G, D, n_ctx, tq), runs in SHAPES:
        units = [(n_ctx + min(tq - 1, (16 * t + 15) // G) + 32) // 32 for t in range(-(-G * tq // 16))]
        for a, b in zip(units[::2], units[1::2]):
            assert 0 <= b - a <= 1
            apart += sum(s * a // runs != s * b // runs for s in range(runs))
    assert apart > 10


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape,runs", SHAPES)
def test_the_plain_launch_bit_for_bit(dtype, shape, runs):
    L, hkv, G, D, n_ctx, tq = shape
    print(f"confined tiles: {dtype} {shape}", flush=True)
    t = torch.bfloat16 if dtype == BF16 else torch.float32
    m = kv.Model(L, hkv, hkv * G, D, t, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV).to(t)
    N = n_ctx + tq
    q, k, v = mk(hkv * G, tq), mk(hkv, N), mk(hkv, N)
    ws = torch.full((max(kv.kvcomm_suffix_attn_workspace(m, n_ctx, tq), 16),), 0xFF, dtype=torch.uint8, device=DEV)
    for scratch in (ws, ws[:0]):
        out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True, workspace=scratch)
        for n in (8, 13, 64):
            ws.fill_(0xFF)
            conf, lse_conf = kv.kvcomm_suffix_attn_confined_ws(m, q, k, v, n_ctx, n, want_lse=True, workspace=scratch)
            torch.cuda.synchronize()
            assert torch.isfinite(out).all() and torch.equal(out, conf) and torch.equal(lse, lse_conf), n
