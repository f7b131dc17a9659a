"""bf16 suffix attention of few rows on 16-row blocks: which launches take them, and their results against the float64 oracle (2e-2 as for all
bf16 attention outputs) at the edges of the 16 rows, the 32-key sub-steps, the wavefronts and the runs that the joining launch shares out
over its four wavefronts; the confined form bit for bit."""
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from launches import BF16, attention_launches
from parity import check_close, to_np

DEV = "cuda"
# L, Hkv, G, D, n_ctx, tq; rows of a block, runs
SHAPES = [((1, 1, 1, 64, 0, 1), 16, 1), ((2, 3, 4, 128, 28, 4), 16, 1), ((1, 2, 3, 256, 31, 5), 16, 1), ((1, 2, 17, 128, 257, 1), 16, 1),
          ((3, 5, 4, 64, 510, 9), 16, 1), ((1, 32, 4, 128, 300, 32), 16, 1), ((1, 33, 4, 128, 300, 32), 32, 1), ((19, 16, 2, 64, 70, 8), 16, 1),
          ((1, 1, 4, 128, 1300, 4), 16, 6), ((2, 8, 4, 128, 1000, 16), 16, 4), ((1, 8, 1, 64, 1000, 16), 16, 1), ((8, 8, 4, 64, 1200, 1), 16, 1), ((13, 5, 2, 64, 2000, 1), 16, 1), ((8, 8, 2, 64, 2000, 1), 16, 4), ((1, 2, 8, 64, 3000, 2), 16, 12), ((1, 8, 2, 128, 6200, 2), 16, 13), ((1, 3, 1, 256, 1500, 16), 16, 12),
          ((1, 8, 4, 128, 4000, 8), 16, 16), ((1, 8, 4, 128, 2000, 64), 16, 1), ((1, 8, 4, 128, 3100, 16), 32, 13)]


def test_which_launches_take_16_rows(tmp_path):
    for (s, rows, runs), r in zip(SHAPES, attention_launches(tmp_path, [s[:4] + (BF16,) + s[4:] + (0, True) for s, _, _ in SHAPES])):
        name, grid = r["launches"][0]
        assert r["status"] == 0 and len(r["launches"]) == (1 if runs == 1 else 2), (s, r)
        assert ("attn_rows_kernel16" if rows == 16 else "attn_rows_kernelI") in name, (s, name)
        assert grid[0] == s[0] * s[1] * -(-s[2] * s[5] // rows) * runs, (s, grid)
        if runs > 1:
            at_once = 4 if runs <= 4 else 8 if runs <= 8 else 16
            assert f"attn_combine_kernelILi{s[3]}ELi{at_once}ELi{rows}E" in r["launches"][1][0], (s, r)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,rows,runs", SHAPES)
def test_against_the_oracle(shape, rows, runs):
    L, hkv, G, D, n_ctx, tq = shape
    print(f"attn rows: {shape}", flush=True)
    m = kv.Model(L, hkv, hkv * G, D, torch.bfloat16, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV).to(torch.bfloat16)
    N = n_ctx + tq
    big_k, big_v = mk(hkv, N + 40), mk(hkv, N + 40)
    big_k[:, :, N:], big_v[:, :, N:] = float("nan"), float("nan")   # behind the cache's end
    q, k, v = mk(hkv * G, tq), big_k[:, :, :N], big_v[:, :, :N]
    ws = torch.full((max(kv.kvcomm_suffix_attn_workspace(m, n_ctx, tq), 16),), 0xFF, dtype=torch.uint8, device=DEV)
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True, workspace=ws)
    conf, lse_conf = kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 9, want_lse=True)
    torch.cuda.synchronize()
    want, want_lse = oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx, want_lse=True)
    check_close(to_np(out), want, torch.bfloat16, str(shape))
    assert float(abs(lse.cpu().numpy() - want_lse).max()) < 2e-2
    assert torch.equal(out, conf) and torch.equal(lse, lse_conf)
    # a key of NaN in a middle run: every query sees it
    if n_ctx > 3:
        k[:, -1, n_ctx // 2] = float("nan")
        bad, bad_lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
        torch.cuda.synchronize()
        assert torch.isnan(bad[:, -G:]).all() and torch.isnan(bad_lse[:, -G:]).all()
        assert torch.equal(bad[:, :-G], out[:, :-G])
