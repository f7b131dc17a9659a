"""Keys whose scores are minus infinity (a channel of -inf as a mask) count as weight 0 wherever they lie: in particular where
they fill the first keys of a run of a launch whose key axis is split, which every run takes its softmax reference from.
Against the float64 oracle, tolerance as for every bf16 / fp32 attention output, with and without a workspace."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from parity import check_close, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"

SHAPES = [  # L, Hkv, G, D, n_ctx, tq, dtype: kernel
    (1, 8, 4, 128, 2560, 512, torch.bfloat16),   # 256-row tiles, split
    (1, 16, 1, 64, 1700, 600, torch.bfloat16),   # the same, D = 64
    (1, 8, 4, 256, 1100, 260, torch.bfloat16),   # 128-row tiles, split
    (4, 8, 4, 128, 1100, 512, torch.bfloat16),   # 256-row tiles, one block per row tile
    (1, 8, 4, 128, 3100, 1, torch.bfloat16),     # rows kernel, split
    (1, 2, 4, 128, 300, 9, torch.bfloat16),      # rows kernel
    (1, 2, 4, 128, 900, 40, torch.float32),
]


def _inputs(L, hkv, G, D, n_ctx, tq, dtype):
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV)
    q, k, v = mk(hkv * G, tq), mk(hkv, n_ctx + tq), mk(hkv, n_ctx + tq)
    q[..., 5] = 1.0      # the masking channel: a key with -inf there scores -inf with every query
    return q.to(dtype), k.to(dtype), v.to(dtype)


def _masks(n_ctx):
    """(name, bool[n_ctx]) of context tokens to hide."""
    t = torch.arange(n_ctx, device=DEV)
    return [("everything between the first 32 keys and the suffix", t >= 32),
            ("every other 64-key tile", (t // 64) % 2 == 1),
            ("the first half of every tile but the first", (t % 64 < 32) & (t >= 64)),
            ("the first 100 keys", t < 100)]


@pytest.mark.parametrize("L,hkv,G,D,n_ctx,tq,dtype", SHAPES)
def test_masked_keys(L, hkv, G, D, n_ctx, tq, dtype):
    m = kv.Model(L, hkv, hkv * G, D, dtype, 5e5)
    q, k, v = _inputs(L, hkv, G, D, n_ctx, tq, dtype)
    none = torch.empty((0,), dtype=torch.uint8, device=DEV)
    for name, mask in _masks(n_ctx):
        print(f"-inf scores: L{L} D{D} n_ctx{n_ctx} tq{tq} {dtype}: {name}", flush=True)
        kk = k.clone()
        kk[:, :, :n_ctx, 5][:, :, mask] = -float("inf")
        heads = [0, hkv * G - 1]     # (query heads compared with the oracle; the others follow from the same code)
        out, lse = kv.kvcomm_suffix_attn(m, q, kk, v, n_ctx, want_lse=True)
        plain, lse_plain = kv.kvcomm_suffix_attn(m, q, kk, v, n_ctx, want_lse=True, workspace=none)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all() and torch.isfinite(plain).all(), name
        assert torch.isfinite(lse).all() and torch.isfinite(lse_plain).all(), name
        for hq in heads:
            pick = lambda x, h: to_np(x[L - 1:, h:h + 1])
            want, want_lse = oracle.suffix_attn(pick(q, hq), pick(kk, hq // G), pick(v, hq // G), n_ctx, want_lse=True)
            for o, s in ((out, lse), (plain, lse_plain)):
                check_close(pick(o, hq), want, dtype, name)
                assert np.abs(pick(s, hq) - want_lse).max() < (1e-4 if dtype == torch.float32 else 2e-2)


@pytest.mark.parametrize("L,hkv,G,D,n_ctx,tq,dtype", SHAPES)
def test_a_query_without_any_finite_score(L, hkv, G, D, n_ctx, tq, dtype):
    """All keys of one kv head hidden: 0 / 0 for its queries (NaN, log-sum-exp -inf) and nothing for the others."""
    print(f"-inf scores, all of them: L{L} D{D} n_ctx{n_ctx} tq{tq} {dtype}", flush=True)
    m = kv.Model(L, hkv, hkv * G, D, dtype, 5e5)
    q, k, v = _inputs(L, hkv, G, D, n_ctx, tq, dtype)
    good, good_lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    k[:, 1, :, 5] = -float("inf")
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    torch.cuda.synchronize()
    assert torch.isnan(out[:, G:2 * G]).all() and (lse[:, G:2 * G] == -float("inf")).all()
    assert torch.equal(out[:, :G], good[:, :G]) and torch.equal(out[:, 2 * G:], good[:, 2 * G:])
    assert torch.equal(lse[:, :G], good_lse[:, :G])
