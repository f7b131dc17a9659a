"""Suffix attention of small launches: the rows kernel (few packed query rows, keys shared out over the wavefronts of a
block) and the launches whose key axis is cut into runs that a second kernel joins.  Against the float64 oracle, at the
edges of the 32-key sub-steps, 64-key tiles and 32-row groups, with and without a workspace, and the persistent form.

Tolerance: as for every bf16 attention output (max-abs 2e-2; the probabilities are rounded to bf16, relative 2^-9,
and the output once more).  Log-sum-exp: 2e-2 as in the other attention tests; split and unsplit agree to 1e-4 (both
sum unrounded fp32 exponentials)."""
import ctypes

import pytest
import torch

import oracle
import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding

from parity import check_close, to_np

DEV = "cuda"


def _model(L, hkv, G, D, dtype=torch.bfloat16):
    return kv.Model(L, hkv, hkv * G, D, dtype, 5e5)


# (L, Hkv, G, D, n_ctx, tq, what the plan is expected to do)
SHAPES = [
    (1, 1, 4, 128, 0, 1, "one key"),
    (1, 2, 1, 128, 31, 1, "one sub-step"),
    (1, 2, 4, 128, 32, 3, "second sub-step of one or two keys"),
    (2, 2, 8, 64, 63, 4, "32 rows exactly"),
    (1, 2, 3, 128, 255, 11, "33 rows, 3 heads a group"),
    (1, 1, 1, 256, 300, 70, "head dimension 256"),
    (1, 8, 4, 128, 3100, 1, "rows, split"),
    (1, 2, 4, 128, 4095, 9, "rows, split, two row tiles, causal edge inside the last run"),
    (1, 2, 2, 64, 6000, 40, "rows, split, queries that see nothing of the last sub-step"),
    (1, 4, 4, 256, 2050, 2, "rows, split, head dimension 256"),
    (1, 8, 4, 128, 1500, 330, "256-row tiles, split, a tile that is not full"),
    (1, 16, 1, 64, 700, 600, "256-row tiles, split, 256 queries a tile"),
    (1, 2, 8, 128, 0, 1000, "256-row tiles, short and long row tiles, runs that are empty"),
    (1, 8, 4, 256, 1100, 260, "128-row tiles, split"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("L,hkv,G,D,n_ctx,tq,what", SHAPES, ids=[s[-1] for s in SHAPES])
def test_small_launches_against_oracle(L, hkv, G, D, n_ctx, tq, what):
    print(f"attn split: L{L} Hkv{hkv} G{G} D{D} n_ctx{n_ctx} tq{tq}", flush=True)
    m = _model(L, hkv, G, D)
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV).to(torch.bfloat16)
    N = n_ctx + tq
    # the cache is a view into a larger one: rows behind its end hold NaN and must not reach the result
    big_k, big_v = mk(hkv, N + 40), mk(hkv, N + 40)
    big_k[:, :, N:], big_v[:, :, N:] = float("nan"), float("nan")
    q, k, v = mk(hkv * G, tq), big_k[:, :, :N], big_v[:, :, :N]
    need = kv.kvcomm_suffix_attn_workspace(m, n_ctx, tq)
    assert (need > 0) == ("split" in what or "runs" in what), need
    # a workspace that held something else, and one byte too few
    ws = torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device=DEV)
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True, workspace=ws)
    out_own, lse_own = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    plain, lse_plain = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True, workspace=ws[:max(need, 16) - 1])
    conf, lse_conf = kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 11, want_lse=True)
    conf_plain, _ = kv.kvcomm_suffix_attn_confined_ws(m, q, k, v, n_ctx, 11, want_lse=True, workspace=ws[:0])
    torch.cuda.synchronize()
    want, want_lse = oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx, want_lse=True)
    for o, s in ((out, lse), (plain, lse_plain)):
        check_close(to_np(o), want, torch.bfloat16, what)
        assert float(abs(s.cpu().numpy() - want_lse).max()) < 2e-2
    assert torch.equal(out, out_own) and torch.equal(lse, lse_own)
    assert torch.equal(out, conf) and torch.equal(lse, lse_conf)
    assert torch.equal(plain, conf_plain)
    assert float((lse - lse_plain).abs().max()) < 1e-4


@pytest.mark.gpu
def test_split_on_another_stream_and_large_scores():
    """Own scratch on a stream that is not the current one, and scores far beyond the range of one reference."""
    m = _model(1, 2, 4, 128)
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    mk = lambda h, n, s=1.0: (torch.randn((1, h, n, 128), generator=g, device=DEV) * s).to(torch.bfloat16)
    n_ctx, tq = 5000, 3
    q, k, v = mk(8, tq, 12.0), mk(2, n_ctx + tq, 12.0), mk(2, n_ctx + tq)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out = torch.empty_like(q)
    kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, out=out, stream=side)
    side.synchronize()
    check_close(to_np(out), oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx), torch.bfloat16, "large scores")


@pytest.mark.gpu
@pytest.mark.parametrize("n_ctx,tq,dtype", [(3100, 1, torch.bfloat16), (1500, 330, torch.bfloat16), (900, 3, torch.float32)])
def test_nan_reaches_every_query_that_sees_it(n_ctx, tq, dtype):
    """NaN keys that fill whole runs (and whole wavefronts' sub-steps), and a NaN query: the affected outputs are NaN and
    no others, as if one block had walked the keys."""
    print(f"attn NaN: n_ctx{n_ctx} tq{tq} {dtype}", flush=True)
    m = _model(1, 8, 4, 128, dtype)
    g = torch.Generator(device=DEV)
    g.manual_seed(tq)
    mk = lambda h, n: torch.randn((1, h, n, 128), generator=g, device=DEV).to(dtype)
    q, k, v = mk(32, tq), mk(8, n_ctx + tq), mk(8, n_ctx + tq)
    good = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx)
    kn, qn = k.clone(), q.clone()
    kn[:, 3, 256:n_ctx - 200] = float("nan")     # kv head 3: query heads 12 ... 15
    qn[:, 21, tq - 1] = float("nan")
    got, lse = kv.kvcomm_suffix_attn(m, q, kn, v, n_ctx, want_lse=True)
    got_q = kv.kvcomm_suffix_attn(m, qn, k, v, n_ctx)
    torch.cuda.synchronize()
    assert torch.isnan(got[:, 12:16]).all() and torch.isnan(lse[:, 12:16]).all()
    assert torch.equal(got[:, :12], good[:, :12]) and torch.equal(got[:, 16:], good[:, 16:])
    assert torch.isnan(got_q[:, 21, tq - 1]).all()
    keep = torch.ones(good.shape[:3], dtype=torch.bool, device=DEV)
    keep[:, 21, tq - 1] = False
    # The 256-row kernel re-references all rows of the wavefront that holds the NaN query: its neighbours' probabilities
    # round differently (relative 2^-9 each, |v| < 5: below 2^-8 * 5 = 2e-2).
    assert float((got_q[keep].float() - good[keep].float()).abs().max()) < 2e-2


@pytest.mark.gpu
@pytest.mark.parametrize("n_ctx,tq", [(3100, 1), (1500, 330)])
def test_split_launches_in_a_graph(n_ctx, tq):
    """Both kinds of split launch, their scratch made during the capture: every replay, with new inputs in place and eager
    calls (which use scratch of their own) between the replays, equals the eager result bit for bit."""
    print(f"attn split in a graph: n_ctx{n_ctx} tq{tq}", flush=True)
    m = _model(1, 8, 4, 128)
    assert kv.kvcomm_suffix_attn_workspace(m, n_ctx, tq) > 0
    g = torch.Generator(device=DEV)
    g.manual_seed(tq)
    mk = lambda h, n: torch.randn((1, h, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = mk(32, tq), mk(8, n_ctx + tq), mk(8, n_ctx + tq)
    out, eager = torch.empty_like(q), torch.empty_like(q)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, out=out)
    for _ in range(3):
        for t, h, n in ((q, 32, tq), (k, 8, n_ctx + tq), (v, 8, n_ctx + tq)):
            t.copy_(mk(h, n))
        kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, out=eager)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)


def test_workspace_query():
    lib = binding.load_library()
    q = lambda m, n_ctx, tq: lib.kvcomm_suffix_attn_workspace(ctypes.byref(m.c()), n_ctx, tq)
    layer = _model(1, 8, 4, 128)
    assert q(layer, 3100, 1) > 0 and q(layer, 2560, 512) > 0
    # nothing to split: short caches, launches that fill the chip, fp32, bad arguments
    assert q(layer, binding.ATTN_MIN_SPLIT_KEYS - 2, 1) == 0
    assert q(_model(32, 8, 4, 128), 3100, 1) == 0 and q(_model(32, 8, 4, 128), 2560, 512) == 0
    assert q(_model(1, 8, 4, 128, torch.float32), 3100, 1) == 0
    assert q(layer, -1, 1) == 0 and q(layer, 10, 0) == 0 and q(_model(1, 8, 4, 96), 3100, 1) == 0
    for L in (1, 2, 4):     # bounded: never more than 16 partial results of the rows of two full rounds of blocks
        for tq in (1, 7, 64, 500, 1024):
            for n_ctx in (512, 3000, 131072):
                assert q(_model(L, 8, 8, 256), n_ctx, tq) <= 2 * 256 * 256 * 16 * 4 * (256 + 2)


# fp32: both kernels (up to 8 keys, 16 at D = 256, and beyond), around the 16-key sub-steps and the tiles of 16 and 32 rows, every head dimension
F32_SHAPES = [(1, 1, 1, 64, 0, 1), (2, 2, 2, 128, 60, 4), (2, 2, 2, 128, 60, 5), (1, 2, 4, 64, 95, 8), (1, 2, 3, 256, 96, 11),
              (1, 1, 8, 256, 300, 33), (2, 1, 1, 64, 1000, 65), (1, 2, 8, 128, 0, 70)]


@pytest.mark.gpu
@pytest.mark.parametrize("L,hkv,G,D,n_ctx,tq", F32_SHAPES)
def test_f32_attention(L, hkv, G, D, n_ctx, tq):
    """1e-5 as for every fp32 output.  Rows behind the cache's end hold NaN.  Then values of the later suffix tokens
    that are not finite: they reach the queries that see them and no other."""
    print(f"f32 attn: L{L} Hkv{hkv} G{G} D{D} n_ctx{n_ctx} tq{tq}", flush=True)
    m = _model(L, hkv, G, D, torch.float32)
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV)
    N = n_ctx + tq
    big_k, big_v = mk(hkv, N + 40), mk(hkv, N + 40)
    big_k[:, :, N:], big_v[:, :, N:] = float("nan"), float("nan")
    q, k, v = mk(hkv * G, tq), big_k[:, :, :N], big_v[:, :, :N]
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    torch.cuda.synchronize()
    want, want_lse = oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx, want_lse=True)
    check_close(to_np(out), want, torch.float32, "O")
    assert float(abs(lse.cpu().numpy() - want_lse).max()) < 1e-4
    if tq < 4:
        return
    first = tq // 2    # queries 0 ... first - 1 do not see it
    v[:, :, n_ctx + first, 1], v[:, :, n_ctx + first, D - 1] = float("inf"), float("nan")
    v[:, :, n_ctx + tq - 1, 1] = -float("inf")
    bad = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx)
    torch.cuda.synchronize()
    assert torch.equal(bad[:, :, :first], out[:, :, :first])
    seen = bad[:, :, first:]
    assert (seen[:, :, :-1, 1] == float("inf")).all() and torch.isnan(seen[:, :, -1, 1]).all()
    assert torch.isnan(seen[..., D - 1]).all()
    assert torch.isfinite(seen[..., 2:D - 1]).all() and torch.isfinite(seen[..., 0]).all()
