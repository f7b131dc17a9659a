"""The bf16 attention kernels that only some launches reach, each at a shape that does: the rows kernel's non-temporal form
(one row tile over a cache beyond the last-level cache) and the 256-row kernel (128 rows at D = 256) at every head dimension,
with and without split keys, with scores that leave the range of one softmax reference."""
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from parity import check_close, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("D,n_ctx", [(128, 3100), (64, 4220), (256, 1090)])
def test_rows_kernel_beyond_the_last_level_cache(D, n_ctx):
    """One decoded token, 32 layers x 8 kv heads in one launch (more than 256 MB of K and V): a few (layer, head) pairs against
    the oracle (bf16 tolerance), and all of them bit for bit against per-layer calls, whose caches fit."""
    print(f"rows kernel, non-temporal: D{D} n_ctx{n_ctx}", flush=True)
    L, hkv, G, tq = 32, 8, 4, 1
    assert L * hkv * (n_ctx + tq) * D * 4 > 256 << 20
    m, layer = (kv.Model(n, hkv, hkv * G, D, torch.bfloat16, 5e5) for n in (L, 1))
    g = torch.Generator(device=DEV)
    g.manual_seed(D)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = mk(hkv * G, tq), mk(hkv, n_ctx + tq), mk(hkv, n_ctx + tq)
    none = torch.empty((0,), dtype=torch.uint8, device=DEV)
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    for l in range(L):
        o, s = kv.kvcomm_suffix_attn(layer, q[l:l + 1], k[l:l + 1], v[l:l + 1], n_ctx, want_lse=True, workspace=none)
        torch.cuda.synchronize()
        assert torch.equal(o[0], out[l]) and torch.equal(s[0], lse[l]), l
    for l, hq in ((0, 0), (13, 17), (L - 1, hkv * G - 1)):
        want = oracle.suffix_attn(to_np(q[l:l + 1, hq:hq + 1]), to_np(k[l:l + 1, hq // G:hq // G + 1]),
                                  to_np(v[l:l + 1, hq // G:hq // G + 1]), n_ctx)
        check_close(to_np(out[l:l + 1, hq:hq + 1]), want, torch.bfloat16, f"layer {l} head {hq}")


# L, Hkv, G, D, n_ctx, tq: launches that the 256-row kernel takes without split keys whatever the workspace (the short
# ones), and some whose keys are split
TILES = [(6, 2, 4, 128, 0, 512), (6, 2, 4, 128, 40, 449), (9, 2, 2, 64, 100, 1000), (9, 2, 2, 64, 0, 513), (9, 2, 2, 256, 70, 700),
         (9, 2, 2, 256, 0, 513), (1, 8, 4, 128, 1500, 330), (1, 16, 1, 64, 1700, 600), (1, 8, 4, 256, 1100, 260)]


@pytest.mark.parametrize("L,hkv,G,D,n_ctx,tq", TILES)
@pytest.mark.parametrize("grow", [1.0, 14.0], ids=["scores", "large_scores"])
def test_256_row_kernel(L, hkv, G, D, n_ctx, tq, grow):
    print(f"256-row kernel: L{L} Hkv{hkv} G{G} D{D} n_ctx{n_ctx} tq{tq} x{grow}", flush=True)
    m = kv.Model(L, hkv, hkv * G, D, torch.bfloat16, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(tq)
    mk = lambda h, n, s=1.0: (torch.randn((L, h, n, D), generator=g, device=DEV) * s).to(torch.bfloat16)
    q, k, v = mk(hkv * G, tq, grow), mk(hkv, n_ctx + tq), mk(hkv, n_ctx + tq, 0.5)
    k[:, :, (n_ctx + tq) // 2:] *= 3.0      # the scores grow along the cache: later keys move the reference
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    conf, lse_conf = kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 24, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out, conf) and torch.equal(lse, lse_conf)
    for l, hq in ((0, 0), (L - 1, hkv * G - 1)):
        pick = lambda x, h: to_np(x[l:l + 1, h:h + 1])
        want, want_lse = oracle.suffix_attn(pick(q, hq), pick(k, hq // G), pick(v, hq // G), n_ctx, want_lse=True)
        check_close(pick(out, hq), want, torch.bfloat16, f"layer {l} head {hq}")
        assert abs(pick(lse, hq) - want_lse).max() < 2e-2


@pytest.mark.parametrize("max_blocks", [8, 13])
@pytest.mark.parametrize("L,hkv,G,D,n_ctx,tq", [(2, 4, 2, 64, 60, 45), (1, 8, 4, 128, 300, 33), (2, 2, 4, 256, 500, 40)])
def test_f32_confined(L, hkv, G, D, n_ctx, tq, max_blocks):
    """Several items per block: the same bits as the plain launch, values that are not finite at the causal edge included."""
    print(f"f32 confined: L{L} Hkv{hkv} G{G} D{D} n_ctx{n_ctx} tq{tq} max_blocks{max_blocks}", flush=True)
    m = kv.Model(L, hkv, hkv * G, D, torch.float32, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV)
    q, k, v = mk(hkv * G, tq), mk(hkv, n_ctx + tq), mk(hkv, n_ctx + tq)
    v[:, 1, n_ctx + tq // 2, 3] = float("inf")
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    conf, lse_conf = kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, max_blocks, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out, conf) and torch.equal(lse, lse_conf)
    want = oracle.suffix_attn(to_np(q[:, :G]), to_np(k[:, :1]), to_np(v[:, :1]), n_ctx)
    check_close(to_np(conf[:, :G]), want, torch.float32, "O")
