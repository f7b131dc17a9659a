"""fp32 suffix attention: both kernels (up to 8 keys, 16 at D = 256, and beyond) and both row tiles of the second one (16 rows up to a block per compute unit, 32
above), at the edges of the 16-key sub-steps, the eight wavefronts and the 16-row groups.  Against the float64 oracle, 1e-5 as for
every fp32 output; the confined form bit for bit; values that are not finite at the causal edge reach the queries that see them."""
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from launches import F32, attention_launches
from parity import check_close, to_np

DEV = "cuda"
# L, Hkv, G, D, n_ctx, tq; groups of 16 rows per block (0: the kernel of short caches)
SHAPES = [((2, 3, 2, 64, 5, 3), 0), ((1, 2, 8, 256, 15, 1), 0), ((1, 1, 4, 128, 8, 1), 1), ((1, 1, 2, 256, 14, 3), 1), ((1, 2, 4, 64, 15, 1), 1), ((2, 2, 3, 128, 16, 11), 1),
          ((1, 2, 1, 256, 113, 15), 1), ((1, 2, 4, 128, 125, 4), 1), ((1, 8, 4, 64, 300, 128), 1), ((1, 8, 4, 64, 300, 129), 2),
          ((1, 17, 8, 128, 40, 33), 2), ((2, 16, 4, 256, 2, 35), 2), ((3, 16, 3, 64, 0, 39), 2), ((3, 12, 1, 128, 130, 150), 2)]


def test_the_shapes_reach_what_they_name(tmp_path):
    for (s, groups), r in zip(SHAPES, attention_launches(tmp_path, [s[:4] + (F32,) + s[4:] + (0, True) for s, _ in SHAPES])):
        (name, grid), = r["launches"]
        assert r["status"] == 0 and r["workspace"] == 0
        L, hkv, G, D, _, tq = s
        if groups:
            assert f"attn_f32_kernelILi{D}ELi{groups}ELb0E" in name and grid == [L * hkv * -(-G * tq // (16 * groups)), 1, 1], (s, name, grid)
        else:
            assert "attn_f32_row_kernel" in name, (s, name)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,groups", SHAPES)
def test_against_the_oracle(shape, groups):
    L, hkv, G, D, n_ctx, tq = shape
    print(f"f32 attn: {shape}", flush=True)
    m = kv.Model(L, hkv, hkv * G, D, torch.float32, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV)
    N = n_ctx + tq
    big_k, big_v = mk(hkv, N + 20), mk(hkv, N + 20)
    big_k[:, :, N:], big_v[:, :, N:] = float("nan"), float("nan")   # behind the cache's end
    q, k, v = mk(hkv * G, tq), big_k[:, :, :N], big_v[:, :, :N]
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    conf, lse_conf = kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 11, want_lse=True)
    torch.cuda.synchronize()
    want, want_lse = oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx, want_lse=True)
    check_close(to_np(out), want, torch.float32, str(shape))
    assert float(abs(lse.cpu().numpy() - want_lse).max()) < 1e-4
    assert torch.equal(out, conf) and torch.equal(lse, lse_conf)
    if tq < 3 or not groups:
        return
    first = tq // 2    # queries before it do not see it
    v[:, -1, n_ctx + first, D - 2], v[:, -1, n_ctx + first, 0] = float("inf"), float("nan")
    bad = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx)
    torch.cuda.synchronize()
    assert torch.equal(bad[:, :, :first], out[:, :, :first]) and torch.equal(bad[:, :-G], out[:, :-G])
    seen = bad[:, -G:, first:]
    assert (seen[..., D - 2] == float("inf")).all() and torch.isnan(seen[..., 0]).all() and torch.isfinite(seen[..., 1:D - 2]).all()
