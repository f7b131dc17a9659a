"""The launch that joins split keys: every number of partial results it is compiled for, behind both kernels, with block counts that
do not divide by the eight XCDs.  Against the float64 oracle (bf16: 2e-2 as for all attention outputs), bit for bit between the plain
and the confined launch of the first kernel."""
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from launches import attention_launches
from parity import check_close, to_np

DEV = "cuda"
# L, Hkv, G, D, n_ctx, tq; kernel in front, partial results the combine launch takes at once
SHAPES = [((1, 3, 4, 128, 6000, 300), "attn_rows", 4),
          ((1, 5, 1, 128, 4000, 200), "attn_rows", 8),
          ((1, 3, 4, 128, 3000, 90), "attn_rows", 8),
          ((1, 3, 3, 64, 6000, 50), "attn_rows", 16),
          ((1, 1, 1, 256, 5000, 150), "attn_rows", 16),
          ((1, 8, 4, 128, 1500, 330), "attn_mfma", 4),
          ((1, 4, 4, 128, 12000, 300), "attn_mfma", 8),
          ((1, 3, 4, 256, 9000, 200), "attn_mfma", 8)]


def test_the_shapes_reach_what_they_name(tmp_path):
    for (s, kernel, at_once), r in zip(SHAPES, attention_launches(tmp_path, [s[:4] + (1,) + s[4:] + (0, True) for s, _, _ in SHAPES])):
        (first, _), (second, grid) = r["launches"]
        assert kernel in first and f"attn_combine_kernelILi{s[3]}ELi{at_once}E" in second, (s, first, second)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,kernel,at_once", SHAPES)
def test_joined_runs_against_the_oracle(shape, kernel, at_once):
    L, hkv, G, D, n_ctx, tq = shape
    print(f"attn combine: {shape}", flush=True)
    m = kv.Model(L, hkv, hkv * G, D, torch.bfloat16, 1e4)
    g = torch.Generator(device=DEV)
    g.manual_seed(n_ctx + tq)
    mk = lambda h, n: torch.randn((L, h, n, D), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = mk(hkv * G, tq), mk(hkv, n_ctx + tq), mk(hkv, n_ctx + tq)
    out, lse = kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, want_lse=True)
    conf, lse_conf = kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 11, want_lse=True)
    torch.cuda.synchronize()
    want, want_lse = oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx, want_lse=True)
    check_close(to_np(out), want, torch.bfloat16, str(shape))
    assert float(abs(lse.cpu().numpy() - want_lse).max()) < 2e-2
    assert torch.equal(out, conf) and torch.equal(lse, lse_conf)
