"""Updates of few rows, a row's anchors over the wavefronts of a block, against the same update in a launch that takes the general kernel (beside a
segment of two anchors): up to the order of at most 64 fp32 additions, each 2^-24 of what has been summed (and one rounding to bf16)."""
import pytest
import torch

import paper_2510_12872_amd as kv

pytestmark = pytest.mark.gpu
DEV = "cuda"


def cache(g, shape, dtype, form):
    L, H, S, D = shape
    make = lambda *s: torch.randn(s, generator=g, device=DEV).to(dtype)
    if form == "tokens":   # [L, S, H, D]
        return make(L, S, H, D).transpose(1, 2)
    if form == "slot":     # rows of a longer cache
        return make(L, H, S + 9, D)[:, :, 5:5 + S]
    return make(L, H, S, D)


@pytest.mark.parametrize("form", ["plain", "tokens", "slot", "in place"])
@pytest.mark.parametrize("gran", [kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT])
@pytest.mark.parametrize("dtype,D,L,H,S,A", [
    (torch.bfloat16, 128, 2, 2, 27, 4), (torch.bfloat16, 128, 2, 2, 33, 5), (torch.bfloat16, 64, 1, 3, 17, 7), (torch.bfloat16, 256, 3, 1, 9, 8),
    (torch.float32, 256, 2, 2, 3, 9), (torch.float32, 64, 1, 2, 1, 31), (torch.float32, 128, 2, 1, 21, 62),
    (torch.bfloat16, 128, 32, 4, 16, 4), (torch.bfloat16, 128, 16, 8, 24, 8), (torch.float32, 128, 4, 8, 33, 11)])   # the last of their sizes
def test_same_as_the_general_launch(dtype, D, L, H, S, A, gran, form):
    print(f"update in parts: {dtype} D{D} {L}x{H} S{S} A{A} gran {gran} {form}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(A * 1000 + S * 10 + gran)
    m = kv.Model(L, H, H, D, dtype, 1e4)
    slots = lambda n: (n, L * H * n, 1)[(kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT).index(gran)]

    def job(S, A):
        new = lambda: cache(g, (L, H, S, D), dtype, form)
        w = torch.softmax(torch.randn(slots(S), A, generator=g, device=DEV), 1)
        d = lambda: [0.3 * new() for _ in range(A)]
        return dict(base_k=new(), base_v=new(), dk=d(), dv=d(), weights=w, len=[S] * A, adp=[(7, 40, 999)[a % 3] for a in range(A)])

    one, other = job(S, A), job(S, 2)

    def as_job(j):
        base_k, base_v = j["base_k"], j["base_v"]
        if form == "in place":
            base_k, base_v = out_k, out_v = base_k.clone(), base_v.clone()
        else:
            out_k, out_v = cache(g, (L, H, S, D), dtype, form), cache(g, (L, H, S, D), dtype, form)
        return dict(base_k=base_k, base_v=base_v, anchor_dk=j["dk"], anchor_dv=j["dv"], anchor_len=j["len"], weights=j["weights"], delta_pos=40,
                    anchor_delta_pos=j["adp"], out_k=out_k, out_v=out_v)

    alone, beside = [as_job(one)], [as_job(one), as_job(other)]
    kv.kvcomm_align_kv_batch(m, alone, gran)
    kv.kvcomm_align_kv_batch(m, beside, gran)
    torch.cuda.synchronize()
    for out, base, ds in (("out_k", "base_k", "dk"), ("out_v", "base_v", "dv")):
        got, want = alone[0][out].double(), beside[0][out].double()
        most = 1.5 * (float(one[base].abs().max()) + max(float(d.abs().max()) for d in one[ds]))
        tol = 2 * (A + 4) * 2.0 ** -24 * most + (2.0 ** -7 * want.abs() if dtype == torch.bfloat16 else 0.0)
        assert bool(((got - want).abs() <= tol).all()), float((got - want).abs().max())
