"""Weight rows of the update kernel: its blocks load whole rows and keep the selected anchors' columns.  Against a double-precision
sum of the same stored values: rows wider than a block's first load, segments that end inside a token tile, every granularity; what
stands in the columns of unselected anchors must not matter.  bf16: half a unit in the last place of the result plus 1e-5 of fp32 sums."""
import pytest
import torch

import paper_2510_12872_amd as kv

DEV = "cuda"


def _rotate(x, pos, theta, D):
    ang = pos * theta ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device=x.device) / D)
    a, b = x[..., :D // 2], x[..., D // 2:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256), (torch.float32, 64), (torch.float32, 256)])
@pytest.mark.parametrize("A,S", [(1, 1), (2, 31), (3, 33), (9, 65), (64, 70)])
def test_selected_columns(dtype, D, A, S):
    _check_columns(dtype, D, A, S, 2, 3)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,D,A,S,L,H", [(torch.bfloat16, 128, 4, 8, 32, 8), (torch.bfloat16, 128, 7, 77, 32, 8), (torch.float32, 128, 6, 33, 24, 8),
                                             (torch.bfloat16, 64, 11, 65, 60, 8), (torch.bfloat16, 256, 33, 5, 80, 8), (torch.bfloat16, 128, 48, 3, 80, 8)])
def test_selected_columns_of_larger_launches(dtype, D, A, S, L, H):
    """On both sides of the lines between two and four anchors in flight."""
    _check_columns(dtype, D, A, S, L, H)


def _check_columns(dtype, D, A, S, L, H):
    theta = 1e4
    m = kv.Model(L, H, H, D, dtype, theta)
    g = torch.Generator(device=DEV)
    g.manual_seed(A * 100 + S + D)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    bk, bv = rnd(L, H, S, D).to(dtype), rnd(L, H, S, D).to(dtype)
    dk, dv = [[(0.1 * rnd(L, H, S, D)).to(dtype) for _ in range(A)] for _ in range(2)]
    lens = [S - 1 if a % 3 == 1 else S for a in range(A)]
    adp = [(7, 131071, 40)[a % 3] for a in range(A)]
    for gran, slots in ((kv.W_TOKEN, S), (kv.W_LAYER_HEAD_TOKEN, L * H * S), (kv.W_SEGMENT, 1)):
        print(f"update weights: {dtype} D{D} A{A} S{S} L{L} H{H} gran{gran}", flush=True)
        w = torch.softmax(rnd(slots, A), 1)
        for a in range(A):
            if lens[a] < S:
                w[:, a] = float("nan")
        out_k, out_v = torch.zeros_like(bk), torch.zeros_like(bv)
        kv.kvcomm_align_kv(m, bk, bv, dk, dv, w, 40, out_k, out_v, lens, adp, gran)
        wt = w.double().t().reshape(A, *{kv.W_TOKEN: (1, 1, S, 1), kv.W_LAYER_HEAD_TOKEN: (L, H, S, 1), kv.W_SEGMENT: (1, 1, 1, 1)}[gran])
        want_k, want_v = _rotate(bk.double(), 40, theta, D), bv.double()
        for a in range(A):
            if lens[a] >= S:
                want_k = want_k + wt[a] * _rotate(dk[a].double(), 40 - adp[a], theta, D)
                want_v = want_v + wt[a] * dv[a].double()
        for got, want in ((out_k, want_k), (out_v, want_v)):
            tol = 1e-5 * want.abs().max() + (want.abs() * 2.0 ** -8 if dtype == torch.bfloat16 else 0.0)
            assert bool(((got.double() - want).abs() <= tol).all())


@pytest.mark.gpu
def test_more_blocks_than_one_axis_of_a_launch_holds():
    """2^24 blocks and a few: the (layer, head) pairs past the grid's first axis.  One token per segment and no anchors (what fits
    memory): keys rotated within half a unit in the last place and 1e-5, values copied."""
    L, H, D, n, theta = 299600, 7, 64, 8, 1e4
    m = kv.Model(L, H, H, D, torch.bfloat16, theta)
    g = torch.Generator(device=DEV)
    g.manual_seed(11)
    bk, bv = (torch.randn((L, H, n, D), generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    out_k, out_v = torch.zeros_like(bk), torch.zeros_like(bv)
    at = lambda t, j: t[:, :, j:j + 1]
    print(f"update blocks: L{L} H{H} {n} segments", flush=True)
    kv.kvcomm_align_kv_batch(m, [dict(base_k=at(bk, j), base_v=at(bv, j), anchor_dk=[], anchor_dv=[], delta_pos=100 * j, out_k=at(out_k, j),
                                      out_v=at(out_v, j)) for j in range(n)])
    torch.cuda.synchronize()
    assert torch.equal(out_v, bv)
    for j in range(n):
        for part in range(0, L, 50000):
            want = _rotate(bk[part:part + 50000, :, j].double(), 100 * j, theta, D)
            assert bool(((out_k[part:part + 50000, :, j].double() - want).abs() <= 1e-5 * want.abs().max() + want.abs() * 2.0 ** -8).all())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_beside_other_work_the_same_bits(dtype):
    """400 tokens, 8 anchors, 32 layers x 8 heads: large enough for the bound on the blocks per compute unit."""
    L, H, S, D, A = 32, 8, 400, 128, 8
    m = kv.Model(L, H, H, D, dtype, 1e4)
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    rnd = lambda: torch.randn((L, H, S, D), generator=g, device=DEV).to(dtype)
    job = dict(base_k=rnd(), base_v=rnd(), anchor_dk=[rnd() for _ in range(A)], anchor_dv=[rnd() for _ in range(A)], delta_pos=70,
               anchor_delta_pos=[70, 3] * 4, weights=torch.softmax(torch.randn((S, A), generator=g, device=DEV), 1))

    def run(call):
        out = dict(out_k=torch.zeros_like(job["base_k"]), out_v=torch.zeros_like(job["base_v"]))
        call([{**job, **out}])
        return out["out_k"], out["out_v"]
    want = run(lambda j: kv.kvcomm_align_kv_batch(m, j))
    for units in (1, 64, 96, 200, 1000):
        print(f"update beside: {dtype} units{units}", flush=True)
        got = run(lambda j: kv.kvcomm_align_kv_batch_beside(m, j, units))
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    with pytest.raises(kv.KVCommError):
        run(lambda j: kv.kvcomm_align_kv_batch_beside(m, j, 0))
