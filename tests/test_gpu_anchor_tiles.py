"""Anchor weights at the edges of the anchor tiles (4, 8 or 16 anchors per lane, several tiles beyond) and of the second
stage's cut into chunks, slots and threads: single-segment and batched calls with pools of different sizes, every
granularity and rule, against the float64 oracle (1e-5 as for all weights; arg-min and selection exact)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from parity import check_close, check_weights, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _want(bk, anc, gran, rule):
    anc = [to_np(a) for a in anc]
    dist, sel = oracle.distances(to_np(bk), anc, gran)
    if rule == kv.RULE_NEAREST:
        return oracle.weights_nearest(dist, sel)
    if rule == kv.RULE_COSINE_SOFTMAX:
        sim, sel = oracle.cosine(to_np(bk), anc, gran)
        return oracle.weights_from_sim(sim, sel, 1.0)
    return oracle.weights(dist, sel, 1.0)


@pytest.mark.parametrize("L,H,D,dtype,S", [(2, 3, 128, torch.bfloat16, 37), (40, 1, 64, torch.bfloat16, 5),
                                           (3, 2, 256, torch.float32, 17)])
def test_pool_sizes_at_tile_edges(L, H, D, dtype, S):
    m = kv.Model(L, H, H, D, dtype, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(L + S)
    mk = lambda n: torch.randn((L, H, n, D), generator=g, device=DEV).to(dtype)
    bk, pool = mk(S), [mk(S + 3) for _ in range(33)]
    for A in (1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 33):
        anc = pool[:A]
        for gran in (kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT):
            for rule in (kv.RULE_L2_SOFTMAX, kv.RULE_NEAREST, kv.RULE_COSINE_SOFTMAX):
                print(f"anchor tiles: L{L} D{D} S{S} A{A} gran{gran} rule{rule}", flush=True)
                w, near, sel = kv.kvcomm_anchor_weights_rule(m, rule, bk, anc, None, 1.0, gran)
                torch.cuda.synchronize()
                want, want_near = _want(bk, anc, gran, rule)
                check_weights(w.cpu().numpy(), want.T)
                assert np.array_equal(near.cpu().numpy(), want_near) and sel.all()


@pytest.mark.parametrize("gran", [kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT])
def test_batch_of_unequal_pools(gran):
    """Pools of 2, 20, 9 and 5 anchors in one launch (its tiles are sized for the largest), one of them with no anchor
    that is long enough: the tiles that a small pool does not have must write nothing."""
    L, H, D = 5, 2, 128
    m = kv.Model(L, H, H, D, torch.bfloat16, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(11)
    mk = lambda n: torch.randn((L, H, n, D), generator=g, device=DEV).to(torch.bfloat16)
    lens = [33, 16, 50, 47]
    jobs = [dict(seg_base_k=mk(S), anchor_base_k=[mk(50) for _ in range(A)], anchor_len=[50 if S != 47 else 46] * A)
            for S, A in zip(lens, (2, 20, 9, 5))]
    print(f"unequal pools gran{gran}", flush=True)
    got = kv.kvcomm_anchor_weights_batch(m, jobs, 1.0, gran)
    torch.cuda.synchronize()
    for (w, near, sel), jd, S in zip(got, jobs, lens):
        if S == 47:
            assert not w.any() and (near == -1).all() and not sel.any()
            continue
        want, want_near = _want(jd["seg_base_k"], jd["anchor_base_k"], gran, kv.RULE_L2_SOFTMAX)
        check_weights(w.cpu().numpy(), want.T)
        assert np.array_equal(near.cpu().numpy(), want_near) and sel.all()


@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 128), (torch.float32, 64)])
@pytest.mark.parametrize("gran", [kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT])
def test_update_pool_sizes(gran, dtype, D):
    """The update at every remainder of its groups of four, two and one anchors, rotated and unrotated deviations mixed,
    plain and E4M3 (against the oracle on the stored values); bf16 2e-2, fp32 1e-5."""
    L, H, S, delta = 2, 3, 35, 300
    m = kv.Model(L, H, H, D, dtype, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(D + gran)
    mk = lambda n, s=1.0: (torch.randn((L, H, n, D), generator=g, device=DEV) * s).to(dtype)
    bk, bv = mk(S), mk(S)
    dk, dv = [mk(S, 0.05) for _ in range(11)], [mk(S, 0.05) for _ in range(11)]
    scale = 2.0 ** -9
    dk8, dv8 = ([kv.kvcomm_quantize_deltas(m, t, scale) for t in x] for x in (dk, dv))
    n = kv.kvcomm_weight_slots(m, S, gran)
    for A in range(1, 12):
        print(f"update pool sizes: D{D} gran{gran} A{A}", flush=True)
        w = torch.softmax(torch.randn((n, A), generator=g, device=DEV), 1).contiguous()
        adp = [delta if a % 3 else 40 * a for a in range(A)]
        ok, ov, ok8, ov8 = (torch.empty_like(bk) for _ in range(4))
        kv.kvcomm_align_kv(m, bk, bv, dk[:A], dv[:A], w, delta, ok, ov, None, adp, gran)
        kv.kvcomm_align_kv_q8(m, bk, bv, dk8[:A], dv8[:A], [scale] * A, [scale] * A, w, delta, ok8, ov8, None, adp, gran)
        torch.cuda.synchronize()
        deq = lambda x: [oracle.dequantize(t.cpu().numpy(), scale) for t in x[:A]]
        for got, devs in (((ok, ov), ([to_np(t) for t in dk[:A]], [to_np(t) for t in dv[:A]])), ((ok8, ov8), (deq(dk8), deq(dv8)))):
            want = oracle.align(to_np(bk), to_np(bv), devs[0], devs[1], w.cpu().numpy().astype(np.float64).T, delta, 5e5, adp, gran)
            check_close(to_np(got[0]), want[0], dtype, "K^")
            check_close(to_np(got[1]), want[1], dtype, "V^")


@pytest.mark.parametrize("gran", [kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT])
def test_nearest_of_infinite_distances(gran):
    """Every anchor infinitely far away: equal distances, so `nearest` is the lowest selected index of the segment's OWN pool
    (pools of 3 and 4 in one launch; the first anchor of the second pool is too short)."""
    print(f"infinite distances gran{gran}", flush=True)
    L, H, D, S = 2, 2, 128, 21
    m = kv.Model(L, H, H, D, torch.bfloat16, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    mk = lambda: torch.randn((L, H, S, D), generator=g, device=DEV).to(torch.bfloat16)
    segs = [mk(), mk()]
    for s in segs:
        s[:, :, 7, 3] = float("inf")
    jobs = [dict(seg_base_k=segs[0], anchor_base_k=[mk() for _ in range(3)]),
            dict(seg_base_k=segs[1], anchor_base_k=[mk() for _ in range(4)], anchor_len=[S - 1, S, S, S])]
    got = kv.kvcomm_anchor_weights_batch(m, jobs, 1.0, gran)
    torch.cuda.synchronize()
    for (w, near, sel), jd, first in zip(got, jobs, (0, 1)):
        bad = near if gran == kv.W_SEGMENT else near.view(-1, S)[:, 7]
        assert (bad == first).all(), bad
        assert near.min() >= first and near.max() < len(jd["anchor_base_k"])


@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128), (torch.float32, 256)])
@pytest.mark.parametrize("gran", [kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN])
def test_update_batches_of_unequal_pools(gran, dtype, D):
    """Pools on both sides of the line between the update's two forms in one launch (the largest pool of a launch chooses):
    bit-identical to the separate calls, rotated and unrotated deviations mixed, plain and E4M3."""
    L, H, S = 2, 3, 35
    m = kv.Model(L, H, H, D, dtype, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(D + gran)
    mk = lambda s=1.0: (torch.randn((L, H, S, D), generator=g, device=DEV) * s).to(dtype)
    n = kv.kvcomm_weight_slots(m, S, gran)
    for pools in ((2, 9), (7, 1, 3), (6, 16, 5)):
        print(f"update of unequal pools: D{D} {dtype} gran{gran} {pools}", flush=True)
        jobs, jobs8 = [], []
        for j, A in enumerate(pools):
            w = torch.softmax(torch.randn((n, A), generator=g, device=DEV), 1).contiguous()
            d = dict(base_k=mk(), base_v=mk(), weights=w, delta_pos=300 + 40 * j, out_k=torch.empty_like(mk()),
                     out_v=torch.empty_like(mk()), anchor_delta_pos=[(300 + 40 * j, 77, 1024)[a % 3] for a in range(A)])
            dk, dv = [mk(0.05) for _ in range(A)], [mk(0.05) for _ in range(A)]
            q8 = lambda x: [kv.kvcomm_quantize_deltas(m, t, 2.0 ** -9) for t in x]
            jobs.append(dict(d, anchor_dk=dk, anchor_dv=dv))
            jobs8.append(dict(d, anchor_dk8=q8(dk), anchor_dv8=q8(dv), scale_k=[2.0 ** -9] * A, scale_v=[2.0 ** -9] * A,
                              out_k=torch.empty_like(d["out_k"]), out_v=torch.empty_like(d["out_v"])))
        kv.kvcomm_align_kv_batch(m, jobs, gran)
        kv.kvcomm_align_kv_q8_batch(m, jobs8, gran)
        for jd, j8 in zip(jobs, jobs8):
            ok, ov = torch.empty_like(jd["out_k"]), torch.empty_like(jd["out_v"])
            kv.kvcomm_align_kv(m, jd["base_k"], jd["base_v"], jd["anchor_dk"], jd["anchor_dv"], jd["weights"],
                               jd["delta_pos"], ok, ov, None, jd["anchor_delta_pos"], gran)
            assert torch.equal(ok, jd["out_k"]) and torch.equal(ov, jd["out_v"])
            kv.kvcomm_align_kv_q8(m, jd["base_k"], jd["base_v"], j8["anchor_dk8"], j8["anchor_dv8"], j8["scale_k"],
                                  j8["scale_v"], jd["weights"], jd["delta_pos"], ok, ov, None, jd["anchor_delta_pos"], gran)
            torch.cuda.synchronize()
            assert torch.equal(ok, j8["out_k"]) and torch.equal(ov, j8["out_v"])


def test_more_groups_than_the_grid_has_room_for_in_z():
    """Two anchor tiles over more than 262144 (chunk, token tile) pairs: groups of more than eight pairs.  The last tokens equal
    the same call on those tokens alone (per-(layer, head, token) weights: rows are independent)."""
    L, H, D, S, A, last = 32, 8, 64, 33000, 17, 70
    print(f"many groups: S{S} A{A}", flush=True)
    m = kv.Model(L, H, H, D, torch.bfloat16, 5e5)
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    mk = lambda: torch.randn((L, H, S, D), generator=g, device=DEV, dtype=torch.bfloat16)
    bk, two = mk(), [mk(), mk()]
    anc = [two[a % 2] for a in range(A)]
    w, near, _ = kv.kvcomm_anchor_weights(m, bk, anc, gran=kv.W_LAYER_HEAD_TOKEN)
    part = lambda t, n: t.view(L * H, S, -1)[:, S - n:].reshape(L * H * n, -1)
    tail = lambda t: t[:, :, S - last:]
    wt, nt, _ = kv.kvcomm_anchor_weights(m, tail(bk), [tail(a) for a in anc], gran=kv.W_LAYER_HEAD_TOKEN)
    torch.cuda.synchronize()
    assert torch.equal(part(w, last), wt) and torch.equal(part(near, last).view(-1), nt)
