"""Per-token weights in one launch (token_weights_kernel) and in two (partial sums, softmax), both
against the float64 oracle (1e-5 as for all weights; arg-min and selection exact) where a block's tokens, the wavefronts' share
of (layer, head) pairs or the anchor tiles do not come out even."""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2510_12872_amd as kv

from launches import record
from parity import check_weights, to_np

DEV = "cuda"
BF, F32 = torch.bfloat16, torch.float32
RULES = (kv.RULE_L2_SOFTMAX, kv.RULE_NEAREST, kv.RULE_COSINE_SOFTMAX)

# L, H, D, dtype, segment lengths, anchors per segment; one launch
ONE = [(1, 1, 64, BF, [1], [1]),              # one token, seven of eight wavefronts without a pair
       (3, 3, 64, BF, [9, 17], [5, 2]),       # eight rows per wavefront, ragged last block
       (5, 5, 128, BF, [130], [16]),          # a full tile
       (7, 5, 128, BF, [11, 3, 6], [9, 1, 4]),
       (3, 7, 256, BF, [5, 8], [4, 8]),
       (2, 3, 64, F32, [33], [7]),
       (3, 5, 128, F32, [21, 4], [3, 12]),
       (9, 1, 256, F32, [7], [6])]            # one row per wavefront
TWO = [(32, 8, 64, BF, [7], [8]), (32, 8, 128, BF, [19], [3]), (40, 4, 128, F32, [9], [13]), (2, 2, 128, BF, [12], [17])]


def _jobs(L, H, D, dtype, lens, pools, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + L + D)
    # (strided views: tokens of a longer cache, heads before layers)
    view = lambda n: torch.randn((H, L, n + 5, D), generator=g, device=DEV).to(dtype).permute(1, 0, 2, 3)[:, :, 2:2 + n]
    cap = max(lens) + 2
    pool = torch.randn((sum(pools), H, L, cap, D), generator=g, device=DEV).to(dtype)
    anc, i = [], 0
    for n in pools:
        anc.append([pool[i + a].permute(1, 0, 2, 3) for a in range(n)])
        i += n
    return [dict(seg_base_k=view(S), anchor_base_k=a) for S, a in zip(lens, anc)]


@pytest.mark.gpu
@pytest.mark.parametrize("L,H,D,dtype,lens,pools", ONE + TWO)
def test_against_the_oracle(L, H, D, dtype, lens, pools):
    m = kv.Model(L, H, H, D, dtype, 5e5)
    jobs = _jobs(L, H, D, dtype, lens, pools)
    for rule in RULES:
        print(f"token weights: L{L} H{H} D{D} {dtype} {lens} {pools} rule{rule}", flush=True)
        got = kv.kvcomm_anchor_weights_batch(m, jobs, 1.0, kv.W_TOKEN, rule)
        torch.cuda.synchronize()
        for (w, near, sel), jd, S in zip(got, jobs, lens):
            bk, anc = to_np(jd["seg_base_k"]), [to_np(a[:, :, :S]) for a in jd["anchor_base_k"]]
            if rule == kv.RULE_COSINE_SOFTMAX:
                want, want_near = oracle.weights_from_sim(*oracle.cosine(bk, anc, kv.W_TOKEN), 1.0)
            elif rule == kv.RULE_NEAREST:
                want, want_near = oracle.weights_nearest(*oracle.distances(bk, anc, kv.W_TOKEN))
            else:
                want, want_near = oracle.weights(*oracle.distances(bk, anc, kv.W_TOKEN), 1.0)
            check_weights(w.cpu().numpy(), want.T)
            assert np.array_equal(near.cpu().numpy(), want_near) and sel.all()


@pytest.mark.gpu
def test_short_anchors_and_empty_pools():
    """A pool none of whose anchors is long enough beside pools that have some; rows behind a short anchor are never read as weights."""
    L, H, D = 3, 2, 128
    m = kv.Model(L, H, H, D, BF, 5e5)
    jobs = _jobs(L, H, D, BF, [13, 7, 10], [4, 3, 2], seed=5)
    lens = [[15, 12, 15, 3], [6, 2, 0], [10, 9]]
    for jd, n in zip(jobs, lens):
        jd["anchor_len"] = n
        for a, k in zip(jd["anchor_base_k"], n):
            a[:, :, k:] = float("nan")
    print("token weights: short anchors", flush=True)
    got = kv.kvcomm_anchor_weights_batch(m, jobs, 1.0, kv.W_TOKEN)
    torch.cuda.synchronize()
    for (w, near, sel), jd, n in zip(got, jobs, lens):
        S = jd["seg_base_k"].shape[2]
        live = [a for a, k in enumerate(n) if k >= S]
        assert [i for i, s in enumerate(sel.tolist()) if s] == live
        want = np.zeros((S, len(n)))
        if live:
            dist, ok = oracle.distances(to_np(jd["seg_base_k"]), [to_np(jd["anchor_base_k"][a][:, :, :S]) for a in live], kv.W_TOKEN)
            lw, ln = oracle.weights(dist, ok, 1.0)
            want[:, live] = lw.T
            assert near.tolist() == [live[i] for i in ln]
        else:
            assert (near == -1).all()
        check_weights(w.cpu().numpy(), want)


DRIVER = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
i32, i64, vp, sz = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t
class Model(ctypes.Structure):
    _fields_ = [(n, i32) for n in ("L", "hkv", "hq", "D", "dtype")] + [("theta", ctypes.c_double)]
class Tensor(ctypes.Structure):
    _fields_ = [("ptr", vp), ("sl", i64), ("sh", i64), ("st", i64)]
class Job(ctypes.Structure):
    _fields_ = [("seg", Tensor), ("S", i32), ("anc", vp), ("len", vp), ("n", i32), ("w", vp), ("near", vp), ("sel", vp)]
shim.rec_name.restype = ctypes.c_char_p
shim.rec_grid.restype = shim.rec_block.restype = ctypes.c_uint
f = lib.kvcomm_anchor_weights_batch
f.argtypes = [vp, i32, i32, ctypes.c_float, Tensor, vp, i32, vp, sz, vp]
res = []
for L, H, D, dtype, lens, pools, rule in json.load(sys.stdin):
    keep, jobs = [], (Job * len(lens))()
    for j, (S, n) in enumerate(zip(lens, pools)):
        anc, ln = (vp * n)(*[0x1000] * n), (i32 * n)(*[S] * n)
        keep += [anc, ln]
        jobs[j] = Job(Tensor(0x1000, H * S * D, S * D, D), S, ctypes.addressof(anc), ctypes.addressof(ln), n, 0x1000, 0x1000, 0x1000)
    shim.rec_clear()
    cap = max(lens)
    st = f(ctypes.byref(Model(L, H, H, D, dtype, 1e4)), 0, rule, 1.0, Tensor(0x1000, H * cap * D, cap * D, D), jobs, len(lens), 0x1000, 1 << 40, None)
    res.append(dict(status=st, names=[shim.rec_name(i).decode() for i in range(shim.rec_count())], grid=shim.rec_grid(0, 0),
                    threads=[shim.rec_grid(i, 0) * shim.rec_block(i, 0) for i in range(shim.rec_count())]))
json.dump(res, sys.stdout)
"""


def _launches(tmp_path, calls):
    return record(tmp_path, DRIVER, [[c[0], c[1], c[2], 0 if c[3] == F32 else 1, c[4], c[5], rule] for c, rule in calls])


def test_the_shapes_of_the_oracle_test_reach_what_they_name(tmp_path):
    """Under every rule; cosine has its own instantiations, one of whose pools takes two anchor tiles."""
    calls = [(c, rule) for c in ONE + TWO for rule in RULES]
    kernels = set()
    for (c, rule), r in zip(calls, _launches(tmp_path, calls)):
        one = len(r["names"]) == 1 and "token_weights_kernel" in r["names"][0]
        assert r["status"] == 0 and one == (c in ONE), (c, rule, r)
        assert one or ("partial_kernel" in r["names"][0] and "finalize_kernel" in r["names"][1])
        if one:
            assert ("ELb1E" in r["names"][0]) == (rule == kv.RULE_COSINE_SOFTMAX)
            kernels.add((re.search(r"token_weights_kernelI(\w+?Li\d+E)Li\d+ELb", r["names"][0])[1], rule == kv.RULE_COSINE_SOFTMAX))
    assert any(max(c[5]) > 8 for c in ONE) and len(kernels) == 12     # three row widths of two types


def test_more_tokens_than_a_launch_holds_blocks(tmp_path):
    """A block per token and 2^23 tokens would be 2^32 threads, which no launch holds: the two stages."""
    below, above = _launches(tmp_path, [((4, 4, 256, F32, [S], [8]), 0) for S in ((1 << 23) - 1, 1 << 23)])
    for r, n in ((below, 1), (above, 2)):
        assert r["status"] == 0 and len(r["names"]) == n and all(t < 1 << 32 for t in r["threads"]), r


def test_rows_that_meet_in_the_same_memory_channels(tmp_path):
    """Heads an odd multiple of 512 KB apart, many of them and four anchors or more: two stages, which do not have several heads in flight."""
    f = lambda L, D, dtype, S, n: (L, 8, D, dtype, [S], [n])
    two = [f(32, 128, BF, 2048, 4), f(16, 128, BF, 2048, 8), f(32, 128, F32, 1024, 8), f(32, 256, BF, 1024, 4), f(24, 64, F32, 2048, 6), f(32, 128, BF, 6144, 4)]
    one = [f(32, 128, BF, 2048, 3), f(15, 128, BF, 2048, 8), f(32, 128, BF, 2000, 8), f(32, 128, BF, 1024, 8), f(32, 128, BF, 4096, 4), f(32, 128, F32, 512, 8)]
    for c, r in zip(two + one, _launches(tmp_path, [(c, 0) for c in two + one])):
        assert r["status"] == 0 and len(r["names"]) == (1 if c in one else 2), (c, r)


def test_few_wide_rows(tmp_path):
    """Two and three anchors of 128 tokens of 256 bf16 channels leave half of the compute units empty: two stages; not for narrower rows or more tokens."""
    calls = [((32, 8, 256, BF, [S], [n]), 0) for S, n in ((128, 2), (140, 3), (170, 2), (200, 3), (140, 4))] + [((32, 8, 128, F32, [140], [3]), 0)]
    assert [len(r["names"]) for r in _launches(tmp_path, calls)] == [2, 2, 1, 1, 1, 1]
