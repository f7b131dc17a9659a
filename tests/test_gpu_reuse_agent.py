"""A whole step of an agent with several segments (batched calls) against the same calls one segment after the other: equal up to the order of
the distance sums, and bit for bit where the segments cannot share a launch."""
import pytest
import torch

import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding, hotpath, workloads
from paper_2510_12872_amd.workloads import scaled

pytestmark = pytest.mark.gpu
DEV = "cuda"
W = scaled(workloads.LLAMA8B_5AGENTS, name="small", n_layers=3, n_kv_heads=2, n_q_heads=4, prefix_len=5, seg_len=21, n_segments=3,
           n_anchors=5, tq=4, anchor_delta_choices=(3, 40))


def one_by_one(w, m, agent, gran=kv.W_TOKEN):
    for j, s in enumerate(agent.segments):
        p0, S = w.seg_offset(j), s.base_k.shape[2]
        hotpath.align_segment(m, s, agent.cache_k[:, :, p0:p0 + S], agent.cache_v[:, :, p0:p0 + S], w.temperature, gran)
    return kv.kvcomm_suffix_attn(m, agent.q, agent.cache_k, agent.cache_v, w.n_ctx)


def both(w, change=lambda agent: None, gran=kv.W_TOKEN, scratches=None):
    m = hotpath.model_of(w)
    a, b = (workloads.make_agent(w, 0, DEV) for _ in range(2))
    change(a), change(b)
    want = one_by_one(w, m, a, gran)
    got = hotpath.reuse_agent(w, m, b, gran=gran, scratches=scratches)
    torch.cuda.synchronize()
    return (want, a.cache_k, a.cache_v), (got, b.cache_k, b.cache_v)


def close(want, got, dtype):
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-5
    for x, y in zip(want, got):
        assert float((x.float() - y.float()).abs().max()) <= tol * max(1.0, float(x.float().abs().max()))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("gran", [kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT])
@pytest.mark.parametrize("nseg,A", [(2, 1), (3, 5), (9, 16)])   # 9 x 16: three launches
def test_several_segments(dtype, gran, nseg, A):
    print(f"reuse_agent: {dtype} gran {gran} {nseg} segments {A} anchors", flush=True)
    w = scaled(W, dtype=dtype, n_segments=nseg, n_anchors=A, anchor_delta_choices=None)
    m = hotpath.model_of(w)
    sc = [hotpath.Scratch(m, w.seg_len, A, gran, DEV) for _ in range(nseg)]
    for scratches in (None, sc):
        want, got = both(w, gran=gran, scratches=scratches)
        close(want, got, dtype)
    assert sc[0].workspace.numel() <= hotpath.JOINT_WORKSPACE
    for s in sc:   # too little for one launch of them all: one after the other, with what that needs
        s.workspace = s.workspace[:max(256, kv.kvcomm_anchor_weights_workspace(m, w.seg_len, A, gran))].clone()
    want, got = both(w, gran=gran, scratches=sc)
    close(want, got, dtype)


def other_layout(agent):
    s = agent.segments[1]
    for name in ("anchor_k", "anchor_dk", "anchor_dv"):
        pad = lambda t: torch.cat([t, torch.zeros_like(t[:, :, :7])], 2)
        setattr(s, name, [pad(t) for t in getattr(s, name)])


def in_place(agent):   # base rows already in their slots of the cache
    for j, s in enumerate(agent.segments):
        p0, S = W.seg_offset(j), s.base_k.shape[2]
        agent.cache_k[:, :, p0:p0 + S], agent.cache_v[:, :, p0:p0 + S] = s.base_k, s.base_v
        s.base_k, s.base_v = agent.cache_k[:, :, p0:p0 + S], agent.cache_v[:, :, p0:p0 + S]


def values_in_place(agent):
    in_place(agent)
    for s in agent.segments:
        s.base_k = s.base_k.clone()


def matched_in_the_cache(agent):   # the second segment's anchor is what the first one's update writes
    s, p0 = agent.segments[1], W.seg_offset(0)
    n = agent.cache_k.shape[2]
    s.anchor_k = [agent.cache_k[:, :, p0:]] + [(agent.cache_k * (i + 1.5)).contiguous()[:, :, p0:] for i in range(len(s.anchor_k) - 1)]
    s.anchor_len = [n - p0] * len(s.anchor_k)
    s.anchor_dk, s.anchor_dv = ([torch.cat([t, t[:, :, :1].expand(-1, -1, n - p0 - t.shape[2], -1)], 2) for t in ts] for ts in (s.anchor_dk, s.anchor_dv))


def delta_in_the_cache(agent):   # the last segment's offsets are rows that the first one's update writes
    s, p0 = agent.segments[-1], W.seg_offset(0)
    n = s.anchor_dk[0].shape[2]
    s.anchor_dk = [agent.cache_k[:, :, p0:p0 + n]]
    s.anchor_dv, s.anchor_k, s.anchor_len, s.anchor_delta_pos = [torch.zeros_like(agent.cache_v)[:, :, p0:p0 + n]], s.anchor_k[:1], s.anchor_len[:1], [0]


class Overlapping(type(W)):   # slots that share rows: the later segment's stay
    def seg_offset(self, j):
        return self.prefix_len + j * (self.seg_len - 4)


def many_rotations(agent):
    for k, s in enumerate(agent.segments):
        s.anchor_delta_pos = [1000 * k + 7 * a for a in range(len(s.anchor_k))]


@pytest.mark.parametrize("change", [other_layout, in_place, values_in_place, matched_in_the_cache, delta_in_the_cache])
def test_segments_that_cannot_share_a_launch(change):
    print(f"reuse_agent: {change.__name__}", flush=True)
    want, got = both(W, change)
    for x, y in zip(want, got):
        assert torch.equal(x, y)


def test_slots_and_scratch_that_segments_share():
    m = hotpath.model_of(W)
    print("reuse_agent: shared", flush=True)
    one = hotpath.Scratch(m, W.seg_len, W.n_anchors, kv.W_TOKEN, DEV)
    for w, scratches in ((Overlapping(**vars(W)), None), (W, [one] * W.n_segments), (W, [None] * W.n_segments)):
        want, got = both(w, scratches=scratches)
        for x, y in zip(want, got):
            assert torch.equal(x, y)


def test_rotations_of_all_segments():
    """Pools of 20 anchors, each recorded elsewhere: 61 ... 63 rotations of three segments fit a launch, and are taken either way."""
    w = scaled(W, n_anchors=20, anchor_delta_choices=None)
    want, got = both(w, many_rotations)
    close(want, got, w.dtype)


@pytest.mark.parametrize("A,runs", [(15, [4]), (16, [3])])   # 4 x 16 rotations fit a launch, 4 x 17 do not
def test_rotations_beyond_a_launch(monkeypatch, A, runs):
    """The library takes the runs that the segments are cut into, each at once."""
    print(f"reuse_agent: 4 segments, {A} anchors recorded elsewhere", flush=True)
    taken, call = [], binding.kvcomm_align_kv_batch

    def noted(model, jobs, *a):
        call(model, jobs, *a)
        taken.append(len(jobs))
    monkeypatch.setattr(binding, "kvcomm_align_kv_batch", noted)
    w = scaled(W, n_segments=4, n_anchors=A, anchor_delta_choices=None)
    want, got = both(w, many_rotations)
    assert taken == runs
    close(want, got, w.dtype)
    with pytest.raises(kv.KVCommError) as refused:   # one rotation too many for the library
        agent = workloads.make_agent(scaled(w, n_anchors=16), 0, DEV)
        many_rotations(agent)
        hotpath.align_agent_batched(w, hotpath.model_of(w), agent)
    assert refused.value.status == binding.EUNSUPPORTED


def test_a_refused_segment_is_refused():
    w = scaled(W, n_segments=2)
    m = hotpath.model_of(w)
    agent = workloads.make_agent(w, 0, DEV)
    agent.segments[1].anchor_dk = [t[..., ::2] for t in agent.segments[1].anchor_dk]
    with pytest.raises(kv.KVCommError):
        hotpath.reuse_agent(w, m, agent)


def test_in_a_graph():
    """Every replay, with other keys in place and eager steps between, equals the eager step."""
    m = hotpath.model_of(W)
    agent, eager = (workloads.make_agent(W, 0, DEV) for _ in range(2))
    sc, sc2 = ([hotpath.Scratch(m, W.seg_len, W.n_anchors, kv.W_TOKEN, DEV) for _ in range(W.n_segments)] for _ in range(2))
    out = torch.empty_like(agent.q)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hotpath.reuse_agent(W, m, agent, out=out, scratches=sc)
    for k in range(3):
        for s, t in zip(agent.segments, eager.segments):
            x = torch.randn_like(s.base_k)
            s.base_k.copy_(x), t.base_k.copy_(x)
        want = hotpath.reuse_agent(W, m, eager, scratches=sc2)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(agent.cache_k, eager.cache_k)
