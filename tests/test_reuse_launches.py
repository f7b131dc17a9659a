"""Which library calls a step of several segments makes: every segment is matched once and updated once, in as few launches as the
batched calls' limits allow.  (CPU only: the calls are replaced by ones that know those limits and note what they were given.)"""
import collections

import pytest
import torch

import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding, hotpath, workloads
from paper_2510_12872_amd.workloads import scaled

W = scaled(workloads.LLAMA8B_5AGENTS, n_layers=2, n_kv_heads=2, n_q_heads=4, head_dim=64, prefix_len=2, seg_len=6, n_segments=4,
           n_anchors=16, tq=0)
M = hotpath.model_of(W)


class Library:
    """The calls of the weights and the update: `calls` lists (name, segments), `attempts` those that `refuse`
    made fail, `declined` counts what their limits refused."""
    def __init__(self, agent):
        self.agent, self.calls, self.attempts, self.refuse, self.declined = agent, [], [], {}, 0

    def index(self, base_k):
        return next(j for j, s in enumerate(self.agent.segments) if s.base_k is base_k)

    def note(self, name, idx):
        for what in (name, "together" if name == "align" and len(idx) > 1 else ""):
            if what in self.refuse:
                self.attempts.append((name, idx))
                raise kv.KVCommError(self.refuse[what], "refused")
        self.calls.append((name, idx))

    def limit(self, status):
        self.declined += 1
        raise kv.KVCommError(status, "limit")

    def layout(self, jobs, *names):
        if len({t.stride() for jd in jobs for n in names for t in jd[n]}) > 1:
            self.limit(-1)

    def weights_batch(self, model, jobs, temperature, gran, workspace, stream):
        idx = [self.index(jd["seg_base_k"]) for jd in jobs]
        pools = [len(jd["anchor_base_k"]) for jd in jobs]
        self.layout(jobs, "anchor_base_k")
        if len(jobs) > 8 or sum(pools) > 64:
            self.limit(-2)
        if workspace.numel() < kv.kvcomm_anchor_weights_batch_workspace(model, [jd["seg_base_k"].shape[2] for jd in jobs], pools, gran):
            self.limit(-3)
        self.note("weights", idx)

    def align_batch(self, model, jobs, gran, stream):
        tables = sum(len({jd["delta_pos"]} | {jd["delta_pos"] - d for d in jd["anchor_delta_pos"] or ()} - {0}) for jd in jobs)
        self.layout(jobs, "anchor_dk", "anchor_dv")
        if len(jobs) > 8 or tables > 65 or sum(len(jd["anchor_dk"]) for jd in jobs) > 64:
            self.limit(-2)
        self.note("align", [self.index(jd["base_k"]) for jd in jobs])

    def weights(self, model, seg_base_k, *rest):
        self.note("weights", [self.index(seg_base_k)])

    def align(self, model, base_k, *rest):
        self.note("align", [self.index(base_k)])


@pytest.fixture
def step(monkeypatch):
    def run(w, change=lambda agent: None, scratches=None, refuse={}, gran=kv.W_TOKEN):
        agent = workloads.make_agent(w, 0)
        change(agent)
        lib = Library(agent)
        lib.refuse = refuse
        for name in ("weights", "align"):
            monkeypatch.setattr(binding, "kvcomm_anchor_weights" if name == "weights" else "kvcomm_align_kv", getattr(lib, name))
        monkeypatch.setattr(binding, "kvcomm_anchor_weights_batch", lib.weights_batch)
        monkeypatch.setattr(binding, "kvcomm_align_kv_batch", lib.align_batch)
        lib.error = None
        try:
            hotpath.reuse_agent(w, hotpath.model_of(w), agent, gran=gran, scratches=scratches(agent) if scratches else None)
        except kv.KVCommError as e:
            lib.error = e.status
        return lib
    kv.load_library()
    return run


def both(*runs):
    """Weights and update of each run in turn."""
    return [(name, list(r)) for r in runs for name in ("weights", "align")]


def each_alone(n):
    return both(*([j] for j in range(n)))


def elsewhere(agent):   # every anchor recorded at a position of its own
    for k, s in enumerate(agent.segments):
        s.anchor_delta_pos = [1000 * k + 7 * a for a in range(len(s.anchor_k))]


def padded(*names):
    def change(agent):
        s = agent.segments[1]
        for n in names:
            setattr(s, n, [torch.cat([t, t], 2) for t in getattr(s, n)])
    return change


def plain(agent):
    return [hotpath.Scratch(M, s.base_k.shape[2], len(s.anchor_k), kv.W_TOKEN, "cpu") for s in agent.segments]


@pytest.mark.parametrize("scratches", [None, plain])
def test_limits_are_known_before_the_first_launch(step, scratches):
    """4 x 16 anchors fit a launch, 4 x 17 rotations do not (65 do); neither do anchors of different layouts, of whichever tensor, nor more
    anchors or segments than a launch holds."""
    assert step(W, scratches=scratches).calls == both([0, 1, 2, 3])
    assert step(W, elsewhere, scratches).calls == both([0, 1, 2], [3])
    fifteen = scaled(W, n_anchors=15)
    assert step(fifteen, elsewhere, scratches).calls == both([0, 1, 2, 3])
    for change in (padded("anchor_k"), padded("anchor_dk", "anchor_dv")):
        assert step(W, change, scratches).calls == both([0], [1], [2, 3])
    assert step(scaled(W, n_segments=9, n_anchors=7), scratches=scratches).calls == both(range(8), [8])
    assert step(scaled(W, n_segments=3, n_anchors=40), scratches=scratches).calls == each_alone(3)


def test_rotations_that_anchors_share_or_do_not_need(step):
    def shared(agent):
        elsewhere(agent)
        for s in agent.segments[:2]:
            s.anchor_delta_pos[1] = s.anchor_delta_pos[0]
            s.anchor_delta_pos[2] = s.delta_pos      # no rotation
    def short(agent):      # an anchor that is not selected needs none either
        elsewhere(agent)
        for s in agent.segments:
            s.anchor_len = [len_ - (a == 0) for a, len_ in enumerate(s.anchor_len)]
    assert step(W, shared).calls == both([0, 1, 2, 3])
    assert [hotpath._rotations(s) for s in step(W, shared).agent.segments] == [14, 15, 17, 17]
    assert [hotpath._rotations(s) for s in step(W, short).agent.segments] == [16] * 4


def ragged(agent):
    """Lengths and pools of which no segment's own scratch holds the launch of them all."""
    agent.segments[:] = [workloads.make_segment(scaled(RAGGED, seg_len=S, n_anchors=A), 0, j)
                         for j, (S, A) in enumerate(zip((595, 772, 354, 378, 1022), (12, 13, 10, 15, 11)))]


class Consecutive(type(W)):
    def seg_offset(self, j):
        return self.prefix_len + sum((595, 772, 354, 378, 1022)[:j])


RAGGED = scaled(W, n_layers=32, n_kv_heads=8, n_q_heads=8, n_segments=5, seg_len=625)


def test_runs_fit_the_scratch_that_there_is(step, monkeypatch):
    """A run whose scratch is too small for it is shortened before anything is launched, nothing is refused, nothing is done twice."""
    monkeypatch.setattr(workloads, "_normal", lambda shape, sigma, dtype, g, device: torch.empty(1, dtype=dtype).expand(shape))
    monkeypatch.setattr(binding, "apart", lambda *a: True)      # (tensors without memory of their own)
    w, m = Consecutive(**vars(RAGGED)), hotpath.model_of(RAGGED)
    own = lambda agent: [hotpath.Scratch(m, s.base_k.shape[2], len(s.anchor_k), kv.W_TOKEN, "cpu") for s in agent.segments]
    for scratches in (own, None):
        lib = step(w, ragged, scratches)
        runs = [idx for name, idx in lib.calls if name == "weights"]
        assert lib.calls == both(*runs) and sum(runs, []) == list(range(5)) and lib.declined == 0
        assert len(runs) == (2 if scratches else 1), runs
    few = lambda agent: [small(s) for s in plain(agent)]

    def small(s):
        s.workspace = s.workspace[:kv.kvcomm_anchor_weights_workspace(M, W.seg_len, W.n_anchors)]
        return s
    lib = step(W, scratches=few)
    assert lib.calls == each_alone(4) and lib.declined == 0
    # weights per layer and head whose joint scratch would pass the limit of what a segment keeps
    big = scaled(RAGGED, n_segments=3, seg_len=600, n_anchors=8)
    lib = step(big, scratches=lambda agent: [hotpath.Scratch(m, 600, 8, kv.W_LAYER_HEAD_TOKEN, "cpu") for _ in range(3)],
               gran=kv.W_LAYER_HEAD_TOKEN)
    assert lib.calls == each_alone(3) and lib.declined == 0


def test_what_is_refused_all_the_same(step):
    """Refused together, the segments are tried one by one, matched again only if they have not been; what the runtime refuses (-4) and
    the caller's own mistakes end the step."""
    for status in (-1, -2):
        assert step(W, refuse={"align": status}).calls == [("weights", [0, 1, 2, 3])]
        assert step(W, refuse={"align": status}).attempts == [("align", [0, 1, 2, 3]), ("align", [0])]
    assert step(W, refuse={"together": -2}).calls == [("weights", [0, 1, 2, 3])] + [("align", [j]) for j in range(4)]
    lib = step(W, refuse={"weights": -1})
    assert lib.calls == [] and lib.error == -1 and lib.attempts == [("weights", [0, 1, 2, 3]), ("weights", [0])]
    for name, before in (("weights", []), ("align", [("weights", [0, 1, 2, 3])])):
        lib = step(W, refuse={name: -4})
        assert lib.error == -4 and lib.calls == before and lib.attempts == [(name, [0, 1, 2, 3])]


def test_pools_without_deviations(step):
    """A segment that is matched, but has no deviations to add, is rotated only: the single update accepts that."""
    def bare(agent):
        agent.segments[1].anchor_dk = agent.segments[1].anchor_dv = []
    def fewer(agent):      # (refused by the single update)
        agent.segments[2].anchor_dv = agent.segments[2].anchor_dv[:3]
    for scratches in (None, plain):
        assert step(W, bare, scratches).calls == each_alone(4)
        assert step(W, fewer, scratches).calls == each_alone(4)


@pytest.mark.parametrize("kind", [tuple, collections.deque, lambda s: dict(enumerate(s)), lambda s: list(s) + list(s)])
def test_scratch_in_any_container(step, kind):
    lib = step(W, scratches=lambda agent: kind(plain(agent)))
    assert lib.calls == both([0, 1, 2, 3])


def test_scratch_that_lacks_something(step):
    """(The single calls make what is not given, or need less.)"""
    for name in ("nearest", "selected", "workspace"):
        def lacks(agent):
            sc = plain(agent)
            setattr(sc[2], name, None)
            return sc
        assert step(W, scratches=lacks).calls == each_alone(4), name
    class Own:
        weights = nearest = selected = workspace = None
    assert step(W, scratches=lambda agent: [Own()] * 4).calls == each_alone(4)
    with pytest.raises(IndexError):
        step(W, scratches=lambda agent: plain(agent)[:3])


def test_scratch_that_segments_share(step):
    """One workspace for all is one launch's; outputs, or an output in another segment's workspace, are not."""
    def shared(agent):
        sc = plain(agent)
        for s in sc:
            s.workspace = sc[0].workspace
        return sc
    assert step(W, scratches=shared).calls == both([0, 1, 2, 3])
    def carved(agent):
        sc = plain(agent)
        sc[1].weights = sc[0].workspace[:sc[1].weights.numel() * 4].view(torch.float32).view(sc[1].weights.shape)
        return sc
    assert step(W, scratches=carved).calls == each_alone(4)
    def in_cache(agent):
        sc = plain(agent)
        sc[0].workspace = agent.cache_k.view(-1).view(torch.uint8)
        return sc
    assert step(W, scratches=in_cache).calls == each_alone(4)
    assert step(W, scratches=lambda agent: [plain(agent)[0]] * 4).calls == each_alone(4)


def test_scratch_of_one_segment_holds_one(monkeypatch):
    """What align_segment makes for itself is for that segment only; a Scratch that is kept also holds a launch of several like it."""
    kv.load_library()
    for name in ("kvcomm_anchor_weights", "kvcomm_align_kv"):
        monkeypatch.setattr(binding, name, lambda *a: None)
    seg = workloads.make_agent(W, 0).segments[0]
    one = kv.kvcomm_anchor_weights_workspace(M, W.seg_len, W.n_anchors)
    assert hotpath.align_segment(M, seg, None, None).workspace.numel() == max(one, 256)
    four = kv.kvcomm_anchor_weights_batch_workspace(M, [W.seg_len] * 4, [W.n_anchors] * 4)
    assert hotpath.Scratch(M, W.seg_len, W.n_anchors, kv.W_TOKEN, "cpu").workspace.numel() == max(four, 256) > one


@pytest.mark.parametrize("at", [[(0, 3), (3, 4), (7, 3)], [(2, 3), (6, 1), (7, 2)], [(4, 6)], [(5, 2), (1, 3)], [(1, 4), (4, 2)], [(7, 5)], [(3, 0), (3, 2)], [(10, 2)], [(-2, 1)]])
def test_slots_of_a_cache(at):
    """The rows that slices give, also of segments with gaps between them, out of order, on each other or past the end."""
    cache = torch.arange(2 * 3 * 10 * 4).view(2, 3, 10, 4)
    for c in (cache, cache.transpose(0, 1), cache[:, :, :, ::2]):
        for got, (p0, S) in zip(hotpath._slots(c, at), at):
            want = c[:, :, p0:p0 + S]
            assert got.shape == want.shape and got.stride() == want.stride() and torch.equal(got, want)
            assert got.numel() == 0 or got.data_ptr() == want.data_ptr()
