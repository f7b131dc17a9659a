"""Host-side sequencing of the reuse step: three library calls per segment/agent.

Nothing is computed here; the functions only issue the calls of include/kvcomm.h in the
order of the reuse branch of Algorithm 1 (weights -> offset approximation per placeholder,
then attention over the concatenated cache), on the current stream or, for consecutive
agents, on two streams (TwoStreamPipeline).
"""
import functools

import torch

from . import binding as kv


def model_of(w):
    """kvcomm model descriptor of a workloads.Workload."""
    return kv.Model(w.n_layers, w.n_kv_heads, w.n_q_heads, w.head_dim, w.dtype, w.rope_theta)


# Up to here a segment's workspace also holds the launch that it shares with as many segments like it as a launch takes (with other
# lengths and pools beside it a run may need more than any of its segments holds: it is shortened then, see _joint_runs()).  32 layers x 8 heads: 77
# tokens, 6 anchors 2.5 MB instead of 0.3, 512 tokens, 8 anchors 4.2 instead of 0.8.  Per-token weights stay below the limit in general (1024
# tokens, 16 anchors: 6 MiB); weights per layer and head pass it with segments that keep the chip busy each by itself (134 MB), and
# those go one after the other.
JOINT_WORKSPACE = 16 << 20


class Scratch:
    """Reusable device buffers for the weight step (so a timed loop allocates nothing)."""

    def __init__(self, model, seg_len, n_anchors, gran, device, joint=True):
        n = kv.kvcomm_weight_slots(model, seg_len, gran)
        self.weights = torch.empty((n, n_anchors), dtype=torch.float32, device=device)
        self.nearest = torch.empty((n,), dtype=torch.int32, device=device)
        self.selected = torch.empty((n_anchors,), dtype=torch.int32, device=device)
        need = kv.kvcomm_anchor_weights_workspace(model, seg_len, n_anchors, gran)
        together = max(1, min(kv.MAX_BATCH, kv.MAX_ANCHORS // max(1, n_anchors))) if joint else 1   # a launch of reuse_agent takes so many like it
        if together > 1:
            all_need = kv.kvcomm_anchor_weights_batch_workspace(model, [seg_len] * together, [n_anchors] * together, gran)
            if all_need <= JOINT_WORKSPACE:
                need = max(need, all_need)
        self.workspace = torch.empty((max(need, 256),), dtype=torch.uint8, device=device)


def align_segment(model, seg, out_k, out_v, temperature=1.0, gran=kv.W_TOKEN, scratch=None, stream=None):
    """Anchor weights, then aligned K/V of one segment written into out_k / out_v."""
    if scratch is None:
        with kv.on_stream(stream):
            scratch = Scratch(model, seg.base_k.shape[2], len(seg.anchor_k), gran, seg.base_k.device, joint=False)
    kv.kvcomm_anchor_weights(model, seg.base_k, seg.anchor_k, seg.anchor_len, temperature, gran,
                             scratch.weights, scratch.nearest, scratch.selected, scratch.workspace, stream)
    kv.kvcomm_align_kv(model, seg.base_k, seg.base_v, seg.anchor_dk, seg.anchor_dv, scratch.weights,
                       seg.delta_pos, out_k, out_v, seg.anchor_len, seg.anchor_delta_pos, gran, stream)
    return scratch


def launch_chunks(n_anchors):
    """Cut the segments of an agent (given by their anchor counts) into launches: one launch carries at
    most MAX_BATCH segments and MAX_ANCHORS anchors over all of them."""
    chunks, cur, n_anc = [], [], 0
    for j, a in enumerate(n_anchors):
        if cur and (len(cur) == kv.MAX_BATCH or n_anc + a > kv.MAX_ANCHORS):
            chunks.append(cur)
            cur, n_anc = [], 0
        cur.append(j)
        n_anc += a
    if cur:
        chunks.append(cur)
    return chunks


class AgentScratch:
    """Reusable device buffers for the batched weight step of all segments of one agent."""

    def __init__(self, model, seg_lens, n_anchors, gran, device, rule=kv.RULE_L2_SOFTMAX):
        self.weights, self.nearest, self.selected = [], [], []
        for S, A in zip(seg_lens, n_anchors):
            n = kv.kvcomm_weight_slots(model, S, gran)
            self.weights.append(torch.empty((n, A), dtype=torch.float32, device=device))
            self.nearest.append(torch.empty((n,), dtype=torch.int32, device=device))
            self.selected.append(torch.empty((A,), dtype=torch.int32, device=device))
        seg_lens, n_anchors = list(seg_lens), list(n_anchors)
        need = max(kv.kvcomm_anchor_weights_batch_workspace(model, [seg_lens[j] for j in c], [n_anchors[j] for j in c],
                                                            gran, rule) for c in launch_chunks(n_anchors))
        self.workspace = torch.empty((max(need, 256),), dtype=torch.uint8, device=device)


def _match_together(w, model, agent, idx, outs, workspace, gran, stream):
    """One batched call for the weights of the agent's segments `idx`; outs[j]: weights, nearest and selected of segment j."""
    segs = agent.segments
    kv.kvcomm_anchor_weights_batch(model, [dict(
        seg_base_k=segs[j].base_k, anchor_base_k=segs[j].anchor_k, anchor_len=segs[j].anchor_len,
        weights_out=outs[j][0], nearest_out=outs[j][1], selected_out=outs[j][2])
        for j in idx], w.temperature, gran, workspace=workspace, stream=stream)


def _update_together(model, agent, idx, outs, at, gran, stream):
    """One batched call for their update; at[j]: first row and rows of segment j's slot."""
    at = [at[j] for j in idx]
    kv.kvcomm_align_kv_batch(model, [dict(
        base_k=s.base_k, base_v=s.base_v, anchor_dk=s.anchor_dk, anchor_dv=s.anchor_dv, anchor_len=s.anchor_len, weights=outs[j][0],
        delta_pos=s.delta_pos, anchor_delta_pos=s.anchor_delta_pos, out_k=out_k, out_v=out_v)
        for j, s, out_k, out_v in zip(idx, [agent.segments[j] for j in idx], _slots(agent.cache_k, at), _slots(agent.cache_v, at))],
        gran, stream)


def align_agent_batched(w, model, agent, gran=kv.W_TOKEN, scratch=None, stream=None):
    """Anchor weights, then aligned K/V of ALL segments of an agent: one batched call per step and
    chunk of segments (a launch holds at most MAX_BATCH segments and MAX_ANCHORS anchors)."""
    segs = agent.segments
    if scratch is None:
        with kv.on_stream(stream):
            scratch = AgentScratch(model, [s.base_k.shape[2] for s in segs], [len(s.anchor_k) for s in segs], gran,
                                   segs[0].base_k.device)
    outs = list(zip(scratch.weights, scratch.nearest, scratch.selected))
    at = [(w.seg_offset(j), s.base_k.shape[2]) for j, s in enumerate(segs)]
    for idx in launch_chunks([len(s.anchor_k) for s in segs]):
        _match_together(w, model, agent, idx, outs, scratch.workspace, gran, stream)
        _update_together(model, agent, idx, outs, at, gran, stream)
    return scratch


def _slot(cache, p0, S):
    """Rows [p0, p0 + S) of a cache."""
    return cache.narrow(2, p0, S) if 0 <= p0 <= cache.shape[2] - S else cache[:, :, p0:p0 + S]   # (narrow: half the time of an index)


def _slots(cache, at):
    """Rows [p0, p0 + S) of a cache for each (p0, S): one call for all where they follow each other (half the time of one each)."""
    sizes, slots, end = [], [], 0
    for p0, S in at:
        if p0 != end:
            sizes.append(p0 - end)
        slots.append(len(sizes))
        sizes.append(S)
        end = p0 + S
    sizes.append(cache.shape[2] - end)
    if min(sizes) < 0:
        return [_slot(cache, p0, S) for p0, S in at]
    parts = cache.split_with_sizes(sizes, 2)
    return [parts[i] for i in slots]


def _rotations(seg):
    """Rotations that the update of a segment needs at most: one per distinct position delta of its keys and its selected deviations."""
    if seg.anchor_delta_pos is None:
        return 1
    S = seg.base_k.shape[2]
    lens = [t.shape[2] for t in seg.anchor_dk] if seg.anchor_len is None else seg.anchor_len
    return len(({seg.delta_pos} | {seg.delta_pos - d for d, n in zip(seg.anchor_delta_pos, lens) if n >= S}) - {0})


@functools.lru_cache(maxsize=256)
def _joint_need(model, lens, pools, gran):
    return kv.kvcomm_anchor_weights_batch_workspace(model, lens, pools, gran)


def _joint_runs(model, segs, lens, pools, gran, room):
    """Cuts the segments of an agent into runs of neighbours that the batched calls take together, known before anything is launched: the
    limits of launch_chunks(), anchors of one layout, the rotations of an update (four pools of 16 anchors, all recorded elsewhere, need 68
    and go as three segments and one), and the largest workspace among the segments' own scratch where that is given (room: its bytes)."""
    layouts = [(s.anchor_k[0].stride(), s.anchor_dk[0].stride()) for s in segs]
    rotations = [_rotations(s) for s in segs]
    runs, j, n = [], 0, len(segs)
    while j < n:
        k, anchors, rots = j + 1, pools[j], rotations[j]
        while k < n and k - j < kv.MAX_BATCH and layouts[k] == layouts[j]:
            anchors, rots = anchors + pools[k], rots + rotations[k]
            if anchors > kv.MAX_ANCHORS or rots > kv.MAX_ROTATIONS:
                break
            k += 1
        while room is not None and k - j > 1 and _joint_need(model, tuple(lens[j:k]), tuple(pools[j:k]), gran) > max(room[j:k]):
            k -= 1
        runs.append(range(j, k))
        j = k
    return runs


def _whole_scratch(scratches, n):
    """The Scratch of each of n segments: itself, its (weights, nearest, selected), its workspace's bytes, and all their tensors (a workspace that
    serves several once).  None where one is missing or lacks something (the single calls make that, or refuse it)."""
    tensor = torch.Tensor
    own, outs, room, tensors, spaces = [], [], [], [], {}
    try:
        for j in range(n):
            s = scratches[j]
            if not isinstance(s, Scratch):
                return None
            out = weights, nearest, selected = s.weights, s.nearest, s.selected
            space = s.workspace
            if not (isinstance(weights, tensor) and isinstance(nearest, tensor) and isinstance(selected, tensor) and isinstance(space, tensor)):
                return None
            own.append(s)
            outs.append(out)
            room.append(space.nbytes)
            tensors += out
            spaces[space.data_ptr()] = space
    except (IndexError, KeyError):
        return None
    tensors += spaces.values()
    return own, outs, room, tensors


def _align_all(w, model, agent, gran, scratches, stream):
    """Aligns the segments of an agent, those that may share a launch in one launch per step.  Returns False where none do; nothing has been launched
    then.  Segments may be matched together and then updated together where their slots, what the weights go to and the workspaces lie
    apart, and nothing else that is used lies in the agent's cache: a key or a delta in a slot that an earlier segment's update writes
    is read after that update."""
    segs, cache_k, cache_v = agent.segments, agent.cache_k, agent.cache_v
    n, outs, room, own, used = len(segs), None, None, (), []
    if scratches is not None:
        whole = _whole_scratch(scratches, n)
        if whole is None:
            return False
        scratches, outs, room, own = whole
    at, lens, pools, end, rotations, alike, layout = [], [], [], 0, 0, n <= kv.MAX_BATCH, None
    for j, s in enumerate(segs):
        base_k, pool, dk, dv, moved = s.base_k, s.anchor_k, s.anchor_dk, s.anchor_dv, s.anchor_delta_pos
        S, A, p0 = base_k.shape[2], len(pool), w.seg_offset(j)
        if p0 < end or A == 0 or len(dk) != A or len(dv) != A:   # (matched, but nothing to add: the single update takes that)
            return False
        end = p0 + S
        at.append((p0, S))
        lens.append(S)
        pools.append(A)
        used += ((base_k, s.base_v), pool, dk, dv)
        rotations += 1 if moved is None else 1 + len(moved)   # at most
        strides = pool[0].stride(), dk[0].stride()
        if strides != layout:
            alike, layout = alike and j == 0, strides
    if end > cache_k.shape[2] or end > cache_v.shape[2] or not kv.apart((cache_k, cache_v), used, own):
        return False
    if (alike and rotations <= kv.MAX_ROTATIONS and sum(pools) <= kv.MAX_ANCHORS and
            (room is None or _joint_need(model, tuple(lens), tuple(pools), gran) <= max(room))):
        runs = (range(n),)
    else:
        runs = _joint_runs(model, segs, lens, pools, gran, room)
    for idx in runs:
        if len(idx) == 1:
            _align_one(w, model, agent, idx[0], gran, scratches, stream)
        else:
            _align_run(w, model, agent, idx, at, gran, scratches, outs, room, stream)
    return True


def _refused(e):
    """Was this call refused for its arguments, so that nothing has been launched?"""
    return e.status in (kv.EINVAL, kv.EUNSUPPORTED, kv.EWORKSPACE)


def _align_run(w, model, agent, idx, at, gran, scratches, outs, room, stream):
    """Aligns the segments `idx` together, or, where that is refused, one after the other: so they may be accepted, or are refused as
    they always were.  outs: weights, nearest and selected of every segment, room: bytes of its workspace; None where these are to be made."""
    matched = False
    try:
        if scratches is None:
            segs = [agent.segments[j] for j in idx]
            with kv.on_stream(stream):
                made = AgentScratch(model, [s.base_k.shape[2] for s in segs], [len(s.anchor_k) for s in segs], gran, segs[0].base_k.device)
            outs, workspace = dict(zip(idx, zip(made.weights, made.nearest, made.selected))), made.workspace
        else:
            workspace = scratches[max(idx, key=room.__getitem__)].workspace
        _match_together(w, model, agent, idx, outs, workspace, gran, stream)
        matched = True
        return _update_together(model, agent, idx, outs, at, gran, stream)
    except torch.OutOfMemoryError:   # (only the scratch allocates)
        pass
    except kv.KVCommError as e:
        if not _refused(e):
            raise
    for j in idx:
        if matched:
            _update_one(w, model, agent, j, outs[j][0], gran, stream)
        else:
            _align_one(w, model, agent, j, gran, scratches, stream)


def _update_one(w, model, agent, j, weights, gran, stream):
    seg = agent.segments[j]
    p0, S = w.seg_offset(j), seg.base_k.shape[2]
    kv.kvcomm_align_kv(model, seg.base_k, seg.base_v, seg.anchor_dk, seg.anchor_dv, weights, seg.delta_pos, _slot(agent.cache_k, p0, S),
                       _slot(agent.cache_v, p0, S), seg.anchor_len, seg.anchor_delta_pos, gran, stream)


def _align_one(w, model, agent, j, gran, scratches, stream):
    """Segment j into its slot."""
    seg = agent.segments[j]
    p0, S = w.seg_offset(j), seg.base_k.shape[2]
    align_segment(model, seg, _slot(agent.cache_k, p0, S), _slot(agent.cache_v, p0, S),
                  w.temperature, gran, None if scratches is None else scratches[j], stream)


def reuse_agent(w, model, agent, out=None, gran=kv.W_TOKEN, scratches=None, stream=None):
    """Whole hot path for one agent: align every segment into its cache slot, then suffix attention.  Several segments go through the
    batched calls: a small agent's step is the number of its launches (4 segments of 10 tokens, 16 anchors, 2 layers x 8 heads: 74 us
    one after the other, 41 us so; as a graph 59 and 18 us).  The weights are then those of the shared launch, summed in another order
    (which the other segments and the size of the workspaces decide): within their tolerance, not bit for bit, align_segment's."""
    if len(agent.segments) < 2 or not _align_all(w, model, agent, gran, scratches, stream):
        for j in range(len(agent.segments)):
            _align_one(w, model, agent, j, gran, scratches, stream)
    if agent.q is None:
        return None
    return kv.kvcomm_suffix_attn(model, agent.q, agent.cache_k, agent.cache_v, w.n_ctx, out=out, stream=stream)


class TwoStreamPipeline:
    """The reuse step of consecutive agents on two streams: weights + alignment of an agent run beside the
    attention of the agent before it.  The attention is launched through kvcomm_suffix_attn_confined as at most
    `attn_blocks` persistent blocks, so that the other compute units are free for the memory-bound alignment
    kernels for the whole launch (attn_blocks = 0: the plain launch, which leaves them only the gaps).

    Ordering: an event per submission puts the attention behind its own alignment; a second one, kept per buffer
    key, puts the next alignment into the same cache behind the attention that still reads it.  HIP maps streams
    onto a few hardware queues and two streams that share one run one after the other: pick_attention_stream()
    tries candidates and keeps the fastest."""

    def __init__(self, model, temperature=1.0, attn_blocks=160, gran=kv.W_TOKEN, align_stream=None, attn_stream=None):
        self.model, self.temperature, self.attn_blocks, self.gran = model, temperature, attn_blocks, gran
        self.s_align = align_stream or torch.cuda.Stream()
        self.s_attn = attn_stream or torch.cuda.Stream()
        self._done = {}

    def fork(self):
        """Both streams wait for the work already queued on the current stream."""
        cur = torch.cuda.current_stream()
        self.s_align.wait_stream(cur)
        self.s_attn.wait_stream(cur)

    def join(self):
        """The current stream waits for everything submitted so far."""
        cur = torch.cuda.current_stream()
        cur.wait_stream(self.s_align)
        cur.wait_stream(self.s_attn)

    def submit(self, key, wjobs, ajobs, workspace, q, cache_k, cache_v, n_ctx, out, q8=False):
        """One agent: batched weights and alignment (job lists as for the batched calls) on the alignment stream,
        then its suffix attention on the attention stream.  `key` names the agent's buffers."""
        with torch.cuda.stream(self.s_align):
            if key in self._done:
                self.s_align.wait_event(self._done[key])
            kv.kvcomm_anchor_weights_batch(self.model, wjobs, self.temperature, self.gran, workspace=workspace)
            if q8:
                kv.kvcomm_align_kv_q8_batch(self.model, ajobs, self.gran)
            elif q is not None and 0 < self.attn_blocks < kv.COMPUTE_UNITS:
                kv.kvcomm_align_kv_batch_beside(self.model, ajobs, kv.COMPUTE_UNITS - self.attn_blocks, self.gran)
            else:
                kv.kvcomm_align_kv_batch(self.model, ajobs, self.gran)
            aligned = torch.cuda.Event()
            aligned.record(self.s_align)
        with torch.cuda.stream(self.s_attn):
            self.s_attn.wait_event(aligned)
            if q is not None:
                if self.attn_blocks > 0:
                    kv.kvcomm_suffix_attn_confined(self.model, q, cache_k, cache_v, n_ctx, self.attn_blocks, out=out)
                else:
                    kv.kvcomm_suffix_attn(self.model, q, cache_k, cache_v, n_ctx, out=out)
            done = torch.cuda.Event()
            done.record(self.s_attn)
            self._done[key] = done

    def pick_attention_stream(self, run_steps, candidates=None, warm=2, timed=3):
        """run_steps(n) must submit n steps through this pipeline (fork ... join).  Tries every candidate stream
        for the attention and keeps the one with the shortest steps."""
        import time
        candidates = candidates or [self.s_attn] + [torch.cuda.Stream() for _ in range(2)]
        best = None
        for cand in candidates:
            self.s_attn = cand
            run_steps(warm)
            torch.cuda.synchronize()
            t = time.perf_counter()
            run_steps(timed)
            torch.cuda.synchronize()
            t = time.perf_counter() - t
            if best is None or t < best[0]:
                best = (t, cand)
        self.s_attn = best[1]
        return best[1]
