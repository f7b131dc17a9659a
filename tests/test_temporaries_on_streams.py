"""Memory that a call makes for itself and drops on return belongs to the stream its kernels run on: the allocator would give
memory of another stream to that stream's next user while the kernels still write it.  (CPU only: the library's calls are replaced.)"""
import contextlib

import pytest
import torch

import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding, hotpath, workloads
from paper_2510_12872_amd.workloads import scaled

W = scaled(workloads.LLAMA8B_5AGENTS, n_layers=1, n_kv_heads=2, n_q_heads=2, head_dim=64, prefix_len=2, seg_len=5, n_segments=2,
           n_anchors=3, tq=2)
M = hotpath.model_of(W)


class Handle:   # a stream of another library
    cuda_stream = 0x77


@pytest.fixture
def made(monkeypatch):
    """(stream that is current, bytes) of everything allocated."""
    made, current = [], [None]

    @contextlib.contextmanager
    def stream(s):
        current.append(s)
        yield
        current.pop()
    empty = torch.empty

    def noted(*a, **k):
        t = empty(*a, **k)
        made.append((current[-1], t.numel() * t.element_size()))
        return t
    kv.load_library()
    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda p: p)
    monkeypatch.setattr(torch, "empty", noted)
    return made


def test_scratch_of_a_step(monkeypatch, made):
    agent = workloads.make_agent(W, 0)
    for name in ("kvcomm_anchor_weights", "kvcomm_align_kv", "kvcomm_anchor_weights_batch", "kvcomm_align_kv_batch", "kvcomm_suffix_attn"):
        monkeypatch.setattr(binding, name, lambda *a, **k: None)
    seg, k, v = agent.segments[0], agent.cache_k[:, :, 2:7], agent.cache_v[:, :, 2:7]
    for step in (lambda s: hotpath.align_segment(M, seg, k, v, stream=s), lambda s: hotpath.align_agent_batched(W, M, agent, stream=s),
                 lambda s: hotpath.reuse_agent(W, M, agent, stream=s)):
        for given, want in ((None, None), (Handle, 0x77)):
            made.clear()
            step(given)
            assert made and all(s == want for s, _ in made)


def test_workspaces_of_the_calls(monkeypatch, made):
    """(Results that are returned stay on the current stream.)"""
    seg = workloads.make_segment(W, 0, 0)
    S, A = W.seg_len, W.n_anchors

    class Takes:
        def __getattr__(self, name):
            return lambda *a: 0
    monkeypatch.setattr(binding, "_native", Takes())

    class OnDevice:
        shape, dtype, is_cuda, device, dim, is_contiguous = (S, A), torch.float32, True, "cpu", lambda self: 2, lambda self: True
    out = [torch.zeros(S, A), torch.zeros(S, dtype=torch.int32), torch.zeros(A, dtype=torch.int32)]
    jobs = [dict(seg_base_k=seg.base_k, anchor_base_k=seg.anchor_k, weights_out=out[0], nearest_out=out[1], selected_out=out[2])]
    for call in (lambda s: kv.kvcomm_anchor_weights(M, seg.base_k, seg.anchor_k, None, 1.0, kv.W_TOKEN, *out, stream=s),
                 lambda s: kv.kvcomm_anchor_weights_rule(M, kv.RULE_COSINE_SOFTMAX, seg.base_k, seg.anchor_k, None, 1.0, kv.W_TOKEN, *out, stream=s),
                 lambda s: kv.kvcomm_anchor_weights_batch(M, jobs, stream=s),
                 lambda s: kv.kvcomm_anchor_predict(OnDevice(), [S] * A, S, 0.5, result_out=out[0], stream=s)):
        for given, want in ((None, None), (Handle, 0x77)):
            made.clear()
            call(given)
            assert len(made) == 1 and made[0][0] == want
