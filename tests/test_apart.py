"""binding.apart(): which tensors come near each other, the native module's answer and the general one, for every form that a step asks about."""
import itertools

import pytest
import torch

import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding


def _tensors(dev):
    x = torch.zeros((4, 3, 10, 8), device=dev)
    y = torch.zeros((64,), device=dev)
    # a cache, its slots, rows interleaved with them, another order of its axes, neighbours that touch and that do not, nothing at all
    return [x, x[:, :, 2:5], x[:, :, 5:9], x[0], x[1], x.permute(2, 0, 1, 3)[3:4], x[..., ::2], y[:32], y[32:], y[31:33], y[:0], x[:, :0], y.view(torch.uint8)[128:129]]


def _bytes(t):
    if t.numel() == 0:   # (as if there were one element)
        return range(t.data_ptr(), t.data_ptr() + t.element_size())
    return range(t.data_ptr(), t.data_ptr() + t.element_size() * (1 + sum((n - 1) * s for n, s in zip(t.shape, t.stride()))))


def _want(own, groups, each):
    meet = lambda a, b: max(_bytes(a).start, _bytes(b).start) < min(_bytes(a).stop, _bytes(b).stop)
    return not (any(meet(a, b) for a in own for g in (*groups, each) for b in g) or any(meet(a, b) for a, b in itertools.combinations(each, 2)))


def _forms(dev):
    t = _tensors(dev)
    for a, b in itertools.product(range(len(t)), repeat=2):
        yield (t[a],), [(t[b],)], ()
        yield (t[a],), [], [t[a], t[b]]
        yield (), [[t[a], t[b]]], [t[b]]
        yield [t[a], t[7]], [[t[8]], [], [t[b]]], (t[1], t[2], t[b])
    yield (), (), ()


@pytest.mark.parametrize("dev", ["cpu", pytest.param("cuda", marks=pytest.mark.gpu)])
def test_apart(dev, monkeypatch):
    print(f"apart: {dev}", flush=True)
    kv.load_library()
    answers = []
    for form in _forms(dev):
        native = binding._native.apart(*form)
        assert (native is None) == (dev == "cpu" and any(map(bool, form))) or native == 1
        answers.append((form, native))
        assert kv.binding.apart(*form) is _want(*form)
    monkeypatch.setattr(binding, "_native", binding._Declines())
    for form, native in answers:
        assert kv.binding.apart(*form) is _want(*form) and native in (None, _want(*form))
