"""The native marshalling module against the ctypes code that it stands in for: the same bits from every entry point for every
form of arguments that it takes, and no call for those that it does not."""
import copy
import os
import subprocess
import sys
import sysconfig

import pytest
import torch

import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding

L, H, G, D = 3, 2, 2, 64
CALLS = ("suffix_attn_workspace", "anchor_weights", "anchor_weights_batch", "align_kv", "align_kv_q8", "align_kv_batch",
         "align_kv_q8_batch", "suffix_attn", "anchor_predict", "capture_offsets", "quantize_deltas")


class Declines:
    def __getattr__(self, name):
        return lambda *a: None


class Counts:
    """The native module, noting which of its functions took a call."""
    def __init__(self, native):
        self.native, self.took, self.declined = native, [], []

    def __getattr__(self, name):
        def call(*a):
            st = getattr(self.native, name)(*a)
            (self.declined if st is None else self.took).append(name)
            return st
        return call


def _views(dtype, dev, order):
    """[L, H, n, D] tensors: whole, as slices of longer caches, with heads before layers."""
    g = torch.Generator(device=dev)
    g.manual_seed(3)

    def make(n, sigma=1.0, h=H, dt=None):
        x = torch.randn((L, h, n, D) if order != "heads_first" else (h, L, n, D), generator=g, device=dev)
        if order == "slice":
            x = torch.cat([x, x, x], 2)[:, :, n:2 * n]
        elif order == "heads_first":
            x = x.permute(1, 0, 2, 3)
        return (x * sigma).to(dt or dtype) if order == "whole" else _like(x, (x * sigma).to(dt or dtype))
    return make


def _like(x, y):
    out = torch.empty_strided(x.shape, x.stride(), dtype=y.dtype, device=y.device)
    return out.copy_(y)


def _everything(dtype, order, seq, dev="cuda"):
    """One call of every entry point, with lists and numbers of type `seq`; returns all outputs."""
    m = kv.Model(L, H, H * G, D, dtype, 1e4)
    make = _views(dtype, dev, order)
    S, A = 21, 3
    anc, dk, dv = (seq(make(S + 2, s) for _ in range(A)) for s in (1.0, 0.1, 0.1))
    lens, adp = seq([S, S - 1, S + 2]), seq([5, 900, 64])
    bk, bv = make(S), make(S)
    new = lambda n, h=H: torch.zeros((L, h, n, D), dtype=dtype, device=dev)
    outs = []
    for gran in (kv.W_TOKEN, kv.W_LAYER_HEAD_TOKEN, kv.W_SEGMENT):
        for rule in (kv.RULE_L2_SOFTMAX, kv.RULE_NEAREST, kv.RULE_COSINE_SOFTMAX):
            outs.append(kv.kvcomm_anchor_weights_rule(m, rule, bk, anc, lens, 1, gran))
        w, near, sel = kv.kvcomm_anchor_weights(m, bk, anc, lens, 0.7, gran)
        outs += [w, near, sel, kv.kvcomm_align_kv(m, bk, bv, dk, dv, w, 64, new(S), new(S), lens, adp, gran),
                 kv.kvcomm_align_kv(m, bk, bv, dk, dv, w, 64, new(S), new(S), lens, None, gran)]
        cache_k, cache_v = new(2 * S + 4), new(2 * S + 4)
        wj = [dict(seg_base_k=bk, anchor_base_k=anc, anchor_len=lens), dict(seg_base_k=bv, anchor_base_k=anc)]
        got = kv.kvcomm_anchor_weights_batch(m, wj, 1.0, gran)
        aj = [dict(base_k=bk, base_v=bv, anchor_dk=dk, anchor_dv=dv, weights=got[j][0], delta_pos=3 + j * S, anchor_delta_pos=adp,
                   anchor_len=lens if j == 0 else None, out_k=cache_k[:, :, 3 + j * S:3 + j * S + S],
                   out_v=cache_v[:, :, 3 + j * S:3 + j * S + S]) for j in range(2)]
        kv.kvcomm_align_kv_batch(m, aj, gran)
        outs += [got, cache_k.clone(), cache_v.clone()]
        kv.kvcomm_align_kv_batch_beside(m, aj, 96, gran)
        outs += [cache_k.clone(), cache_v.clone()]
        q8 = lambda x: kv.kvcomm_quantize_deltas(m, x, 2.0 ** -8)
        dk8, dv8 = seq(q8(t) for t in dk), seq(q8(t) for t in dv)
        sc = seq([2.0 ** -8, 2.0 ** -7, 1])
        outs += [dk8, dv8, kv.kvcomm_align_kv_q8(m, bk, bv, dk8, dv8, sc, sc, w, 64, new(S), new(S), lens, adp, gran)]
        for j in aj:
            j.update(anchor_dk8=dk8, anchor_dv8=dv8, scale_k=sc, scale_v=sc)
        kv.kvcomm_align_kv_q8_batch(m, aj, gran)
        outs += [cache_k, cache_v, kv.kvcomm_anchor_predict(w, lens, S, 0.4, want_entropy=True)]
    outs.append(kv.kvcomm_capture_offsets(m, bk, bv, make(S), make(S), 77))
    for n_ctx, tq in ((0, 1), (40, 9), (700, 3)):
        q, k, v = make(tq, h=H * G), make(n_ctx + tq), make(n_ctx + tq)
        outs += [kv.kvcomm_suffix_attn(m, q, k, v, n_ctx), kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, 0.2, want_lse=True),
                 kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 16, stream=torch.cuda.current_stream()),
                 kv.kvcomm_suffix_attn_confined_ws(m, q, k, v, n_ctx, 9, 1)]
    torch.cuda.synchronize()
    return outs


def _flat(x):
    return [x] if isinstance(x, torch.Tensor) else [t for y in x for t in _flat(y)]


@pytest.mark.gpu
@pytest.mark.parametrize("order", ["whole", "slice", "heads_first"])
@pytest.mark.parametrize("dtype,seq", [(torch.bfloat16, list), (torch.float32, tuple)])
def test_the_same_bits_as_through_ctypes(monkeypatch, dtype, seq, order):
    print(f"marshalling: {dtype} {seq.__name__} {order}", flush=True)
    kv.load_library()
    counts = Counts(binding._native)
    monkeypatch.setattr(binding, "_native", counts)
    native = _flat(_everything(dtype, order, seq))
    assert set(counts.took) == set(CALLS) and not counts.declined
    monkeypatch.setattr(binding, "_native", Declines())
    general = _flat(_everything(dtype, order, seq))
    assert len(native) == len(general)
    for i, (a, b) in enumerate(zip(native, general)):
        assert a.dtype == b.dtype and torch.equal(a, b), f"output {i}"


class Sub(torch.Tensor):
    pass


def _device_odd_arguments():
    x = torch.randn((L, H, 12, D), device="cuda").to(torch.bfloat16)
    m = kv.Model(L, H, H * G, D, torch.bfloat16, 1e4)
    w = torch.full((12, 2), 0.5, device="cuda")
    good = dict(model=m, base_k=x, base_v=x, anchor_dk=[x, x], anchor_dv=[x, x], weights=w, delta_pos=3, out_k=torch.empty_like(x),
                out_v=torch.empty_like(x), anchor_len=[12, 12], anchor_delta_pos=[3, 3], gran=kv.W_TOKEN)
    odd = [dict(base_k=x.float()), dict(base_k=x.cpu()), dict(base_k=x.transpose(2, 3)), dict(base_k=x[0]), dict(base_k=None),
           dict(base_k=x.as_subclass(Sub)), dict(anchor_dk=[x, x[:, :, :11].contiguous()]), dict(anchor_dk=[x, x.float()]),
           dict(anchor_dk=[x]), dict(anchor_dk=[], anchor_dv=[], anchor_len=None, anchor_delta_pos=None), dict(anchor_len=[12]),
           dict(anchor_len=[12, 12, 12]), dict(anchor_len=[12, 12.0]), dict(anchor_delta_pos=[3]), dict(delta_pos=3.0),
           dict(delta_pos=1 << 40), dict(weights=None), dict(weights=w.double()), dict(weights=w[:6]), dict(weights=w.t()),
           dict(gran=True), dict(model=kv.Model(L, H, H * G, D, torch.float16, 1e4)), dict(anchor_dk=iter([x, x])),
           dict(anchor_dk=[x] * 65, anchor_dv=[x] * 65, anchor_len=[12] * 65, anchor_delta_pos=[3] * 65)]
    return good, odd


@pytest.mark.gpu
def test_what_is_not_plain_takes_the_general_path(monkeypatch):
    """Declined without a launch; then the general path's result or its error, as without the module."""
    kv.load_library()
    native = binding._native
    good, odd = _device_odd_arguments()

    def outcome(kw):
        kw = {k: (copy.copy(v) if k.startswith("anchor") and not isinstance(v, type(iter([]))) else v) for k, v in kw.items()}
        kw["out_k"], kw["out_v"] = torch.zeros_like(good["out_k"]), torch.zeros_like(good["out_v"])
        try:
            return [t.cpu() for t in kv.kvcomm_align_kv(**kw)]
        except Exception as e:
            return type(e), str(e)
    names = ("model", "gran", "base_k", "base_v", "anchor_dk", "anchor_dv", "weights", "delta_pos", "out_k", "out_v", "anchor_len",
             "anchor_delta_pos")
    assert native.align_kv(*(good[n] for n in names), None) == 0
    for i, change in enumerate(odd):
        print(f"marshalling: odd argument {i}", flush=True)
        kw = {**good, **change}
        assert native.align_kv(*(kw[n] for n in names), None) is None, (i, list(change))
        if isinstance(kw["anchor_dk"], type(iter([]))):
            continue
        monkeypatch.setattr(binding, "_native", native)
        a = outcome(kw)
        monkeypatch.setattr(binding, "_native", Declines())
        b = outcome(kw)
        assert type(a) is type(b)
        assert a == b if isinstance(a, tuple) else all(torch.equal(x, y) for x, y in zip(a, b))
    seen, x = [], good["base_k"]
    batched = lambda t: (seen.append(native.align_kv(good["model"], 0, t, *(good[n] for n in names[3:]), None)), t)[1]
    torch.vmap(batched)(torch.stack([x, x]))
    torch.func.grad(lambda t: batched(t).float().sum())(x)
    assert seen == [None, None]
    torch.cuda.synchronize()


def test_host_tensors_and_wrappers_are_declined():
    kv.load_library()
    native, m = binding._native, kv.Model(L, H, H * G, D, torch.bfloat16, 1e4)
    x = torch.zeros((L, H, 12, D), dtype=torch.bfloat16)
    w = torch.full((12, 1), 1.0)
    call = lambda t: native.align_kv(m, 0, t, t, [t], [t], w, 3, t, t, None, None, None)
    assert call(x) is None and call(x.as_subclass(Sub)) is None and call(x.to("meta")) is None
    seen = []
    torch.vmap(lambda t: (seen.append(call(t)), t)[1])(torch.stack([x, x]))
    assert seen == [None]
    assert native.suffix_attn_workspace(m, 2560, 512) == kv.kvcomm_suffix_attn_workspace(m, 2560, 512)
    for bad in ((m, 1.0, 1), (m, 1 << 40, 1), (None, 1, 1), (kv.Model(L, H, H, D, torch.float16, 1e4), 1, 1), (m, True, 1)):
        assert native.suffix_attn_workspace(*bad) is None
    with pytest.raises(TypeError):
        native.suffix_attn_workspace(m, 1)


@pytest.mark.parametrize("why", ["missing", "another torch"])
def test_the_library_works_without_the_module(monkeypatch, why):
    """No _marshal, or one built against another torch: a warning, and every call through ctypes."""
    m = kv.Model(L, H, H * G, D, torch.bfloat16, 1e4)
    want = kv.kvcomm_suffix_attn_workspace(m, 2560, 512)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    if why == "missing":
        monkeypatch.delattr(kv, "_marshal", raising=False)
        monkeypatch.setitem(sys.modules, kv.__name__ + "._marshal", None)
    else:
        monkeypatch.setattr(binding, "MARSHAL_FOR", "torch 1.0, Python 3.0")
    with pytest.warns(RuntimeWarning, match="_marshal"):
        binding.load_library()
    assert kv.kvcomm_suffix_attn_workspace(m, 2560, 512) == want
    assert binding._native.suffix_attn_workspace(m, 2560, 512) is None and binding._native.align_kv() is None
    x = torch.zeros((L, H, 12, D), dtype=torch.bfloat16)
    with pytest.raises(kv.KVCommError, match="device tensor"):     # refused by the ctypes code, as with the module
        kv.kvcomm_quantize_deltas(m, x, 1.0)


# A module that makes tensors which say that they lie in device memory (their address is never used), and a library call that
# takes a while.
FAKE_DEVICE = r"""
#include <torch/csrc/autograd/python_variable.h>
#include <unistd.h>
extern "C" int slow_call(...) { usleep(300000); return 0; }
static PyObject *tensor(PyObject *, PyObject *)
{
    const c10::Device dev(c10::DeviceType::CUDA, 0);
    c10::Storage st(c10::Storage::use_byte_size_t(), 1 << 20, c10::DataPtr((void *)0x100000, dev), nullptr, false);
    at::Tensor t = at::detail::make_tensor<c10::TensorImpl>(std::move(st), c10::DispatchKeySet(c10::DispatchKey::CUDA), caffe2::TypeMeta::Make<float>());
    t.unsafeGetTensorImpl()->set_sizes_contiguous({4, 4});
    return THPVariable_Wrap(t);
}
static PyObject *address(PyObject *, PyObject *) { return PyLong_FromVoidPtr((void *)&slow_call); }
static PyMethodDef methods[] = {{"tensor", tensor, METH_NOARGS, nullptr}, {"address", address, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "fake_device", nullptr, -1, methods};
PyMODINIT_FUNC PyInit_fake_device(void) { return PyModule_Create(&module); }
"""

EXIT = r"""
import sys, threading, time
sys.path[:0] = sys.argv[1:3]
import torch, fake_device
import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding
kv.load_library()
binding._native.bind({n: fake_device.address() for n in binding._NATIVE_CALLS}, binding.Model, lambda: 0, lambda d: 0)
t, entered = fake_device.tensor(), threading.Event()
def work():
    entered.set()
    binding._native.anchor_predict(t, [1, 1, 1, 1], 1, 0.5, None, t, None, None)
    raise SystemError("the call was declined")
threading.Thread(target=work, daemon=True).start()
entered.wait()
time.sleep(0.1)      # the thread is inside the call, without the interpreter lock
class Late:
    def __del__(self, sleep=time.sleep):
        sleep(0.6)   # ... and comes back during the shutdown
late = Late()
"""


def test_a_call_that_outlives_the_interpreter_ends_its_thread_only(tmp_path):
    """A daemon thread whose call returns while the interpreter shuts down is ended where it asks for the lock again; that must not
    reach std::terminate, nor be taken for a call that was declined."""
    top = os.path.dirname(torch.__file__)
    (tmp_path / "fake.cpp").write_text(FAKE_DEVICE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    "-isystem", os.path.join(top, "include"), "-isystem", os.path.join(top, "include", "torch", "csrc", "api", "include"),
                    "-isystem", sysconfig.get_paths()["include"], "-o", str(tmp_path / "fake_device.so"), str(tmp_path / "fake.cpp"),
                    "-L", os.path.join(top, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"], check=True)
    ran = subprocess.run([sys.executable, "-c", EXIT, str(tmp_path),
                          os.path.dirname(os.path.dirname(os.path.abspath(kv.__file__)))], capture_output=True, text=True, timeout=120)
    assert ran.returncode == 0, (ran.returncode, ran.stderr[-2000:])
