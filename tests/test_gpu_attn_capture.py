"""A HIP graph captured without torch: torch's allocator does not know of it, so scratch that the binding made during the capture
would be handed out again while the graph still writes to it.  The call has to do without."""
import ctypes

import pytest
import torch

import oracle
import paper_2510_12872_amd as kv
from paper_2510_12872_amd import binding

from parity import check_close, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _hip(name, *args):
    fn = getattr(binding.load_library(), name)    # the HIP runtime that the library is linked to
    fn.restype = ctypes.c_int
    status = fn(*args)
    assert status == 0, f"{name}: {status}"


@pytest.mark.parametrize("n_ctx,tq", [(3100, 1), (1500, 330)])
@pytest.mark.parametrize("confined,mode", [(False, 2), (True, 2), (False, 0)])   # mode: relaxed, relaxed, global
def test_capture_that_torch_does_not_manage(n_ctx, tq, confined, mode):
    print(f"attention in a graph captured without torch: n_ctx{n_ctx} tq{tq} confined {confined} mode {mode}", flush=True)
    m = kv.Model(1, 8, 32, 128, torch.bfloat16, 5e5)
    need = kv.kvcomm_suffix_attn_workspace(m, n_ctx, tq)
    assert need > 0
    g = torch.Generator(device=DEV)
    g.manual_seed(tq)
    mk = lambda h, n: torch.randn((1, h, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = mk(32, tq), mk(8, n_ctx + tq), mk(8, n_ctx + tq)
    out = torch.empty_like(q)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())

    def call():
        if confined:
            kv.kvcomm_suffix_attn_confined(m, q, k, v, n_ctx, 100, out=out, stream=side)
        else:
            kv.kvcomm_suffix_attn(m, q, k, v, n_ctx, out=out, stream=side)

    call()
    torch.cuda.synchronize()
    s = ctypes.c_void_p(side.cuda_stream)
    graph, execg = ctypes.c_void_p(), ctypes.c_void_p()
    if mode == 0:
        torch.cuda.empty_cache()     # nothing cached: the allocator asks the runtime for memory during the capture
    _hip("hipStreamBeginCapture", s, mode)
    call()
    _hip("hipStreamEndCapture", s, ctypes.byref(graph))
    _hip("hipGraphInstantiate", ctypes.byref(execg), graph, None, None, ctypes.c_size_t(0))
    with torch.cuda.stream(side):          # what takes up memory that was returned during the capture
        later = [torch.full((need,), 0x5A, dtype=torch.uint8, device=DEV) for _ in range(3)]
    out.zero_()
    torch.cuda.synchronize()
    for _ in range(2):
        _hip("hipGraphLaunch", execg, s)
    torch.cuda.synchronize()
    assert all(bool((t == 0x5A).all()) for t in later)
    check_close(to_np(out), oracle.suffix_attn(to_np(q), to_np(k), to_np(v), n_ctx), torch.bfloat16, "O")
    _hip("hipGraphExecDestroy", execg)
    _hip("hipGraphDestroy", graph)
