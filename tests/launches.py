"""Which kernels a call launches, with which grids, seen without a GPU: the library runs in a process of its own in which a
few functions of the HIP runtime are replaced by recording ones (nothing is executed, so any pointers will do)."""
import json
import os
import subprocess
import sys

from paper_2510_12872_amd import build

F32, BF16 = 0, 1   # dtype codes

RECORDER = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
static struct { const void *fn; const char *name; } fns[1024];
static int n_fns;
static struct { const void *fn; unsigned grid[3], block[3]; size_t lds; } rec[256];
static int n_rec;
static void *module;
void **__hipRegisterFatBinary(const void *data) { (void)data; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *hv, char *dv, int e, size_t s, int c, int g)
{ (void)m; (void)v; (void)hv; (void)dv; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *fn, char *df, const char *name, unsigned lim, void *a, void *b, void *c,
                           void *d, int *e)
{
    (void)m; (void)df; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_fns < 1024) { fns[n_fns].fn = fn; fns[n_fns++].name = name; }
}
int hipLaunchKernel(const void *fn, dim3_t g, dim3_t b, void **args, size_t lds, void *stream)
{
    (void)args; (void)stream;
    if (n_rec < 256) {
        rec[n_rec].fn = fn;
        rec[n_rec].lds = lds;
        memcpy(rec[n_rec].grid, &g, 12);
        memcpy(rec[n_rec++].block, &b, 12);
    }
    return 0;
}
int rec_count(void) { return n_rec; }
void rec_clear(void) { n_rec = 0; }
const char *rec_name(int i) { for (int f = 0; f < n_fns; ++f) if (fns[f].fn == rec[i].fn) return fns[f].name; return ""; }
unsigned rec_grid(int i, int axis) { return rec[i].grid[axis]; }
unsigned rec_block(int i, int axis) { return rec[i].block[axis]; }
size_t rec_lds(int i) { return rec[i].lds; }
"""

DRIVER = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)     # ahead of the HIP runtime in the lookup order
lib = ctypes.CDLL(sys.argv[2])
i32, f32, vp, sz = ctypes.c_int32, ctypes.c_float, ctypes.c_void_p, ctypes.c_size_t
class Model(ctypes.Structure):
    _fields_ = [(n, i32) for n in ("L", "hkv", "hq", "D", "dtype")] + [("theta", ctypes.c_double)]
class Tensor(ctypes.Structure):
    _fields_ = [("ptr", vp), ("sl", ctypes.c_int64), ("sh", ctypes.c_int64), ("st", ctypes.c_int64)]
shim.rec_name.restype = ctypes.c_char_p
shim.rec_grid.restype = ctypes.c_uint
lib.kvcomm_suffix_attn_workspace.restype = sz
lib.kvcomm_suffix_attn_workspace.argtypes = [vp, i32, i32]
attn = [vp, Tensor, Tensor, Tensor, i32, i32, f32, Tensor, vp]
lib.kvcomm_suffix_attn.argtypes = attn + [vp, sz, vp]
lib.kvcomm_suffix_attn_confined_ws.argtypes = attn + [i32, vp, sz, vp]
res = []
for L, hkv, G, D, dtype, n_ctx, tq, max_blocks, scratch in json.load(sys.stdin):
    m = Model(L, hkv, hkv * G, D, dtype, 1e4)
    t = lambda h, n: Tensor(0x1000, h * n * D, n * D, D)
    need = lib.kvcomm_suffix_attn_workspace(ctypes.byref(m), n_ctx, tq)
    ws = (0x1000, need) if scratch and need else (None, 0)
    a = (ctypes.byref(m), t(hkv * G, tq), t(hkv, n_ctx + tq), t(hkv, n_ctx + tq), n_ctx, tq, 0.0, t(hkv * G, tq), None)
    shim.rec_clear()
    st = lib.kvcomm_suffix_attn_confined_ws(*a, max_blocks, *ws, None) if max_blocks else lib.kvcomm_suffix_attn(*a, *ws, None)
    res.append(dict(status=st, workspace=need,
                    launches=[(shim.rec_name(i).decode(), [shim.rec_grid(i, k) for k in range(3)]) for i in range(shim.rec_count())]))
json.dump(res, sys.stdout)
"""


ALIGN_DRIVER = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
class Model(ctypes.Structure):
    _fields_ = [(n, i32) for n in ("L", "hkv", "hq", "D", "dtype")] + [("theta", ctypes.c_double)]
class Tensor(ctypes.Structure):
    _fields_ = [("ptr", vp), ("sl", i64), ("sh", i64), ("st", i64)]
class Job(ctypes.Structure):
    _fields_ = [(n, Tensor) for n in ("bk", "bv", "ok", "ov")] + [("S", i32), ("delta", i32), ("dk", vp), ("dv", vp), ("len", vp), ("adp", vp),
                ("n", i32), ("w", vp), ("slots", i64)]
shim.rec_name.restype = ctypes.c_char_p
shim.rec_grid.restype = shim.rec_block.restype = ctypes.c_uint
shim.rec_lds.restype = ctypes.c_size_t
res = []
for L, H, D, dtype, lens, pools, units in json.load(sys.stdin):
    keep, jobs, at = [], (Job * len(lens))(), [1 << 44]
    def place():                      # tensors that share no bytes
        at[0] += 1 << 40
        return at[0]
    for j, (S, n) in enumerate(zip(lens, pools)):
        t = lambda: Tensor(place(), H * S * D, S * D, D)
        anc, ln = (vp * max(n, 1))(*[place()] * n), (i32 * max(n, 1))(*[S] * n)
        keep += [anc, ln]
        jobs[j] = Job(t(), t(), t(), t(), S, 3, ctypes.addressof(anc), ctypes.addressof(anc), ctypes.addressof(ln), None, n, place(), S)
    shim.rec_clear()
    cap = max(lens)
    lib.kvcomm_align_kv_batch.argtypes = [vp, i32, Tensor, vp, i32, vp]
    lib.kvcomm_align_kv_batch_beside.argtypes = [vp, i32, Tensor, vp, i32, i32, vp]
    a = (ctypes.byref(Model(L, H, H, D, dtype, 1e4)), 0, Tensor(None, H * cap * D, cap * D, D), jobs, len(lens))
    st = lib.kvcomm_align_kv_batch(*a, None) if units is None else lib.kvcomm_align_kv_batch_beside(*a, units, None)
    res.append(dict(status=st, launches=[dict(name=shim.rec_name(i).decode(), grid=[shim.rec_grid(i, k) for k in range(3)],
                                              block=[shim.rec_block(i, k) for k in range(3)], lds=shim.rec_lds(i)) for i in range(shim.rec_count())]))
json.dump(res, sys.stdout)
"""


def record(tmp_path, driver, calls):
    """What `driver` prints for `calls` with the recorder in the HIP runtime's place."""
    src, shim = tmp_path / "rec.c", tmp_path / "librec.so"
    src.write_text(RECORDER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(shim), str(src)], check=True)
    lib = os.environ.get("KVCOMM_LIBRARY") or build.LIB
    ran = subprocess.run([sys.executable, "-c", driver, str(shim), lib], input=json.dumps([list(c) for c in calls]),
                         capture_output=True, text=True)
    assert ran.returncode == 0, ran.stderr[-2000:]
    return json.loads(ran.stdout)


def attention_launches(tmp_path, calls):
    """calls: (L, Hkv, G, D, dtype code, n_ctx, tq, max_blocks or 0, with scratch) -> per call its status, the size of its
    workspace and the launches as (mangled kernel name, grid)."""
    return record(tmp_path, DRIVER, calls)


def align_launches(tmp_path, calls):
    """Batched updates with per-token weights; calls: (L, Hkv, D, dtype code, segment lengths, anchors per segment, units or None) -> per call
    its status and its launches."""
    return record(tmp_path, ALIGN_DRIVER, calls)
