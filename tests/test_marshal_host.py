"""The binding's native marshalling hands the library what the ctypes path hands it, for every form of argument, and leaves to
that path what it does not read.  A stand-in library that only records its arguments takes the place of the HIP one."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORD = r"""
#include <string.h>
#include "moe_rbf.h"
long long seen[64];
int answer;
static int note(const moe_shape *s, const moe_plan_t *p, const void *a, const void *b, const void *c, const void *d, void *st) {
  memset(seen, 0, sizeof(seen));
  if (s) memcpy(seen, s, sizeof(*s));
  if (p) memcpy(seen + 8, p, sizeof(*p));
  seen[40] = !!s, seen[41] = !!p;
  const void *x[] = {a, b, c, d, st};
  memcpy(seen + 42, x, sizeof(x));
  ++seen[50];
  return answer;
}
int moe_plan(const moe_shape *s, const int32_t *k, moe_plan_t *p, void *st) { return note(s, p, k, 0, 0, (void *)1, st); }
int moe_plan_static(const moe_shape *s, const int32_t *k, moe_plan_t *p, void *st) { return note(s, p, k, 0, 0, (void *)2, st); }
int moe_dispatch(const moe_shape *s, const void *x, const int32_t *k, moe_plan_t *p, void *w, void *st) { return note(s, p, x, k, w, (void *)3, st); }
int moe_dispatch_quant(const moe_shape *s, const void *x, const int32_t *k, moe_plan_t *p, void *w, float *f, void *st) { return note(s, p, x, k, w, f, st); }
int moe_combine(const moe_shape *s, const void *e, const float *w, const moe_plan_t *p, void *y, void *st) { return note(s, p, e, w, y, (void *)4, st); }
int moe_workspace_bytes(const moe_shape *s, size_t *o) { *o = 512; return 0; }
int moe_window_rows(const moe_shape *s, int64_t *o) { *o = (int64_t)s->T * s->k; return 0; }
int moe_resolve_schedule(const moe_shape *s, int32_t *o) { *o = s->schedule; return 0; }
const char *moe_strerror(int c) { return "recorded"; }
const char *moe_last_launch_error(void) { return "none"; }
"""

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
import numpy as np, torch
import paper_2605_06055_amd as moe
from paper_2605_06055_amd import binding as B
from paper_2605_06055_amd.layer import MoeLayer
lib = moe.load_library()
assert B._native is not None
seen, answer = (ctypes.c_longlong * 64).in_dll(lib, "seen"), ctypes.c_int.in_dll(lib, "answer")
shape = moe.MoeShape(T=5, H=16, k=2, E=4, R=2, schedule=1, region_stride_rows=7)
x, ids, w = torch.zeros(5, 16), torch.zeros(5, 2, dtype=torch.int32), torch.zeros(5, 2)
window, y, scale = torch.zeros(10, 16), torch.zeros(5, 16), torch.zeros(10)
plan = moe.MoePlan(shape, device="cpu")
plan.prefetch = x
bare = moe.MoePlan(shape, device="cpu", with_send_idx=False, with_order=False)
class Sub(torch.Tensor): pass
slow = []
real = B._slow
B._slow = lambda *a: (slow.append(a[0]), real(*a))[1]
def call(name, *a):
    seen[50] = 0
    try:
        getattr(moe, name)(*a)
    except Exception as e:
        return type(e), str(e)
    assert seen[50] == 1
    return list(seen)
def both(name, *a):
    fast, native, n = call(name, *a), B._native, len(slow)
    B._native = None
    assert call(name, *a) == fast, (name, a)
    B._native = native
    return n                                                   # the slow path was taken by so many calls before
for p in (plan, plan.struct(), bare):
    for name, before, after in (("moe_plan", (ids,), ()), ("moe_plan_static", (ids,), ()), ("moe_dispatch", (x, ids), (window,)),
                                ("moe_dispatch_quant", (x, ids), (window, scale)), ("moe_combine", (window, w), (y,))):
        for code in (0, -3):
            answer.value = code
            n = len(slow)
            assert both(name, shape, *before, p, *after, 77) == n, (name, "natively")
            # None and addresses in each place
            for other in (None, 4096, -1):
                for i in range(len(before) + len(after)):
                    t = list(before + after)
                    t[i] = other
                    n = len(slow)
                    assert both(name, shape, *t[:len(before)], p, *t[len(before):], 77) == n
answer.value = 0
for bad in (x.t(), x.as_subclass(Sub), torch.nn.Parameter(x), np.zeros(3), 1.5, "x", x.to_sparse(), torch.empty(5, 16, device="meta"), True):
    both("moe_dispatch", shape, bad, ids, plan, window, 77)
    both("moe_combine", shape, window, w, plan, bad, 77)
for bad in (None, ctypes.byref(shape), 3, plan.struct()):
    both("moe_dispatch", bad, x, ids, plan, window, 77)
for bad in (None, ctypes.byref(plan.struct()), 3, shape):
    both("moe_dispatch", shape, x, ids, bad, window, 77)
plan.workspace = None
both("moe_plan", shape, ids, plan, 77)
class Stream: cuda_stream = 99
both("moe_plan", shape, ids, bare, Stream())
# bound calls: the structures are read at each call, the schedule's plan comes first, errors name the call
for schedule in (1, 2):
    layer = MoeLayer(5, 16, 2, 4, 2, dtype=moe.MOE_DTYPE_F32, schedule=schedule, device="cpu")
    dispatch, combine = layer.bind(x, ids, w, stream=55)
    dispatch()
    got = list(seen)
    layer.dispatch(x, ids, stream=55)
    assert got == list(seen)
    layer._plan_struct.send_idx = 4096
    combine()
    got = list(seen)
    layer.combine(w, stream=55)
    assert got == list(seen)
    answer.value = -4
    for f, where in ((dispatch, "moe_plan" if schedule == 1 else "moe_dispatch"), (combine, "moe_combine")):
        try:
            f()
            raise SystemExit("no error")
        except moe.MoeError as e:
            assert e.code == -4 and where in str(e)
    answer.value = 0
"""


def test_native_and_ctypes_marshalling_agree(tmp_path):
    src, so = tmp_path / "record.c", str(tmp_path / "librecord.so")
    src.write_text(RECORD)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-o", so, str(src)])
    res = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=dict(os.environ, MOE_RBF_LIB=so), capture_output=True, text=True,
                         timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-3000:]


def test_native_marshalling_has_no_thread_local_storage():
    """One would slow down every thread-local access of the libraries that are there already (see build_marshal)."""
    import struct
    import paper_2605_06055_amd as moe
    with open(os.path.join(os.path.dirname(moe.__file__), "_marshal.so"), "rb") as f:
        elf = f.read()
    offset, size, count = struct.unpack_from("<Q", elf, 32)[0], *struct.unpack_from("<HH", elf, 54)
    kinds = [struct.unpack_from("<I", elf, offset + i * size)[0] for i in range(count)]
    assert 1 in kinds and 7 not in kinds                       # PT_LOAD, PT_TLS
