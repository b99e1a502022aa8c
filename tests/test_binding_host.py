"""The binding where its native half is missing or was built for another torch, and the calls that MoeLayer binds, for every form of
argument and for as long as a caller holds them.  A stand-in library that only records its arguments takes the place of the HIP one."""
import os
import subprocess
import sys

import pytest

from test_marshal_host import RECORD, ROOT

PRELUDE = r"""
import ctypes, gc, sys, weakref
sys.path.insert(0, sys.argv[1])
import torch
import paper_2605_06055_amd as moe
from paper_2605_06055_amd import binding as B
from paper_2605_06055_amd.layer import MoeLayer
def library():
    lib = moe.load_library()
    return lib, (ctypes.c_longlong * 64).in_dll(lib, "seen"), ctypes.c_int.in_dll(lib, "answer")
x, ids, w = torch.zeros(5, 16), torch.zeros(5, 2, dtype=torch.int32), torch.zeros(5, 2)
def layer(schedule=1, **more):
    return MoeLayer(5, 16, 2, 4, 2, dtype=moe.MOE_DTYPE_F32, schedule=schedule, device="cpu", **more)
def all_alive(refs):
    return all(r() is not None for r in refs)
def every_call(expected_native):
    lib, seen, answer = library()
    assert (B._native is not None) == expected_native
    for schedule in (1, 2):
        l = layer(schedule)
        l.dispatch(x, ids, stream=55)
        assert seen[42] == x.data_ptr() and seen[44] == l.window.data_ptr() and seen[46] == 55
        l.combine(w, stream=55)
        assert seen[42] == l.expert_out.data_ptr() and seen[44] == l.y.data_ptr()
        moe.moe_plan(l.shape, ids, l.plan, 55)
        assert seen[42] == ids.data_ptr() and seen[46] == 55
        bound(seen, answer, l, schedule, *l.bind(x, ids, w, stream=55))
def bound(seen, answer, l, schedule, dispatch, combine, stream=55):
    seen[50] = 0
    dispatch()
    assert seen[50] == 1 and seen[42] == x.data_ptr() and seen[44] == l.window.data_ptr() and seen[46] == stream
    combine()
    assert seen[42] == l.expert_out.data_ptr() and seen[43] == w.data_ptr() and seen[44] == l.y.data_ptr() and seen[46] == stream
    answer.value = -4
    for f, where in ((dispatch, "moe_plan" if schedule == 1 else "moe_dispatch"), (combine, "moe_combine")):
        try:
            f()
            raise SystemExit("no error")
        except moe.MoeError as e:
            assert e.code == -4 and where in str(e)
    answer.value = 0
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("record")
    src, so = folder / "record.c", str(folder / "librecord.so")
    src.write_text(RECORD)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-o", so, str(src)])

    def child(body):
        res = subprocess.run([sys.executable, "-c", PRELUDE + body, ROOT], env=dict(os.environ, MOE_RBF_LIB=so), capture_output=True,
                             text=True, timeout=300)
        assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-3000:]
    return child


def test_bind_takes_what_ctypes_takes(run):
    """Forms that the native half does not read: integers of a subclass, structures of a subclass."""
    run("""
lib, seen, answer = library()
class Handle(int): pass
class Shape(moe.MoeShape): pass
for schedule in (1, 2):
    l = layer(schedule)
    bound(seen, answer, l, schedule, *l.bind(x, ids, w, stream=Handle(66)), stream=66)
    bound(seen, answer, l, schedule, *l.bind(x, ids, w, stream=True), stream=1)
    l.shape = Shape(*(getattr(l.shape, f) for f, _ in l.shape._fields_))
    bound(seen, answer, l, schedule, *l.bind(x, ids, w, stream=55))
    assert list(seen)[40:42] == [1, 1]
""")


def test_without_the_native_half(run):
    """The library alone is enough: every call then goes by way of ctypes."""
    run("sys.modules['paper_2605_06055_amd._marshal'] = None\nevery_call(False)\n")


def test_native_half_of_another_torch(run):
    """It reads torch's objects by their layout, so one built for another version is left aside."""
    run("torch.__version__ = '1.2.3'\nevery_call(False)\n")


def test_native_half_of_this_torch(run):
    run("every_call(True)\n")


@pytest.mark.parametrize("native", [True, False])
def test_bound_calls_keep_their_buffers(run, native):
    """Each of the two calls alone keeps everything that the launches read and write, whatever the caller drops and however often the
    layer is bound again; nothing is kept once they are gone."""
    run(("" if native else "sys.modules['paper_2605_06055_amd._marshal'] = None\n") + """
lib, seen, answer = library()
for which in (0, 1):
    refs, at, held = [], [], []
    l = layer(source_count=torch.zeros(2, 4, dtype=torch.int32), window_rows=10)
    for n in range(2):
        mine = torch.full((5, 16), float(n)), torch.zeros(5, 2, dtype=torch.int32), torch.ones(5, 2)
        held.append(l.bind(*mine, stream=55)[which])
        all = [*mine, l.window, l.expert_out, l.y, *(t for t in vars(l.plan).values() if t is not None)]
        refs.append([weakref.ref(t) for t in all])
        at.append(mine[0].data_ptr() if which == 0 else mine[2].data_ptr())
        del mine, all
    del l
    gc.collect()
    for n in range(2):
        assert all_alive(refs[n])
        held[n]()
        assert seen[42 if which == 0 else 43] == at[n]
    held.clear()
    gc.collect()
    assert not any(r() is not None for r in refs[0] + refs[1])
""")


def test_prefetch_is_named_for_one_call_only(run):
    """The address of x goes to the plan call and does not stay behind for later calls, whose x may be another."""
    run("""
lib, seen, answer = library()
at_plan = []
l = layer()
real = B.moe_plan
B.moe_plan = lambda *a: (real(*a), at_plan.append((seen[8 + 13], seen[8 + 14])))[0]
l.prefetch_x = True
for code in (0, -3):
    answer.value = code
    try:
        l.dispatch(x, ids, stream=55)
    except moe.MoeError as e:
        at_plan.append((seen[8 + 13], seen[8 + 14]))
    answer.value = 0
    assert at_plan.pop() == (x.data_ptr(), 5 * 16 * 4) and not at_plan
    assert l._plan_struct.prefetch is None and l._plan_struct.prefetch_bytes == 0
l.prefetch_x = False
l.dispatch(x, ids, stream=55)
assert at_plan.pop() == (0, 0)
""")
