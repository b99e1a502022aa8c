"""The calls that MoeLayer binds, for every form of argument.  A stand-in library that only records its arguments takes the place of the HIP
one."""
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
