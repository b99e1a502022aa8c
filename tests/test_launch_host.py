"""What the library asks of the HIP runtime when it launches, seen without a GPU: a stand-in for the four runtime calls of its
launch path is loaded in front of the real runtime, in a process of its own.  Nothing is executed; the stand-in refuses what
the runtime refuses (2^32 threads or more along one axis, more dynamic LDS than the kernel's limit on that device)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FAKE = r"""
#include <stddef.h>
#include <stdint.h>
typedef struct { uint32_t x, y, z; } dim3;
int fake_device, fake_refuse_raise, fake_launches, fake_raises;
uint64_t fake_most_threads, fake_most_lds;
static struct { const void *kernel; int device; size_t lds; } limit[256];
static int limits;
int hipGetDevice(int *d) { *d = fake_device; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipFuncSetAttribute(const void *kernel, int attr, int value) {
  (void)attr;
  if (fake_refuse_raise) return 1;
  limit[limits].kernel = kernel, limit[limits].device = fake_device, limit[limits].lds = (size_t)value;
  ++limits, ++fake_raises;
  return 0;
}
int hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  (void)args; (void)stream;
  size_t most = 64 * 1024;
  for (int i = 0; i < limits; ++i)
    if (limit[i].kernel == kernel && limit[i].device == fake_device && limit[i].lds > most) most = limit[i].lds;
  const uint64_t threads = (uint64_t)grid.x * block.x;
  if (threads > 0xffffffffull || (uint64_t)grid.y * block.y > 0xffffffffull || lds > most) return 9;
  if (threads > fake_most_threads) fake_most_threads = threads;
  if (lds > fake_most_lds) fake_most_lds = lds;
  ++fake_launches;
  return 0;
}
"""

PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
import paper_2605_06055_amd as moe
from paper_2605_06055_amd.binding import _PlanStruct
moe.load_library()
word = lambda name, kind=ctypes.c_int: kind.in_dll(fake, name)
most_lds = lambda: word("fake_most_lds", ctypes.c_uint64).value
X, K, W, WINDOW = 1 << 40, 1 << 36, 1 << 37, 1 << 44        # never dereferenced
PLAN = _PlanStruct(expert_count=0x1000, rank_count=0x2000, expert_offset=0x3000, region_base=0x4000, send_idx=0x5000,
                   row_map=0x6000, status=0x7000, workspace=0x8000, workspace_bytes=1 << 40)
def shape(**kw):
    return moe.MoeShape(**{{**dict(E=64, R=8, dtype=moe.MOE_DTYPE_BF16, schedule=moe.MOE_SCHEDULE_PREFILL), **kw}})
def refused(f, *a):
    try:
        f(*a)
    except moe.MoeError as e:
        return e.code
    return 0
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("fake_hip")
    src, so = folder / "fake_hip.c", str(folder / "libfake_hip.so")
    src.write_text(FAKE)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, str(src)])

    def child(body):
        res = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + body], capture_output=True,
                             text=True, timeout=300)
        assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-3000:]
    return child


def test_lds_limit_is_raised_on_every_device(run):
    """Combine's held results (46 a thread: 80 KB) and the plan's tables (1024 experts) need more than 64 KB of LDS: on each
    device the first such launch raises the limit, later ones do not, and a failure is not remembered."""
    run("""
big = shape(T=6700, H=7168, k=8)
wide = shape(T=4000, H=64, k=8, E=1024)
for device in (3, 0, 70):
    word("fake_device").value = device
    for s in (0, 1):
        word("fake_refuse_raise").value = 1
        fails = 0 if s and device < 64 else -6
        assert refused(moe.moe_combine, big, X, W, PLAN, WINDOW, s) == fails, device
        assert refused(moe.moe_plan, wide, K, PLAN, s) == fails, device
        word("fake_refuse_raise").value = 0
        raises = word("fake_raises").value
        assert refused(moe.moe_combine, big, X, W, PLAN, WINDOW, s) == 0, device
        assert refused(moe.moe_plan, wide, K, PLAN, s) == 0, device
        assert (word("fake_raises").value == raises) == (fails == 0)
assert most_lds() > 64 * 1024
""")


def test_dispatch_launches_stay_below_the_thread_limit(run):
    """Batches whose prefill dispatch has 2^32 threads or more as one launch are split; none is refused."""
    run("""
for H16, k, T in ((1, 8, 1 << 24), (1, 7, 38347922), (9, 8, 1 << 24), (64, 8, 1 << 23), (64, 5, 1 << 23), (80, 2, 1 << 25),
                  (120, 8, 1 << 24), (128, 3, 1 << 23), (456, 512, 36000), (512, 8, 1 << 22), (513, 8, 1 << 21),
                  (897, 8, 600000), (896, 1, 9000000), (896, 4000, 8000), (4095, 8, 200000), (4096, 4000, 2000),
                  (4096, 1, 2100000)):
    for order in (None, 1 << 45):
        PLAN.dispatch_order = order
        for shift in (0, 16):                                  # windows that start at a line and inside one
            s = shape(T=T, H=H16 * 8, k=k)
            assert refused(moe.moe_dispatch, s, X, None, PLAN, WINDOW + shift, 0) == 0, (H16, k, T, order, shift)
assert word("fake_launches").value > 17 * 4                   # some were split
""")
