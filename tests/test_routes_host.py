"""Which kernel a call takes where both of two forms would be right and only one is fast, seen without a GPU: a stand-in for the
runtime's launch call notes the kernel's name and the workgroup, and how the prefill dispatch cuts its slices.  The rules and their measurements stand beside the code."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FAKE = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
int fake_launches, fake_block, fake_cut[3];
char fake_names[4096];
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipFuncSetAttribute(const void *kernel, int attr, int value) { (void)kernel; (void)attr; (void)value; return 0; }
int hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  (void)grid; (void)lds; (void)stream;
  Dl_info at;
  const char *name = dladdr(kernel, &at) && at.dli_sname ? at.dli_sname : "?";
  if (strlen(fake_names) + strlen(name) + 2 < sizeof(fake_names)) strcat(strcat(fake_names, name), " ");
  if (strstr(name, "dispatch_units_kernel")) {       /* its last arguments: warm_blocks, stretch, piece, shift */
    fake_cut[0] = *(const int *)args[11] > 0;
    fake_cut[1] = *(const int *)args[13];
    fake_cut[2] = *(const int *)args[14];
  }
  fake_block = (int)block.x;
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
X, K, W, WINDOW = 1 << 40, 1 << 36, 1 << 37, 1 << 44        # never dereferenced
PLAN = _PlanStruct(expert_count=0x1000, rank_count=0x2000, expert_offset=0x3000, region_base=0x4000, send_idx=0x5000,
                   row_map=0x6000, status=0x7000, workspace=0x8000, workspace_bytes=1 << 40)
names = (ctypes.c_char * 4096).in_dll(fake, "fake_names")
def shape(**kw):
    return moe.MoeShape(**{{**dict(E=64, R=1, dtype=moe.MOE_DTYPE_BF16, schedule=moe.MOE_SCHEDULE_PREFILL), **kw}})
def launched(call, *a):
    ctypes.memset(names, 0, 4096)
    call(*a, 0)
    return names.value.decode().split(), ctypes.c_int.in_dll(fake, "fake_block").value
def combine(H16, k, T=60000):
    return launched(moe.moe_combine, shape(T=T, H=8 * H16, k=k), X, W, PLAN, WINDOW)[0][0]
def plan(N, k, E):
    return len(launched(moe.moe_plan, shape(T=N // k, H=8, k=k, E=E), K, PLAN)[0])
def decode(N, k, E=64, H16=512, quant=False):
    s = shape(T=N // k, H=8 * H16, k=k, E=E, schedule=moe.MOE_SCHEDULE_DECODE)
    n, block = launched(moe.moe_dispatch_quant, s, X, K, PLAN, WINDOW, W) if quant else launched(moe.moe_dispatch, s, X, K, PLAN, WINDOW)
    assert len(n) == 1
    return ("histogram" if "decode_hist" in n[0] else "ballots"), block
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("fake_hip")
    src, so = folder / "fake_hip.c", str(folder / "libfake_hip.so")
    src.write_text(FAKE)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, str(src), "-ldl"])

    def child(body):
        res = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + body], capture_output=True,
                             text=True, timeout=300)
        assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-3000:]
    return child


def test_combine_of_padded_rows(run):
    """Degrees of 10 and 5 do not hold results back where too many of the padded columns are idle."""
    run("""
held = lambda *a: "combine_deferred" in combine(*a)
for H16 in (65, 66, 72, 80, 88, 92, 95):
    assert not held(H16, 10) and not held(H16, 5), H16
for H16 in (96, 112, 128, 144, 160, 513, 896):
    assert held(H16, 10), H16
for H16 in (48, 52, 56, 129, 160):
    assert not held(H16, 5), H16
for H16 in (60, 64, 112, 128, 224, 449, 640, 641, 896):
    assert held(H16, 5), H16
""")


BLOCK = """
def block(H16, k, T, shift=0):
    n, b = launched(moe.moe_combine, shape(T=T, H=8 * H16, k=k), X + 16 * shift, W, PLAN, WINDOW)
    return n[0].split("combine_")[1].split("_kernel")[0], b
"""


def test_combine_workgroups(run):
    """Whole rows, or equal parts of 3 to 10 waves, where rows are no multiple of a line or leave columns idle; one wave in the smallest
    launches.  Degrees of 8 and 6 hold their results back unless too many columns are idle."""
    run(BLOCK + """
for H16, waves in ((65, 2), (129, 3), (193, 4), (72, 2), (96, 2)):                  # up to 4 waves, whole lines up to 2
    T = -(-100000 // H16)
    assert block(H16, 8, T) == ("rows", 64 * waves), H16
    assert block(H16, 8, T - 1) == ("rows", 64), H16
# wider rows: 2.4 M vectors of window and 2.5 workgroups a compute unit
for H16, waves, k in ((257, 5, 8), (333, 6, 4), (513, 9, 6), (641, 6, 2), (705, 6, 10), (801, 7, 8), (897, 5, 6), (1089, 9, 8), (1350, 8, 4), (1857, 10, 8)):
    groups = -(-H16 // (64 * waves))
    def even(T):                                                                    # 1.7 M, 1.75 a unit and the units 85 % full
        n = T * groups
        return k > 2 and T * k * H16 >= 1700000 and n >= 448 and n / (-(-n // 256) * 256) >= 0.85
    T = max(-(-2400000 // (k * H16)), -(-640 // groups))
    assert block(H16, k, T) == ("rows", 64 * waves), H16
    for t in (T - 1, T * 9 // 10, T * 8 // 10, T * 3 // 4, T * 2 // 3):
        assert block(H16, k, t) == ("rows", 64 * waves if even(t) else 64), (H16, t)
for H16, k, T, row in ((625, 10, 640, 1), (625, 10, 639, 0), (625, 10, 512, 1), (625, 10, 513, 0), (625, 10, 448, 1), (625, 10, 447, 0), (333, 8, 700, 1),
                       (333, 8, 652, 0), (333, 8, 638, 0), (257, 8, 827, 0), (257, 8, 871, 1), (257, 2, 3307, 0), (513, 2, 2300, 0)):
    assert block(H16, k, T) == ("rows", (64 * -(-H16 // 64) if row else 64)), (H16, k, T)
for H16, k, T, waves in ((513, 1, 195, 9), (513, 1, 5000, 9), (513, 2, 584, 9), (264, 2, 1136, 5), (264, 1, 2272, 5), (144, 1, 4166, 3), (208, 1, 7000, 4),
                         (208, 4, 2885, 4), (208, 8, 1443, 4)):                     # little work; 4 waves of whole lines
    assert block(H16, k, T) == ("rows", 64 * waves), (H16, k, T)
for H16, k, T in ((513, 8, 262), (513, 2, 585), (1350, 8, 96), (264, 2, 1137), (264, 1, 2273), (264, 8, 5000), (144, 8, 5000), (144, 1, 4167), (208, 8, 1050)):
    assert block(H16, k, T) == ("rows", 64), (H16, k, T)
assert block(112, 8, 2000) == ("rows", 64) and block(512, 8, 2000) == ("rows", 64) and block(512, 8, 2000, 1) == ("rows", 512)
assert block(512, 4, 60000) == ("rows", 128) and block(513, 4, 60000) == ("rows", 576) and block(272, 4, 60000) == ("rows", 128)
for H16 in (65, 72, 80):
    assert block(H16, 8, 60000) == ("rows", 128)
for H16 in (81, 96, 129, 513):
    assert block(H16, 8, 60000)[0] == "deferred", H16
for H16 in (40, 48, 72, 100, 144, 152, 200, 257, 513):
    assert block(H16, 6, 60000)[0] == "rows", H16
for H16 in (50, 54, 57, 64, 104, 112, 160, 208, 272, 288, 512, 525, 625, 896):         # a fifth idle, of one wave a quarter, ragged a tenth
    assert block(H16, 6, 60000)[0] == "deferred", H16
""")


def test_combine_of_more_threads_than_a_launch_takes(run):
    """Rows of 22 waves as 3 times 8: beyond 2^32 threads they take workgroups of two waves, which leave none idle."""
    run(BLOCK + """
assert block(1350, 1, (1 << 32) // 1536) == ("rows", 512)
assert block(1350, 1, (1 << 32) // 1536 + 1) == ("rows", 128)
""")


def test_dispatch_pieces(run):
    """Equal slices are written in pieces of the largest power of two that divides them, from 256 bytes on; with bulk reads narrow rows only from
    512; not by units that are alone in a workgroup, and never where the slices differ."""
    run("""
LISTED = _PlanStruct.from_buffer_copy(PLAN)
LISTED.dispatch_order = 0x9000
cut = (ctypes.c_int * 3).in_dll(fake, "fake_cut")
def pieces(H16, mib, k=8, shift=0):
    T = (mib << 20) // (16 * H16)
    n, _ = launched(moe.moe_dispatch, shape(T=T, H=8 * H16, k=k), X, K, LISTED, WINDOW + 16 * shift)
    assert "dispatch_units" in n[0], (H16, mib)
    return tuple(cut)
BLOCK = 31                     # the whole slice as one piece
for H16, piece, bulk in ((256, 32, 32), (384, 16, 0), (448, 0, 0), (512, 64, 64), (640, 16, 16), (768, 32, 32), (832, 0, 0), (896, 0, 16), (960, 0, 0),
                         (1152, 16, 16), (1536, 64, 64), (1792, 32, 32), (2048, 256, 256)):
    for mib, warm, want in ((50, 0, piece), (120, 1, bulk)):
        assert pieces(H16, mib) == (warm, want or H16 // 8, want.bit_length() - 1 if want else BLOCK), (H16, mib)
for H16 in (513, 520, 1000, 2000):
    assert pieces(H16, 50)[2] == pieces(H16, 120)[2] == BLOCK, H16
assert pieces(1536, 50, shift=1)[2] == BLOCK
""")


def test_plan_of_few_experts(run):
    """A single launch counts all ids in every workgroup: not beyond 2048 branches an expert."""
    run("""
for k in (4, 8):
    for N, E, launches in ((12288, 1, 1), (12296, 1, 2), (12296, 4, 2), (16384, 8, 1), (16392, 8, 2), (24576, 8, 2), (24576, 12, 1),
                           (24584, 12, 2), (28672, 14, 1), (28672, 256, 1), (28680, 256, 2)):
        assert plan(N, k, E) == launches, (N, k, E)
""")


def test_decode_kernel(run):
    """Compares and ballots up to a number of branches, the histogram beyond; one line of a rule each."""
    run("""
for k, E, H16, quant, last in ((8, 256, 512, 0, 1408), (8, 512, 512, 0, 1408), (8, 256, 640, 0, 1536), (8, 256, 896, 0, 1536), (7, 512, 896, 0, 2044),
                               (8, 512, 896, 0, 2048), (8, 1024, 896, 0, 3072), (8, 256, 1280, 0, 1408), (8, 256, 1792, 0, 1536),
                               (6, 256, 832, 0, 1536), (6, 256, 896, 0, 3582), (6, 64, 1792, 0, 3582), (6, 256, 1280, 0, 1404),
                               (10, 64, 896, 0, 1400), (16, 64, 896, 0, 1536), (16, 64, 256, 0, 1408),
                               (5, 256, 256, 0, 1150), (5, 512, 256, 0, 1405), (5, 256, 264, 0, 600), (5, 512, 896, 0, 600), (5, 1024, 896, 0, 1365),
                               (4, 512, 512, 0, 600), (4, 1024, 512, 0, 1368), (4, 1024, 1032, 0, 600), (2, 1024, 512, 0, 600), (1, 256, 512, 0, 600),
                               (8, 256, 256, 1, 1280), (6, 256, 256, 1, 1152), (8, 256, 512, 1, 1024), (8, 1024, 512, 1, 1280), (8, 1024, 1032, 1, 1024),
                               (10, 64, 256, 1, 1020), (5, 256, 256, 1, 600), (5, 512, 256, 1, 855), (5, 256, 264, 1, 0), (5, 512, 264, 1, 255),
                               (4, 256, 256, 1, 0), (4, 512, 256, 1, 256), (2, 512, 1032, 1, 0)):
    for N in ([last] if last else []) + [k]:
        if N <= last:
            assert decode(N, k, E, H16, quant)[0] == "ballots", (k, E, H16, quant, N)
    assert decode(last + k, k, E, H16, quant)[0] == "histogram", (k, E, H16, quant, last)
""")
