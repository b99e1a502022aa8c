"""Prefill dispatch where its column slices, cut at cache lines of the destination, can go wrong: rows of one vector, of
fewer lines than slices, one vector short of and past a line and a slice, slices that differ by a line, slices longer than
a workgroup, windows that do not start at a line; along the order list and in token order."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def moe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_06055_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("H16", [1, 7, 8, 9, 63, 64, 65, 72, 96, 97, 128, 136, 257, 320, 321, 513, 576, 776, 832, 840, 896, 960, 1000, 4096,
                                 4104, 5001])
@pytest.mark.parametrize("shift", [0, 1, 7])                   # 16-byte vectors from a line to the window's first row
def test_dispatch_writes_every_vector_once(moe, H16, shift):
    from paper_2605_06055_amd.layer import to_device, to_host
    rng = np.random.default_rng(H16 * 8 + shift)
    H, k, E, R = H16 * 8, (8, 6, 5)[shift % 3], 48, 4
    T = max(40, min(4000, (6 << 20) // (H * 2)))               # X just past the size from which the list is used
    listed = H16 >= 96 and (H16 >= 128 or k >= 8)
    N = T * k
    K = wl.random_routing(rng, T, k, E, p_masked=0.04, p_invalid=0.01)
    X = rng.integers(0, 1 << 16, size=(T, H), dtype=np.uint16)                     # any bits: dispatch copies
    ref = oracle.plan(K, E, R)
    want = oracle.dispatch(X, ref.row_map, ref.window_rows, fill=np.uint16(0x7B7B))
    xd, kd = to_device(X), to_device(K)
    for with_order in (True, False):
        print(f"[slices] H16={H16} T={T} k={k} shift={shift} list={with_order}", flush=True)
        shape = moe.MoeShape(T=T, H=H, k=k, E=E, R=R, dtype=moe.MOE_DTYPE_BF16, schedule=moe.MOE_SCHEDULE_PREFILL)
        plan = moe.MoePlan(shape, with_order=with_order)
        buf = torch.full(((N + 2) * H + 128,), 0x7B7B, dtype=torch.int16, device="cuda")
        assert buf.data_ptr() % 128 == 0
        window = buf[shift * 8:shift * 8 + N * H].view(N, H)
        if with_order:
            plan.dispatch_order.fill_(-77)
        moe.moe_plan(shape, kd, plan)
        moe.moe_dispatch(shape, xd, kd, plan, window)
        torch.cuda.synchronize()
        if with_order:
            assert bool((plan.dispatch_order[:2 * N] == -77).any()) != listed
        got = to_host(buf).view(np.uint16)
        rows = got[shift * 8:shift * 8 + N * H].reshape(N, H)
        assert np.array_equal(rows[:ref.window_rows], want)
        # nothing else is written: in front of the window, in its unused rows, behind it
        assert np.all(got[:shift * 8] == 0x7B7B) and np.all(rows[ref.window_rows:] == 0x7B7B)
        assert np.all(got[shift * 8 + N * H:] == 0x7B7B)


@pytest.mark.parametrize("T,H,k,stride", [(4200, 16392, 3, 0),       # ragged rows, slices longer than a wave
                                          (9001, 4872, 3, 0),        # stretches that begin and end inside a token
                                          (9000, 4864, 5, 7000),     # unequal slices, dropped branches, ragged last stretch
                                          (29000, 1600, 3, 0),       # two branches per unit, rows of 25 lines
                                          (28500, 1544, 4, 14500),   # two branches per unit, ragged rows, dropped branches
                                          (29000, 1536, 2, 0),       # degree 2, equal slices
                                          (14001, 3072, 5, 0),       # three pieces of 256 bytes: one block
                                          (8501, 5120, 3, 0),        # five pieces of 256 bytes
                                          (7002, 6144, 3, 3340),     # three of 512, dropped branches
                                          (1300, 49152, 10, 0)])     # three of 4 KB, slices longer than a workgroup
def test_dispatch_with_bulk_reads_of_x(moe, T, H, k, stride):
    """X of more than 80 MiB: the list's stretches are read in bulk ahead of their copies."""
    assert T * H * 2 > 80 << 20
    dispatch_large(moe, T, H, k, stride, True)


@pytest.mark.parametrize("H16", [384, 640, 768, 1152, 1536, 1792, 3072, 6144, 7168])
@pytest.mark.parametrize("shift", [0, 8])                      # a window that starts at another line
def test_slices_in_pieces(moe, H16, shift):
    """Equal slices that are no power of two are written in pieces of 256 bytes to 4 KB (that they are: test_routes_host.py);
    H16 >= 6144: longer than a workgroup."""
    test_dispatch_writes_every_vector_once(moe, H16, shift)


@pytest.mark.parametrize("T,H,k,stride,given,used", [(2700, 16392, 3, 0, True, True),      # a single-launch plan: one stretch, no bulk reads
                                                     (33000, 4096, 8, 0, False, False)])   # no list, X beyond the caches: 8 branches per unit
def test_dispatch_of_large_x_without_bulk_reads(moe, T, H, k, stride, given, used):
    dispatch_large(moe, T, H, k, stride, used, given)


def dispatch_large(moe, T, H, k, stride, used, given=True):
    from paper_2605_06055_amd.layer import MoeLayer, to_device, to_host
    rng = np.random.default_rng(T)
    E, R = 48, 6
    K = wl.random_routing(rng, T, k, E, p_masked=0.03, p_invalid=0.01)
    ref = oracle.plan(K, E, R, stride)
    print(f"[large X] T={T} H={H} k={k} stride={stride} list={used}", flush=True)
    layer = MoeLayer(T, H, k, E, R, region_stride_rows=stride, schedule=moe.MOE_SCHEDULE_PREFILL)
    layer.plan.dispatch_order.fill_(-77)
    if not given:
        layer._plan_struct.dispatch_order = None
    x = torch.randint(-(1 << 15), 1 << 15, (T, H), dtype=torch.int16, device="cuda")
    bits = layer.window.view(torch.int16)
    bits.fill_(0x7B7B)
    layer.dispatch(x.view(torch.bfloat16), to_device(K))
    torch.cuda.synchronize()
    assert bool((layer.plan.dispatch_order[:2 * T * k] == -77).any()) != used
    assert np.array_equal(to_host(layer.plan.row_map)[:T * k].reshape(T, k), ref.row_map)
    assert stride == 0 or ref.status[1] > 0
    rows = torch.from_numpy(ref.row_map.reshape(-1).astype(np.int64)).cuda()
    at = torch.full((bits.shape[0],), -1, dtype=torch.int64, device="cuda")
    at[rows[rows >= 0]] = (torch.arange(T * k, device="cuda") // k)[rows >= 0]
    assert torch.equal(bits[at >= 0], x[at[at >= 0]])
    assert bool((bits[at < 0] == 0x7B7B).all())


@pytest.mark.parametrize("H16", [1 << 27, (1 << 27) + 1])      # 2^24 lines, and one vector more (rows that start inside a line)
@pytest.mark.parametrize("with_order", [True, False])
def test_rows_of_2_gib(moe, H16, with_order):
    """Slice cuts of rows of 2^24 lines and more: the product of slice and lines needs more than 24 bits."""
    from paper_2605_06055_amd.layer import to_device, to_host
    H, k = H16 * 8, 3
    print(f"[2 GiB rows] H16={H16} list={with_order}", flush=True)
    shape = moe.MoeShape(T=1, H=H, k=k, E=k, R=1, dtype=moe.MOE_DTYPE_BF16, schedule=moe.MOE_SCHEDULE_PREFILL)
    plan = moe.MoePlan(shape, with_order=with_order)
    kd = to_device(np.array([[2, 0, 1]], dtype=np.int32))
    x = torch.arange(H // 2, dtype=torch.int32, device="cuda")                      # every vector is different
    window = torch.full((k, H // 2), -7, dtype=torch.int32, device="cuda")
    moe.moe_plan(shape, kd, plan)
    moe.moe_dispatch(shape, x, kd, plan, window)
    torch.cuda.synchronize()
    assert to_host(plan.row_map)[:k].tolist() == [2, 0, 1]
    for row in range(k):
        assert torch.equal(window[row], x), row


@pytest.mark.parametrize("shift", [0, 1])
def test_more_threads_than_one_launch_may_have(moe, shift):
    """Rows of one vector, 2^27 + 8 branches: 2^32 threads and more, so the copy is split over two launches."""
    from paper_2605_06055_amd.layer import to_device
    T, k, H = (1 << 24) + 1, 8, 8
    N = T * k
    print(f"[split] N={N} shift={shift}", flush=True)
    shape = moe.MoeShape(T=T, H=H, k=k, E=8, R=1, dtype=moe.MOE_DTYPE_BF16, schedule=moe.MOE_SCHEDULE_PREFILL)
    plan = moe.MoePlan(shape)
    rows = torch.arange(N, dtype=torch.int64, device="cuda") * 1000003 % N         # 1000003 does not divide N: a permutation
    plan.row_map.copy_(rows)
    x = torch.arange(T * 2, dtype=torch.int64, device="cuda").view(T, 2)
    buf = torch.full(((N + 2) * 2,), -7, dtype=torch.int64, device="cuda")
    window = buf[shift * 2:shift * 2 + N * 2].view(N, 2)
    moe.moe_dispatch(shape, x, None, plan, window)
    torch.cuda.synchronize()
    for j in range(k):
        assert torch.equal(window[rows.view(T, k)[:, j]], x), j
    assert bool((buf[:shift * 2] == -7).all()) and bool((buf[shift * 2 + N * 2:] == -7).all())


@pytest.mark.parametrize("T,H,k,dtype,used", [(3200, 8192, 3, "f32", False),   # 100 MiB of X in the one stretch of a single-launch plan
                                              (4800, 8192, 3, "f32", True),    # 150 MiB in stretches: read in bulk
                                              (11702, 896, 6, "bf16", False), (11702, 896, 8, "bf16", True),
                                              (12288, 2560, 4, "bf16", False), (12288, 2560, 2, "bf16", True),
                                              (17408, 2560, 4, "bf16", True), (8777, 3200, 2, "bf16", False),
                                              (8777, 3200, 4, "bf16", False), (8777, 3200, 3, "bf16", True),
                                              (13897, 3584, 4, "bf16", False), (13897, 3584, 6, "bf16", True)])
def test_which_plans_carry_the_order_list(moe, T, H, k, dtype, used):
    from paper_2605_06055_amd.layer import to_device
    rng = np.random.default_rng(T)
    shape = moe.MoeShape(T=T, H=H, k=k, E=64, R=8, dtype=moe.MOE_DTYPE_F32 if dtype == "f32" else moe.MOE_DTYPE_BF16,
                         schedule=moe.MOE_SCHEDULE_PREFILL)
    plan = moe.MoePlan(shape)
    plan.dispatch_order.fill_(-77)
    moe.moe_plan(shape, to_device(wl.random_routing(rng, T, k, 64)), plan)
    torch.cuda.synchronize()
    written = plan.dispatch_order[:2 * T * k] != -77
    assert bool(written.all()) if used else not bool(written.any())
