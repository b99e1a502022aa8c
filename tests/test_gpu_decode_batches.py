"""The fused decode dispatch at the batches where its form changes: sets of tokens that end inside the batch, degrees beyond one
round of slots, rows of one vector, of several chunks and of more vectors than a workgroup has lanes, one expert and the most,
dropped branches, the largest batch; plain and quantised rows, from one source rank and several, against the oracle."""
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


CASES = [  # T, H, k, E, R, stride
    (1, 8, 1, 1, 1, 0), (601, 8, 1, 5, 5, 0), (3077, 1032, 1, 64, 2, 0), (8192, 64, 1, 1024, 8, 0), (5001, 4104, 1, 16, 2, 0),
    (401, 520, 2, 32, 4, 0), (1539, 8200, 2, 96, 12, 300), (4096, 256, 2, 257, 1, 0),
    (333, 4096, 3, 16, 1, 0), (769, 2056, 3, 48, 4, 0), (1025, 3384, 4, 64, 8, 480), (130, 10248, 5, 24, 4, 0), (1638, 136, 5, 40, 2, 0),
    (235, 7168, 6, 128, 32, 0), (640, 2784, 8, 256, 32, 0), (512, 7168, 8, 256, 32, 130), (289, 4104, 8, 256, 1, 0),
    (150, 2048, 10, 64, 8, 0), (100, 264, 17, 12, 3, 0), (45, 1024, 40, 16, 2, 0), (7, 72, 1001, 30, 5, 0), (1024, 128, 8, 2, 1, 0),
    # several chunks and half a token's slots each; 4 vectors a lane and two quantised rows; scans of several pieces a wave
    (300, 14336, 8, 256, 32, 0), (184, 9216, 8, 64, 4, 120), (769, 16392, 3, 48, 4, 0), (700, 2048, 2, 1024, 8, 0), (41, 2048, 6, 1000, 8, 0),
    (100, 1032, 16, 513, 3, 0),
]


@pytest.mark.parametrize("T,H,k,E,R,stride", CASES)
@pytest.mark.parametrize("quant", [False, True])
def test_decode_dispatch(moe, T, H, k, E, R, stride, quant):
    from paper_2605_06055_amd.layer import MoeLayer, to_device, to_host
    rng = np.random.default_rng(T * 31 + H + k)
    K = wl.random_routing(rng, T, k, E, p_masked=0.05, p_invalid=0.02)
    X = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    ref = oracle.plan(K, E, R, stride)
    print(f"[decode] T={T} H={H} k={k} E={E} R={R} stride={stride} quant={quant}", flush=True)
    layer = MoeLayer(T, H, k, E, R, schedule=moe.MOE_SCHEDULE_DECODE, region_stride_rows=stride)
    p = layer.plan
    for t in (p.expert_count, p.rank_count, p.expert_offset, p.region_base, p.send_idx, p.row_map, p.status):
        t.fill_(-7)
    xd, kd, rows = to_device(X), to_device(K), max(layer.rows, 1)
    if quant:
        codes = torch.full((rows, H), 0xAA, dtype=torch.uint8, device="cuda")
        scales = torch.full((rows,), -1.0, device="cuda")
        moe.moe_dispatch_quant(layer.shape, xd, kd, p, codes, scales)
        want = oracle.dispatch_quant(X, ref.row_map, rows, fill=0xAA)
        assert codes.cpu().numpy().tobytes() == want[0].tobytes() and scales.cpu().numpy().tobytes() == want[1].tobytes()
    else:
        layer.window.view(torch.int16).fill_(0x7B7B)
        layer.dispatch(xd, kd)
        assert to_host(layer.window).tobytes() == oracle.dispatch(X, ref.row_map, rows, fill=np.uint16(0x7B7B)).tobytes()
    N = T * k
    assert np.array_equal(to_host(p.row_map)[:N].reshape(T, k), ref.row_map)
    assert np.array_equal(to_host(p.send_idx)[:N].reshape(T, k), ref.s)
    for got, exp in ((p.expert_count, ref.c_exp), (p.rank_count, ref.c_rank), (p.expert_offset, ref.expert_offset),
                     (p.region_base, ref.region_base), (p.status[:3], ref.status)):
        assert np.array_equal(to_host(got), exp)


@pytest.mark.parametrize("T,k,E,R,me", [(3, 8, 256, 32, 0), (3, 8, 256, 32, 31), (130, 8, 256, 32, 16), (200, 8, 512, 256, 100),
                                        (150, 4, 6, 3, 1), (40, 2, 1024, 2, 1), (64, 6, 12, 12, 5), (64, 6, 1024, 1024, 1023),
                                        (601, 1, 4, 1, 0), (700, 3, 20, 5, 2), (100, 17, 36, 9, 8)])
@pytest.mark.parametrize("most", [50, 40000])                 # elements of the count matrix (40000: its total is taken in 64 bits)
@pytest.mark.parametrize("schedule", ["decode", "prefill"])
def test_several_sources(moe, T, k, E, R, me, most, schedule):
    from paper_2605_06055_amd.layer import MoeLayer, to_device, to_host
    rng = np.random.default_rng(T + E + R + me)
    K = wl.random_routing(rng, T, k, E, p_masked=0.05, p_invalid=0.02)
    M = rng.integers(0, most, size=(R, E)).astype(np.int32)
    if most > 50:
        M[rng.random((R, E)) > 20 / (R * E)] = 0               # few of them: the window stays small
    ref = oracle.plan_multi(K, M, me, E, R)
    print(f"[sources] T={T} k={k} E={E} R={R} me={me} most={most} rows={ref.window_rows} {schedule}", flush=True)
    X = rng.integers(0, 1 << 15, size=(T, 8), dtype=np.uint16)
    layer = MoeLayer(T, 8, k, E, R, schedule=moe.MOE_SCHEDULE_DECODE if schedule == "decode" else moe.MOE_SCHEDULE_PREFILL,
                     rank_id=me, source_count=to_device(M), window_rows=max(1, ref.window_rows))
    layer.window.view(torch.int16).fill_(0x7B7B)
    layer.dispatch(to_device(X), to_device(K))
    p, N = layer.plan, T * k
    assert np.array_equal(to_host(p.row_map)[:N].reshape(T, k), ref.row_map)
    assert np.array_equal(to_host(p.send_idx)[:N].reshape(T, k), ref.s)
    for got, exp in ((p.expert_count, ref.c_exp), (p.rank_count, ref.c_rank), (p.expert_offset, ref.expert_offset),
                     (p.recv_count, ref.recv_count), (p.recv_offset, ref.recv_offset), (p.status[:3], ref.status)):
        assert np.array_equal(to_host(got), exp)
    want = oracle.dispatch(X, ref.row_map, max(1, ref.window_rows), fill=np.uint16(0x7B7B))
    assert to_host(layer.window).tobytes() == want.tobytes()


@pytest.mark.parametrize("T,H,k,E,R,me,stride", [
    (3077, 264, 1, 32, 4, 2, 0), (1539, 1032, 2, 48, 8, 0, 700), (769, 8200, 3, 30, 5, 4, 0), (1600, 4104, 4, 64, 4, 1, 0),      # 8, 4 and 2 tokens
    (130, 8200, 5, 16, 2, 1, 0), (130, 9216, 8, 64, 4, 2, 400), (90, 14336, 8, 40, 5, 2, 0), (101, 1032, 10, 513, 3, 1, 0),    # one, or part of one
    (770, 16392, 3, 16, 2, 0, 0)])
@pytest.mark.parametrize("quant", [False, True])
def test_several_sources_rows(moe, T, H, k, E, R, me, stride, quant):
    from paper_2605_06055_amd.layer import MoeLayer, to_device, to_host
    rng = np.random.default_rng(T + H + k)
    K = wl.random_routing(rng, T, k, E, p_masked=0.05, p_invalid=0.02)
    M = rng.integers(0, 6, size=(R, E)).astype(np.int32)
    ref = oracle.plan_multi(K, M, me, E, R, stride)
    rows = max(1, R * stride if stride else ref.window_rows)
    X = wl.f32_to_bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    print(f"[sources] T={T} H={H} k={k} E={E} R={R} me={me} stride={stride} quant={quant} rows={rows}", flush=True)
    layer = MoeLayer(T, H, k, E, R, schedule=moe.MOE_SCHEDULE_DECODE, region_stride_rows=stride, rank_id=me, source_count=to_device(M),
                     window_rows=rows)
    p, N = layer.plan, T * k
    for t in (p.expert_count, p.expert_offset, p.recv_count, p.recv_offset, p.send_idx, p.row_map, p.status):
        t.fill_(-7)
    if quant:
        codes = torch.full((rows, H), 0xAA, dtype=torch.uint8, device="cuda")
        scales = torch.full((rows,), -1.0, device="cuda")
        moe.moe_dispatch_quant(layer.shape, to_device(X), to_device(K), p, codes, scales)
        want = oracle.dispatch_quant(X, ref.row_map, rows, fill=0xAA)
        assert codes.cpu().numpy().tobytes() == want[0].tobytes() and scales.cpu().numpy().tobytes() == want[1].tobytes()
    else:
        layer.window.view(torch.int16).fill_(0x7B7B)
        layer.dispatch(to_device(X), to_device(K))
        assert to_host(layer.window).tobytes() == oracle.dispatch(X, ref.row_map, rows, fill=np.uint16(0x7B7B)).tobytes()
    assert np.array_equal(to_host(p.row_map)[:N].reshape(T, k), ref.row_map)
    assert np.array_equal(to_host(p.send_idx)[:N].reshape(T, k), ref.s)
    for got, exp in ((p.expert_count, ref.c_exp), (p.rank_count, ref.c_rank), (p.expert_offset, ref.expert_offset),
                     (p.recv_count, ref.recv_count), (p.recv_offset, ref.recv_offset), (p.status[:3], ref.status)):
        assert np.array_equal(to_host(got), exp)
