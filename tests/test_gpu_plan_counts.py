"""The explicit plan at the numbers of branches and experts where its counting changes form: one launch and two, histogram rows of
whole and of ragged pieces, more columns than threads' parts, runs of tiles that end inside a range, tiles of 2048 branches, tiles too
long for 16-bit counts; against the oracle."""
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


def expected_list(K, row_map, E, H):
    """The dispatch order list of rows of H bf16: inside each stretch the counted branches by (expert, flat index) as (token, row),
    then unused entries.  A single-launch plan of up to 12288 branches is one stretch; otherwise stretches are whole tiles of 1024
    branches (2048 from 196608 on), about 28 MB of X and as equal as whole tiles allow."""
    T, k = K.shape
    N, flat = T * k, K.reshape(-1)
    tile = 1024 if N < 196608 else 2048
    tiles, most = -(-N // tile), (28 << 20) // (2 * H) * k // tile
    stretch = N if N <= 12288 else -(-tiles // -(-tiles // most)) * tile
    out = np.full((N, 2), -1, np.int32)
    for a in range(0, N, stretch):
        at = np.arange(a, min(a + stretch, N))
        at = at[(flat[at] >= 0) & (flat[at] < E)]
        at = at[np.argsort(flat[at], kind="stable")]
        out[a:a + len(at)] = np.stack([at // k, row_map.reshape(-1)[at]], 1)
    return out


@pytest.mark.parametrize("T,k,E,R", [(3073, 4, 256, 8), (4097, 3, 255, 5), (7168, 4, 512, 2), (7169, 4, 512, 2), (28672, 1, 3, 1), (4099, 4, 8, 8), (6144, 4, 12, 4),
                                     (3584, 8, 1024, 8), (5734, 5, 1, 1), (12800, 1, 2, 2), (4096, 8, 7, 7), (4096, 8, 1024, 1),
                                     (4100, 8, 257, 1), (24575, 8, 512, 4), (24576, 8, 1023, 3), (65537, 8, 64, 8),
                                     (131073, 8, 1024, 4), (16777217, 1, 5, 5)])
@pytest.mark.parametrize("one", [False, True])                # all ids the same
def test_plan(moe, T, k, E, R, one):
    from paper_2605_06055_amd.layer import to_device, to_host
    rng = np.random.default_rng(T + E)
    K = np.full((T, k), E - 1, np.int32) if one else rng.integers(-1, E, size=(T, k), dtype=np.int32)
    K[rng.integers(0, T, 5), 0] = E + 3
    ref = oracle.plan(K, E, R)
    H = 1024 if T <= 32768 else 8                              # with and without the order list
    shape = moe.MoeShape(T=T, H=H, k=k, E=E, R=R, dtype=moe.MOE_DTYPE_BF16, schedule=moe.MOE_SCHEDULE_PREFILL)
    print(f"[plan] T={T} k={k} E={E} R={R} H={H} one={one}", flush=True)
    p = moe.MoePlan(shape)
    p.dispatch_order.fill_(-77)
    moe.moe_plan(shape, to_device(K), p)
    N = T * k
    assert np.array_equal(to_host(p.row_map)[:N].reshape(T, k), ref.row_map)
    assert np.array_equal(to_host(p.send_idx)[:N].reshape(T, k), ref.s)
    for got, exp in ((p.expert_count, ref.c_exp), (p.rank_count, ref.c_rank), (p.expert_offset, ref.expert_offset),
                     (p.region_base, ref.region_base), (p.status[:3], ref.status)):
        assert np.array_equal(to_host(got), exp)
    pairs = to_host(p.dispatch_order)[:2 * N].reshape(N, 2)
    want = expected_list(K, ref.row_map, E, H) if H == 1024 else np.full((N, 2), -77, np.int32)
    assert np.array_equal(pairs, want)
