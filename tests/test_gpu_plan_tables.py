"""Count and offset tables at the numbers of experts per rank region where they are formed differently: one region
for all experts, one expert per region, segments shorter and longer than a wave, ragged ones."""
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


@pytest.mark.parametrize("E,R", [(1, 1), (1024, 1), (1024, 1024), (65, 1), (63, 3), (260, 4), (512, 2)])
@pytest.mark.parametrize("T,k", [(40, 3), (1900, 8)])          # decode and explicit schedule
def test_rank_counts(moe, E, R, T, k):
    from paper_2605_06055_amd.layer import MoeLayer, to_device, to_host
    rng = np.random.default_rng(E * 7 + R)
    H = 16
    K = wl.random_routing(rng, T, k, E, p_masked=0.05, p_invalid=0.02)
    for multi in (False, True):
        M = rng.integers(0, 50, size=(R, E)).astype(np.int32) if multi else None
        me = R // 2
        ref = oracle.plan_multi(K, M, me, E, R) if multi else oracle.plan(K, E, R)
        print(f"[tables] E={E} R={R} T={T} k={k} multi={multi}", flush=True)
        layer = MoeLayer(T, H, k, E, R, rank_id=me if multi else 0, source_count=to_device(M) if multi else None,
                         window_rows=max(1, ref.window_rows))
        for t in (layer.plan.rank_count, layer.plan.region_base, layer.plan.expert_count, layer.plan.expert_offset):
            t.fill_(-7)
        layer.dispatch(torch.zeros((T, H), dtype=torch.bfloat16, device="cuda"), to_device(K))
        torch.cuda.synchronize()
        p = layer.plan
        assert np.array_equal(to_host(p.rank_count), ref.c_rank)
        assert np.array_equal(to_host(p.region_base), ref.region_base)
        assert np.array_equal(to_host(p.expert_count), ref.c_exp)
        assert np.array_equal(to_host(p.expert_offset), ref.expert_offset)
        assert np.array_equal(to_host(p.row_map)[:T * k].reshape(T, k), ref.row_map)
