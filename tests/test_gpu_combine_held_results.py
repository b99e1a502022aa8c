"""The streaming form of combine at the numbers of results per thread where they move: the last of the short form, the last
that fit in registers, the first held in LDS, the last of one launch, the first of two; for rows that are a whole number of
waves, rows padded to one, and rows over which a thread's column wraps."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def moe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_06055_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("per_thread", [28, 36, 56])
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("k,dtype,H16", [(6, "bf16", 64), (8, "f32", 64), (6, "bf16", 513), (8, "f32", 514), (8, "bf16", 896),
                                         (8, "bf16", 513)])
def test_results_held_in_registers_and_lds(moe, per_thread, more, k, dtype, H16):
    threads = torch.cuda.get_device_properties(0).multi_processor_count * 512
    bf16 = dtype == "bf16"
    H = H16 * (8 if bf16 else 4)
    padded = (H16 + 63) // 64 * 64
    T = threads * per_thread // padded + more                  # more: one unit a thread more, for some threads
    assert -(-T * padded // threads) == per_thread + more
    print(f"[held] T={T} H={H} k={k} {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + k)
    storage = torch.bfloat16 if bf16 else torch.float32
    # small integers: every product and partial sum is exact in fp32, so only the last rounding is left
    out = torch.randint(-8, 9, (T * k, H), generator=gen, device="cuda", dtype=torch.int8).to(storage)
    w = torch.randint(-4, 5, (T, k), generator=gen, device="cuda").float()
    rows = torch.randperm(T * k, generator=gen, device="cuda").to(torch.int32).view(T, k)
    rows[torch.rand((T, k), generator=gen, device="cuda") < 0.05] = -1
    shape = moe.MoeShape(T=T, H=H, k=k, E=16, R=2, dtype=moe.MOE_DTYPE_BF16 if bf16 else moe.MOE_DTYPE_F32,
                         schedule=moe.MOE_SCHEDULE_PREFILL)
    plan = moe.MoePlan(shape)
    plan.row_map.copy_(rows.view(-1))
    y = torch.full((T + 1, H), 77.0, dtype=storage, device="cuda")
    moe.moe_combine(shape, out, w, plan, y[:T])
    want = torch.zeros((T, H), dtype=torch.float32, device="cuda")
    for j in range(k):
        at = rows[:, j].long()
        want += torch.where(at[:, None] >= 0, w[:, j:j + 1] * out[at.clamp_min(0)].float(), 0.0)
    assert torch.equal(y[:T], want.to(storage))
    assert bool((y[T] == 77.0).all())
