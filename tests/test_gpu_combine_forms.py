"""Combine at the degrees and widths that choose its form: 5 and 10 rows with results held back (at the numbers of results per thread
where they move), rows of 3 and 9 waves in workgroups of 3, one row past and short of them, small launches, workgroups of whole rows."""
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


STREAMS = 1536 * 1024                                          # vectors of Y beyond which a launch streams


def cases():
    threads = 256 * 512
    for k, dtype, H16 in ((10, "bf16", 144), (10, "f32", 513), (5, "bf16", 256), (5, "f32", 224)):
        padded = (H16 + 63) // 64 * 64
        yield k, dtype, H16, STREAMS // H16 + 1
        for per_thread in (36, 56):
            for more in (0, 1):
                yield k, dtype, H16, threads * per_thread // padded + more
    for k in (1, 2, 3, 4, 5, 7):
        for H16 in (128, 129, 192, 193, 513, 576):
            yield k, "bf16", H16, STREAMS // H16 + 1
    for k in (3, 5, 10, 11):
        for H16 in (1, 64, 129, 513):
            yield k, "f32", H16, 77
    # workgroups of a whole row or an equal part of it: ragged rows, idle columns; each width at two degrees, each degree at several widths
    forms = ((1, "bf16"), (6, "bf16"), (8, "f32"), (10, "bf16"), (11, "bf16"))
    for n, H16 in enumerate((1, 65, 80, 96, 333, 641, 705, 833, 897, 1089, 1857)):
        for k, dtype in (forms[n % 5], forms[(n + 2) % 5]):
            yield k, dtype, H16, -(-100000 // H16) if H16 <= 256 or k == 1 else max(640, -(-2400000 // (k * H16)))
    for k, H16 in ((8, 72), (6, 144), (6, 513)):               # streaming launches that do not hold their results back
        yield k, "bf16", H16, STREAMS // H16 + 1


@pytest.mark.parametrize("k,dtype,H16,T", list(cases()))
def test_combine(moe, k, dtype, H16, T, shift=0):
    bf16 = dtype == "bf16"
    H = H16 * (8 if bf16 else 4)
    print(f"[forms] T={T} H={H} k={k} {dtype}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + k)
    storage = torch.bfloat16 if bf16 else torch.float32
    # small integers: every product and partial sum is exact in fp32, so only the last rounding is left
    out = torch.empty(T * k * H + shift * (H // H16), dtype=storage, device="cuda")[shift * (H // H16):].view(T * k, H)
    out.copy_(torch.randint(-8, 9, (T * k, H), generator=gen, device="cuda", dtype=torch.int8))
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


@pytest.mark.parametrize("k,H16,T", [(8, 896, 128), (6, 512, 400), (8, 512, 700), (8, 512, 3200), (3, 576, 3000)])
def test_combine_of_rows_past_a_line(moe, k, H16, T):
    """expert_out that starts 16 bytes past a cache line: rows of whole lines that all start inside one."""
    test_combine(moe, k, "bf16", H16, T, shift=1)
