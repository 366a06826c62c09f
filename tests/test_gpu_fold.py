"""GPU: the folded dense product (256 channels and more; FP32, BF16, BF16x3, FP8)
against the FP64 oracle at the edges of its tiles (64 and 128 rows, a row being
a real frame or half a complex one), of the tap rings and of the channel range,
and its kernels against each other bit for bit.

Bounds: those of the forms at every size (unit roundoff times the operand and
product roundings; FP32 1e-5 as required; FP8 half an E4M3 step, 2^-4 / sqrt 12
= 0.018 to 0.036 over a binade, 0.024 on average)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
BOUND = {"fp32": 1e-5, "bf16": 8e-3, "bf16x3": 1e-5, "fp8": 0.03}


def rel_l2(got, ref):
    return float(np.linalg.norm(got.astype(np.complex128) - ref) / np.linalg.norm(ref))


def _x(P, F, cplx, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    n = P * F + P // 3
    x = g.standard_normal(n)
    if cplx:
        return (x + 1j * g.standard_normal(n)).astype(np.complex64)
    return x.astype(np.float32)


def _plan(P, M, cplx, prec, dft="dense"):
    from paper_2408_16551_amd.pfb import Plan
    return Plan(P, M, "c64" if cplx else "r32", "hann", prec, dft=dft)


def _run(plan, x, state=None):
    return plan(torch.from_numpy(x).cuda(), state=state).cpu().numpy()


def _us(plan, x, frames):
    out, best = plan.alloc_out(frames), 1e9
    for _ in range(6):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(10):
            plan(x, out=out)
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 100)
    return best


@pytest.mark.gpu
@pytest.mark.parametrize("prec", list(BOUND))
@pytest.mark.parametrize("P,M,cplx,F", [
    (256, 1, False, 1), (256, 5, True, 33), (256, 16, False, 129), (512, 9, True, 65), (512, 17, False, 64),
    (1024, 8, True, 31), (1024, 12, False, 200), (2048, 33, True, 18), (4096, 8, False, 70), (8192, 3, True, 9),
])
def test_folded_product_matches_oracle(oracle, P, M, cplx, F, prec):
    x = _x(P, F, cplx, P + 10 * M + F)
    X = _run(_plan(P, M, cplx, prec), x)
    ref = oracle.pfb(x, P, M, oracle.window(P, M, "hann"))
    assert X.shape == ref.shape
    assert rel_l2(X, ref) < BOUND[prec]
    if not cplx:
        assert np.all(X[:, [0, P // 2]].imag == 0.0)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", list(BOUND))
@pytest.mark.parametrize("P,M,cplx,F", [(256, 4, True, 9000), (1024, 16, False, 9001), (4096, 8, True, 1030)])
def test_short_and_long_calls_agree_bitwise(P, M, cplx, F, prec):
    """A long call (128-row tiles), a short one (64-row tiles, a wave a part),
    uneven chunks through a state, an input off 16-byte alignment and a batch."""
    from paper_2408_16551_amd.pfb import Batch, State
    x = _x(P, F, cplx, 7)
    plan = _plan(P, M, cplx, prec)
    want = _run(plan, x)
    assert np.array_equal(_run(plan, x[: 37 * P + 5]), want[:37])
    st = State(plan)
    cut = [0, 3 * P + 1, 11 * P + 1, 11 * P + 7, 60 * P, 60 * P + 2, x.size]
    parts = [_run(plan, x[a:b], st) for a, b in zip(cut[:-1], cut[1:])]
    assert np.array_equal(np.concatenate(parts), want)
    off = torch.empty(x.size + 1, dtype=torch.from_numpy(x[:1]).dtype, device="cuda")
    off[1:] = torch.from_numpy(x).cuda()
    assert np.array_equal(plan(off[1:]).cpu().numpy(), want)
    b = Batch(prec, max_items=2, workspace_bytes=1 << 30)
    xs = [torch.from_numpy(x).cuda(), torch.from_numpy(x[: 41 * P]).cuda()]
    outs = [plan.alloc_out(t.numel() // P) for t in xs]
    b.execute([(plan, t, o) for t, o in zip(xs, outs)])
    assert np.array_equal(outs[0].cpu().numpy(), want) and np.array_equal(outs[1].cpu().numpy(), want[:41])


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp8"])
def test_batch_mixes_folded_and_unfolded_items_bitwise(prec):
    from paper_2408_16551_amd.pfb import Batch
    items, want = [], []
    for i, (P, M, cplx, F) in enumerate([(64, 5, True, 300), (256, 9, False, 131), (128, 16, False, 77),
                                         (2048, 20, True, 40), (512, 3, True, 0), (1024, 40, False, 65)]):
        x = torch.from_numpy(_x(P, F, cplx, 50 + i)[: P * F]).cuda()
        plan = _plan(P, M, cplx, prec)
        want.append(plan(x).cpu().numpy())
        items.append((plan, x, plan.alloc_out(F)))
    Batch(prec, max_items=len(items), workspace_bytes=1 << 28).execute(items)
    for (_, _, out), w in zip(items, want):
        assert np.array_equal(out.cpu().numpy(), w)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("P,M,F", [(256, 3, 1), (256, 16, 129), (512, 8, 33), (1024, 1, 65), (4096, 5, 34), (8192, 2, 7)])
def test_folded_synthesis_matches_oracle(oracle, P, M, F, prec):
    """Synthesis through the folded inverse, also in workspace pieces and
    chunks through a state, bit for bit."""
    from paper_2408_16551_amd.pfb import Plan, State
    g = np.random.Generator(np.random.PCG64(P + M + F))
    X = (g.standard_normal((F, P)) + 1j * g.standard_normal((F, P))).astype(np.complex64)
    plan = Plan(P, M, "c64", "hann", prec, "inverse")
    Xd = torch.from_numpy(X).cuda()
    got = plan.synthesize(Xd).cpu().numpy()
    ref = oracle.synthesize(X.astype(np.complex128), P, M, oracle.window(P, M, "hann"))
    assert rel_l2(got, ref) < BOUND[prec]
    small = Plan(P, M, "c64", "hann", prec, "inverse", workspace_bytes=P * 16 * 5)
    assert np.array_equal(small.synthesize(Xd).cpu().numpy(), got)
    st, cut = State(plan), sorted({0, F // 3, F // 2, F})
    parts = [plan.synthesize(Xd[a:b].clone(), state=st).cpu().numpy() for a, b in zip(cut[:-1], cut[1:])]
    assert np.array_equal(np.concatenate(parts), got)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", list(BOUND))
@pytest.mark.parametrize("P,M,F", [(512, 1, 1), (512, 8, 17), (1024, 16, 31), (1024, 20, 33), (2048, 16, 15),
                                   (2048, 7, 66), (2048, 17, 40), (8192, 64, 3)])
def test_split_frames_match_oracle_and_batch(oracle, P, M, F, prec):
    """Complex frames about the sizes and tap counts where they go in two halves:
    the oracle, every value by itself, and a batch that mixes them (tap counts
    up to 16, then with a longer one) bit for bit."""
    from paper_2408_16551_amd.pfb import Batch
    x = _x(P, F, True, P + 7 * M + F)
    plan = _plan(P, M, True, prec)
    got = _run(plan, x)
    ref = oracle.pfb(x, P, M, oracle.window(P, M, "hann"))
    assert rel_l2(got, ref) < BOUND[prec]
    # Every value: white noise in, so each channel's error is complex normal of the
    # forms' relative size times the spectrum's level, and beyond eight times it
    # with probability exp(-64); a value at the wrong place is off by the level.
    assert np.abs(got - ref).max() < 8 * BOUND[prec] * np.sqrt(np.mean(np.abs(ref) ** 2))
    xd = torch.from_numpy(x).cuda()
    for other in (_plan(1024, 5, True, prec), _plan(256, 33, False, prec)):
        z = torch.from_numpy(_x(other.P, 40, other.sample_type == "c64", 3)).cuda()
        items = [(plan, xd, plan.alloc_out(F)), (other, z, other.alloc_out(40))]
        Batch(prec, max_items=2, workspace_bytes=1 << 28).execute(items)
        assert np.array_equal(items[0][2].cpu().numpy(), got)
        assert np.array_equal(items[1][2].cpu().numpy(), other(z).cpu().numpy())


@pytest.mark.gpu
def test_folded_fp8_plan_holds_no_scale_workspace():
    """1 GiB of workspace: the plan's device memory is BF16's (within 4 MiB of
    allocation granularity), without 36 MiB of frame maxima and exponents."""
    from paper_2408_16551_amd.pfb import Plan
    Plan(1024, 4, "r32", "hann", "bf16", workspace_bytes=1 << 20).close()
    used = {}
    for prec in ("bf16", "fp8"):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        plan = Plan(1024, 4, "r32", "hann", prec, workspace_bytes=1 << 30)
        used[prec] = before - torch.cuda.mem_get_info()[0]
        plan.close()
    assert used["bf16"] >= 1000 << 20 and abs(used["fp8"] - used["bf16"]) <= 4 << 20


@pytest.mark.gpu
@pytest.mark.parametrize("prec", list(BOUND))
@pytest.mark.parametrize("P,cplx", [(256, False), (512, True), (2048, True)])
def test_more_than_16_taps(oracle, P, cplx, prec):
    """Tap and frame counts about the 32 frames and 8 taps that the long FIR takes at
    a time (whole and split frames): the oracle, and chunks through a state bit for
    bit."""
    from paper_2408_16551_amd.pfb import State
    for M, F in ((17, 33), (24, 16), (25, 31), (31, 64), (32, 1), (33, 32), (40, 65), (63, 47), (64, 100)):
        x = _x(P, F, cplx, P + M)
        plan = _plan(P, M, cplx, prec)
        got = _run(plan, x)
        assert rel_l2(got, oracle.pfb(x, P, M, oracle.window(P, M, "hann"))) < BOUND[prec]
        st, cut = State(plan), sorted({0, P // 2 + 1, x.size // 3, x.size // 2 // P * P, x.size})
        parts = [_run(plan, x[a:b], st) for a, b in zip(cut[:-1], cut[1:])]
        assert np.array_equal(np.concatenate(parts), got)


@pytest.mark.gpu
def test_64_taps_cost_no_more_than_four_times_16():
    """1024 real channels, BF16, 4763 frames: measured 1.05 times; 23.7 times with a
    ring of 64 taps in registers, 2.0 with the plain product."""
    x = torch.randn(4763 * 1024, device="cuda")
    assert _us(_plan(1024, 64, False, "bf16"), x, 4763) < 4 * _us(_plan(1024, 16, False, "bf16"), x, 4763)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", list(BOUND))
@pytest.mark.parametrize("P,cplx", [(256, False), (256, True), (512, True), (2048, True), (1024, False)])
def test_few_taps(oracle, P, cplx, prec):
    """Tap counts of which several rings fill a phase of the folding FIR, frame counts
    about whole phases, rings and units: the oracle, and bit for bit chunks through a
    state, an input off 16-byte alignment and a batch."""
    from paper_2408_16551_amd.pfb import Batch, State
    items, want = [], []
    for M, F in ((1, 15), (1, 49), (2, 33), (3, 47), (4, 17), (5, 31), (6, 61), (7, 100), (7, 6)):
        x = _x(P, F, cplx, P + M)
        plan = _plan(P, M, cplx, prec)
        got = _run(plan, x)
        assert rel_l2(got, oracle.pfb(x, P, M, oracle.window(P, M, "hann"))) < BOUND[prec]
        st, cut = State(plan), sorted({0, P // 2 + 1, x.size // 3, x.size // 2 // P * P, x.size})
        parts = [_run(plan, x[a:b], st) for a, b in zip(cut[:-1], cut[1:])]
        assert np.array_equal(np.concatenate(parts), got)
        off = torch.empty(x.size + 1, dtype=torch.from_numpy(x[:1]).dtype, device="cuda")
        off[1:] = torch.from_numpy(x).cuda()
        assert np.array_equal(plan(off[1:]).cpu().numpy(), got)
        items.append((plan, off[1:], plan.alloc_out(F)))
        want.append(got)
    Batch(prec, max_items=len(items), workspace_bytes=1 << 28).execute(items)
    for (_, _, out), w in zip(items, want):
        assert np.array_equal(out.cpu().numpy(), w)



@pytest.mark.gpu
def test_one_tap_costs_no_more_than_sixteen():
    """256 complex channels, BF16, 2^24 samples: at most 1.5 times (measured 0.94; 2.2
    with a barrier for every M frames, 1.1 with the plain product)."""
    x = torch.randn(1 << 24, dtype=torch.complex64, device="cuda")
    assert _us(_plan(256, 1, True, "bf16"), x, 1 << 16) < 1.5 * _us(_plan(256, 16, True, "bf16"), x, 1 << 16)
