"""GPU: the one-kernel path of frames of at most 128 floats (FP32, BF16, BF16x3)
against the two-kernel path (a batch of one item) bit for bit and the FP64
oracle: partial and single tiles of every row width and block size, states,
inputs off 16-byte alignment, more taps than it takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
BOUND = {"fp32": 1e-5, "bf16": 8e-3, "bf16x3": 1e-5}  # the forms' bounds at every size


@pytest.mark.parametrize("prec", list(BOUND))
@pytest.mark.parametrize("P,M,cplx,F", [
    (16, 4, False, 1), (16, 1, False, 65), (16, 9, True, 700), (32, 33, False, 130), (32, 5, True, 33),
    (64, 16, False, 31), (64, 8, True, 2500), (128, 32, False, 97), (128, 7, True, 40), (16, 3, False, 270000),
    (128, 16, True, 20000),
])
def test_one_kernel_equals_two_bitwise(oracle, P, M, cplx, F, prec):
    from paper_2408_16551_amd.pfb import Batch, Plan, State
    g = np.random.Generator(np.random.PCG64(P + M + F))
    n = P * F + P // 2
    x = g.standard_normal(n)
    x = (x + 1j * g.standard_normal(n)).astype(np.complex64) if cplx else x.astype(np.float32)
    plan = Plan(P, M, "c64" if cplx else "r32", "hamming", prec)
    xd = torch.from_numpy(x).cuda()
    got = plan(xd).cpu().numpy()
    out = plan.alloc_out(F)
    Batch(prec, max_items=1, workspace_bytes=1 << 28).execute([(plan, xd, out)])
    assert np.array_equal(got, out.cpu().numpy())
    k = min(F, 700)
    ref = oracle.pfb(x[: k * P], P, M, oracle.window(P, M, "hamming"))
    assert np.linalg.norm(got[:k] - ref) < BOUND[prec] * np.linalg.norm(ref)
    off = torch.empty(n + 1, dtype=xd.dtype, device="cuda")
    off[1:] = xd
    assert np.array_equal(plan(off[1:]).cpu().numpy(), got)
    st, cut = State(plan), sorted({0, n // 5, n // 5 + 3, n // 2 // P * P, n})
    parts = [plan(xd[a:b].clone(), state=st).cpu().numpy() for a, b in zip(cut[:-1], cut[1:])]
    assert np.array_equal(np.concatenate(parts), got)


@pytest.mark.parametrize("P,M,cplx,F", [(16, 4, True, 50000), (64, 9, True, 20000), (32, 16, False, 40000)])
def test_output_over_the_input(P, M, cplx, F):
    """A call whose output lies over its input, at once and (the rows' start a
    frame later) in part: the two-kernel path, bit for bit the call with both apart."""
    from paper_2408_16551_amd.pfb import Plan
    g = torch.Generator(device="cuda").manual_seed(P)
    plan = Plan(P, M, "c64" if cplx else "r32", "hann", "fp32")
    for at in (0, 1):
        buf = torch.empty((F + 1, plan.channels_out), dtype=torch.complex64, device="cuda")
        flat = torch.view_as_real(buf).view(-1)
        src = torch.randn(F * P * (2 if cplx else 1), generator=g, device="cuda")
        x = flat[: src.numel()]
        x.copy_(src)
        x = torch.view_as_complex(x.view(-1, 2)) if cplx else x
        want = plan(x.clone())
        assert torch.equal(plan(x, out=buf[at: at + F]), want)


@pytest.mark.parametrize("P,M,cplx,prec,F", [(128, 9, False, "bf16", 131075), (64, 16, True, "bf16x3", 131073),
                                             (128, 32, False, "bf16x3", 32770), (64, 32, True, "fp32", 131072),
                                             (64, 32, False, "bf16", 262147)])
def test_long_calls_of_many_taps_take_two_kernels_with_the_same_bits(P, M, cplx, prec, F):
    """About the sizes from which these tap counts leave the one kernel: a shorter call
    (one kernel) gives the same frames."""
    from paper_2408_16551_amd.pfb import Plan
    plan = Plan(P, M, "c64" if cplx else "r32", "hann", prec)
    x = torch.randn(F * P * (2 if cplx else 1), device="cuda")
    x = torch.view_as_complex(x.view(-1, 2)) if cplx else x
    assert torch.equal(plan(x)[:1000], plan(x[:1000 * P]))
