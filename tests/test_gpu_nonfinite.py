"""GPU: samples that are infinite or NaN through the folded product, the
one-kernel narrow frames and the factored DFT.  A frame whose taps reach such a
sample has no finite channel (the zero imaginary parts of a real frame's first
and last channel aside), every other frame keeps the bits of the clean call.

The patterns: both infinities, the default NaN, NaNs whose payload is all ones
(what a buffer filled with 0xFF bytes holds) and one with the smallest payload."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
BAD = [0x7F800000, 0xFF800000, 0x7FC00000, 0x7FFFFFFF, 0xFFFFFFFF, 0x7FF80000, 0x7F800001]


def _x(P, F, cplx, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    x = g.standard_normal(P * F * (2 if cplx else 1)).astype(np.float32)
    return x.view(np.complex64) if cplx else x


def _plan(P, M, cplx, prec, dft="dense"):
    from paper_2408_16551_amd.pfb import Plan
    return Plan(P, M, "c64" if cplx else "r32", "hamming", prec, dft=dft)


def _check(X, want, hit):
    assert np.array_equal(X[~hit], want[~hit])
    assert not np.isfinite(X[hit]).any()


@pytest.mark.parametrize("P,M,cplx,F,prec,dft", [
    (P, M, cplx, F, prec, "dense")
    for P, M, cplx, F in [(256, 5, False, 70), (1024, 3, False, 6200), (512, 16, True, 70), (2048, 8, True, 70),
                          (2048, 1, True, 900)]
    for prec in ("fp32", "bf16", "bf16x3", "fp8")
] + [(P, M, cplx, F, prec, "dense") for P, M, cplx, F in [(16, 4, False, 300), (64, 3, True, 70)]
     for prec in ("fp32", "bf16", "bf16x3")]
  + [(256, 4, False, 70, "fp32", "factored"), (4096, 8, True, 40, "fp32", "factored")])
def test_not_finite_samples_leave_no_finite_channel(P, M, cplx, F, prec, dft):
    from paper_2408_16551_amd.pfb import Batch
    plan = _plan(P, M, cplx, prec, dft)
    x = _x(P, F, cplx, P + M)
    want = plan(torch.from_numpy(x).cuda()).cpu().numpy()
    batch = Batch(prec, max_items=1, workspace_bytes=1 << 28)
    floats = P * (2 if cplx else 1)
    for i, bits in enumerate(BAD):
        f = 3 + 4 * i
        y = x.copy()
        y.view(np.uint32)[f * floats + (37 * i + 11) % floats] = bits
        hit = np.zeros(F, bool)
        hit[f:f + M] = True
        yd = torch.from_numpy(y).cuda()
        _check(plan(yd).cpu().numpy(), want, hit)
        out = plan.alloc_out(F)
        batch.execute([(plan, yd, out)])
        _check(out.cpu().numpy(), want, hit)


@pytest.mark.parametrize("P,cplx", [(256, False), (1024, True), (2048, True)])
def test_largest_finite_values_stay_finite_in_fp8(P, cplx):
    """One sample a frame, up to the largest float, through a unit tap: the
    rounding to four significant bits saturates at 1.875 2^127, as E4M3's does at
    its largest value.  A channel is the sample times a root of unity: relative
    2^-4 at most for the value, 2^-8 for the bfloat16 coefficient of each of its
    two parts."""
    F = 6
    x = np.zeros(P * F, np.complex64 if cplx else np.float32)
    vals = np.array([0x7F7FFFFF, 0xFF7FFFFF, 0x7F780000, 0x7F77FFFF, 0x7F700001, 0x3F780000], np.uint32).view(np.float32)
    at = np.arange(F) * P + np.array([0, 5, P // 2 - 1, P // 2, P - 1, 77])
    x[at] = vals
    from paper_2408_16551_amd.pfb import Plan
    plan = Plan(P, 1, "c64" if cplx else "r32", "custom", "fp8", custom_taps=np.ones(P))
    X = plan(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.complex128)
    ref = np.fft.fft if cplx else np.fft.rfft
    want = ref(x.reshape(F, P).astype(np.complex128 if cplx else np.float64))
    assert np.isfinite(X).all()
    assert (np.abs(X - want).max(axis=1) <= (2.0 ** -4 + 2.0 ** -7) * np.abs(vals.astype(np.float64))).all()
