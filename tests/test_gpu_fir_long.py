"""GPU: the FIR of more than 16 taps (tap after tap; whole rings of 32 and 64 taps in
long calls), in every output form: against the batched FIR (a ring of all taps, another
kernel) and chunks through a state bit for bit, and the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
# The forms' bounds at every size.
BOUND = {"fp32": 1e-5, "bf16": 8e-3, "bf16x3": 1e-5, "fp16": 1e-3, "fp16x3": 2.5e-6, "fp8": 0.1, "mxfp8": 0.05}


def _x(n, cplx, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    x = g.standard_normal(n * (2 if cplx else 1)).astype(np.float32)
    return x.view(np.complex64) if cplx else x


@pytest.mark.parametrize("P,cplx,prec,dft,out", [
    (64, False, "fp32", "compensated", "pfb"), (64, True, "bf16", "dense", "pfb"), (128, True, "bf16x3", "dense", "pfb"),
    (256, False, "fp16", "dense", "pfb"), (2048, True, "fp16", "dense", "pfb"), (1024, True, "fp16x3", "dense", "pfb"),
    (128, True, "fp8", "dense", "pfb"), (128, False, "mxfp8", "dense", "pfb"), (512, True, "mxfp8", "dense", "pfb"),
    (512, True, "fp32", "factored", "pfb"), (16, False, "fp32", "table", "pfb"), (32, True, "fp32", "dense", "fir")])
def test_tap_and_frame_counts(oracle, P, cplx, prec, dft, out):
    from paper_2408_16551_amd.pfb import Batch, Plan, State
    for M, F in ((17, 33), (24, 7), (31, 65), (32, 64), (32, 95), (33, 32), (48, 31), (63, 100), (64, 130), (64, 1)):
        x = _x(P * F + P // 2, cplx, P + M)
        plan = Plan(P, M, "c64" if cplx else "r32", "hann", prec, out, dft=dft)
        xd = torch.from_numpy(x).cuda()
        got = plan(xd).cpu().numpy()
        h = oracle.window(P, M, "hann")
        ref = oracle.pfb(x, P, M, h) if out == "pfb" else oracle.fir(x, P, M, h)
        assert np.linalg.norm(got - ref) < BOUND[prec] * np.linalg.norm(ref)
        st, cut = State(plan), sorted({0, P // 2 + 1, x.size // 3, x.size // 2 // P * P, x.size})
        parts = [plan(xd[a:b].clone(), state=st).cpu().numpy() for a, b in zip(cut[:-1], cut[1:])]
        assert np.array_equal(np.concatenate(parts), got)
        if out == "pfb" and dft in ("dense", "factored"):
            o = plan.alloc_out(F)
            Batch(prec, max_items=1, workspace_bytes=1 << 28).execute([(plan, xd, o)])
            assert np.array_equal(o.cpu().numpy(), got)


@pytest.mark.parametrize("M", [32, 64])
@pytest.mark.parametrize("P,cplx,prec", [(128, False, "fp16"), (64, True, "bf16"), (128, True, "mxfp8"), (128, False, "fp8")])
def test_long_calls_in_whole_rings_first_and_last_frames(P, cplx, prec, M):
    """2^25 floats and more (the rings apart from the rest), 2^22 and 3 * 2^23 (whole
    rings and a few frames more), frames left over, the first one begun in the history:
    the same stream in one call, in two through a state and in a batch, bit for bit."""
    from paper_2408_16551_amd.pfb import Batch, Plan, State
    W = P * (2 if cplx else 1)
    F = (1 << 25) // W + 77
    x = torch.from_numpy(_x(P * (F + 3) + 5, cplx, M)).cuda()
    plan = Plan(P, M, "c64" if cplx else "r32", "hann", prec)
    got = plan(x)
    st = State(plan)
    parts = [plan(x[a:b].clone(), state=st).clone() for a, b in ((0, 2 * P + 3), (2 * P + 3, x.numel()))]
    assert torch.equal(torch.cat(parts), got)
    o = plan.alloc_out(F + 3)
    Batch(prec, max_items=1, workspace_bytes=1 << 28).execute([(plan, x, o)])
    assert torch.equal(o, got)
    for n in ((1 << 22) // W + 4, (1 << 22) // W + 5, (3 << 23) // W + 8, (3 << 23) // W + 9):
        assert torch.equal(plan(x[:n * P]), got[:n])
