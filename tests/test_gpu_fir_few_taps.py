"""GPU: the FIR of 1 to 8 taps, several short rings at a time, where a wave holds runs of
several lengths (narrow rows, a last run that ends early): against the FP64 oracle, and
chunks through a state and a batch bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
BOUND = {"fp32": 1e-6, "fp16": 1e-3, "fp8": 0.1, "mxfp8": 0.05}  # the FIR alone in FP32; the forms' bounds


@pytest.mark.parametrize("P,cplx,prec,out", [(16, False, "fp32", "fir"), (32, True, "fp32", "fir"), (1024, False, "fp32", "fir"),
                                             (16, True, "fp16", "pfb"), (256, True, "fp16", "pfb"), (64, False, "fp8", "pfb"),
                                             (128, False, "mxfp8", "pfb")])
def test_tap_and_frame_counts(oracle, P, cplx, prec, out):
    from paper_2408_16551_amd.pfb import Batch, Plan, State
    g = np.random.Generator(np.random.PCG64(P))
    items, want = [], []
    for M in range(1, 9):
        for F in (1, 7, 8, 23, 40 + M, 1000 + 3 * M):
            n = P * F + P // 2
            x = g.standard_normal(n) + (1j * g.standard_normal(n) if cplx else 0)
            x = x.astype(np.complex64 if cplx else np.float32)
            plan = Plan(P, M, "c64" if cplx else "r32", "hamming", prec, out)
            xd = torch.from_numpy(x).cuda()
            got = plan(xd).cpu().numpy()
            h = oracle.window(P, M, "hamming")
            ref = oracle.pfb(x, P, M, h) if out == "pfb" else oracle.fir(x, P, M, h)
            assert np.linalg.norm(got - ref) < BOUND[prec] * np.linalg.norm(ref)
            st, cut = State(plan), sorted({0, P // 2 + 1, n // 3, n // 2 // P * P, n})
            parts = [plan(xd[a:b].clone(), state=st).cpu().numpy() for a, b in zip(cut[:-1], cut[1:])]
            assert np.array_equal(np.concatenate(parts), got)
            if out == "pfb":
                items.append((plan, xd, plan.alloc_out(F)))
                want.append(got)
    if items:
        Batch(prec, max_items=len(items), workspace_bytes=1 << 28).execute(items)
        for (_, _, o), w in zip(items, want):
            assert np.array_equal(o.cpu().numpy(), w)
