"""GPU: the standalone FIR on the matrix units at the edges of its tiles (16
outputs, 1024- and 4096-float blocks, 16-tap slabs), off alignment, and with
samples that are not finite.

Bound: K products summed in FP32, each rounded to 2^-24: sqrt(K) 2^-24 relative
to the terms' root sum square, under 1e-5 up to K = 8192."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _filter(K, cplx, seed=0):
    from paper_2408_16551_amd.pfb import Fir
    a = np.random.Generator(np.random.PCG64(K + seed)).standard_normal(K)
    return a, Fir(a, "c64" if cplx else "r32")


def _ref(x, a):
    w = x.astype(np.complex128 if np.iscomplexobj(x) else np.float64)
    return np.convolve(w, a.astype(np.float32).astype(np.float64))[: x.size]


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 18, 33, 129])
@pytest.mark.parametrize("n,cplx", [(1, False), (15, True), (1023, False), (1025, True), (4097, False),
                                    ((1 << 21) + 3, False), ((1 << 20) + 5, True),
                                    ((1 << 23) + 3, False), ((1 << 22) + 5, True)])
def test_edges_and_alignment(K, n, cplx):
    a, f = _filter(K, cplx)
    g = np.random.Generator(np.random.PCG64(n))
    x = g.standard_normal(n) + (1j * g.standard_normal(n) if cplx else 0)
    x = x.astype(np.complex64 if cplx else np.float32)
    ref = _ref(x, a)
    xd = torch.from_numpy(x).cuda()
    y = f(xd).cpu().numpy()
    assert np.linalg.norm(y - ref) <= 1e-5 * np.linalg.norm(ref)
    off = torch.zeros(n + 1, dtype=xd.dtype, device="cuda")
    f(xd, out=off[1:])
    assert np.array_equal(off[1:].cpu().numpy(), y) and complex(off[0]) == 0


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_samples_that_are_not_finite_reach_their_taps_only(bad):
    K, n, at = 40, 9000, 4100
    a, f = _filter(K, False)
    x = np.random.Generator(np.random.PCG64(3)).standard_normal(n).astype(np.float32)
    ref = _ref(x, a)
    x[at] = bad
    y = f(torch.from_numpy(x).cuda()).cpu().numpy()
    hit = np.zeros(n, bool)
    hit[at: at + K] = True
    assert np.all(np.isfinite(y[~hit])) and np.linalg.norm((y - ref)[~hit]) <= 1e-5 * np.linalg.norm(ref)
    want = bad * a.astype(np.float32)
    assert np.array_equal(np.isnan(y[hit]), np.isnan(want))
    ok = ~np.isnan(want)
    assert np.array_equal(y[hit][ok], want[ok])
