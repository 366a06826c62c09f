"""GPU: the FIR's 16-byte stores write what its narrower stores write.

A 16-byte aligned input takes 4 floats per thread (16-byte stores) for up to 8
taps; the same samples 8 bytes off alignment take 2 (8-byte stores), with the
same multiply-adds in the same order, so the two outputs are equal bit for bit.
Long streams, because a store whose data registers were overwritten too early
showed in 1-3 frames of 10^5.
"""
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("P,M,log2n", [(128, 6, 24), (256, 8, 24), (4096, 8, 25), (64, 4, 22)])
def test_wide_stores_equal_narrow_stores_bitwise(P, M, log2n):
    from paper_2408_16551_amd.pfb import Plan
    n = 1 << log2n
    g = torch.Generator(device="cuda").manual_seed(P + M)
    buf = torch.view_as_complex(torch.randn(n + 1, 2, generator=g, device="cuda"))
    x = buf[1:].clone()
    plan = Plan(P, M, "c64", "rect", "fp32", "fir")
    want = torch.view_as_real(plan(buf[1:])).view(torch.int32)   # 8 bytes off: 2 floats per thread
    assert x.data_ptr() % 16 == 0 and buf[1:].data_ptr() % 16 == 8
    out = plan.alloc_out(n // P)
    for _ in range(6):
        got = torch.view_as_real(plan(x, out=out)).view(torch.int32)
        assert int((got != want).sum()) == 0
