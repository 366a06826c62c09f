"""Host-side helpers of the benchmark: the NumPy filter bank it times beside
the oracle must compute the same thing, and the per-channel error figures must
name the right channels."""
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from oracle import Oracle  # noqa: E402
from paper_2408_16551_amd import workloads  # noqa: E402


def test_numpy_pfb_real_matches_oracle():
    w = workloads.small_pfb()
    o = Oracle()
    h = o.window(w.P, w.M, w.window)
    ref = o.pfb(w.x, w.P, w.M, h)
    X64 = bench.numpy_pfb(w.x, w.P, w.M, h, np.dtype(np.float64))
    assert X64.shape == ref.shape
    assert bench.rel_l2(X64, ref) < 1e-13
    X32 = bench.numpy_pfb(w.x, w.P, w.M, h, np.dtype(np.float32))
    assert X32.dtype == np.complex64
    assert bench.rel_l2(X32, ref) < 1e-5


def test_numpy_pfb_complex_matches_oracle():
    g = np.random.Generator(np.random.PCG64(5))
    P, M, n = 32, 5, 32 * 40 + 7   # ragged tail: the last 7 samples make no frame
    x = (g.standard_normal(n) + 1j * g.standard_normal(n)).astype(np.complex64)
    o = Oracle()
    h = o.window(P, M, "blackman")
    ref = o.pfb(x, P, M, h)
    X = bench.numpy_pfb(x, P, M, h, np.dtype(np.complex128))
    assert X.shape == ref.shape == (40, P)
    assert bench.rel_l2(X, ref) < 1e-13


def test_channel_errors_names_worst_channel_and_weakest_tone():
    class W:
        P, M = 8, 2
        tones = [(2 / 8, 1.0, 0.0), (5 / 8, 1e-3, 0.0), (0.3, 1e-4, 0.0)]   # the last is off-centre
    fr = np.arange(6, dtype=np.int64)
    ref = np.ones((6, 8), dtype=np.complex128)
    got = ref.copy()
    got[1:, 3] += 0.5          # channel 3 is the worst past the warm-up frame
    got[1:, 5] += 1e-3         # the weakest centre tone sits in channel 5
    got[0, :] += 100.0         # frame 0 is warm-up (M - 1 = 1) and is not counted
    e = bench.channel_errors(got, ref, W, fr)
    assert abs(e["worst_channel_rel_l2"] - 0.5) < 1e-12
    assert e["weakest_tone"]["channel"] == 5
    assert abs(e["weakest_tone"]["rel_l2"] - 1e-3) < 1e-12


def test_line_of_a_full_run_stays_short_and_keeps_the_headline():
    """A result of every leg at its full size (ten forms on two workloads, three
    batches, ten serving runs with their latency parts): the printed line holds the
    headline's fields and stays under LINE_BYTES."""
    import json
    form = {k: 123456.789 for k in ("gsps", "ms_per_step", "dft_ms", "fir_ms", "dft_useful_tflops", "dft_mfma_frac",
                                    "worst_channel_rel_l2", "fir_hbm_gbs")}
    form.update(rel_l2_vs_fp64_oracle=1.234e-07, weakest_tone={"channel": 2812, "rel_l2": 1e-3})
    names = ["fp32", "bf16", "bf16x3", "fp16", "fp16x3", "fp8", "mxfp8", "fp32/factored", "fp32/compensated", "fp32/table"]
    head = {"metric": "PFB input GSamples/s (FP32 DFT GEMM; reduced-precision forms at their rel. error in 'forms')",
            "value": 144.123, "unit": "GSamples/s", "n_gpus": 1, "steps": 50, "warmup": 20, "ms_per_step": 0.4661,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
            "data": "synthetic (seeded N(0,1) noise + 8 channel-centre tones)",
            "config": {"workload": "real_stream_r32_p1024_m16", "channels": 1024, "taps": 16, "window": "sinc x hann",
                       "samples": 1 << 26, "sample_type": "r32", "precision": "fp32"}}
    stage = {"kernel": "fold_gemm_kernel<FP32>", "bound": "mfma", "achieved": 101.23, "peak": 157.3, "unit": "TFLOP/s",
             "frac": 0.6436, "avg_launch_ms": 0.3181}
    served = {"precision": "fp32/factored", "hbm_budget_bytes": 8 << 30, "rho": 0.5, "buffers": "device (in place)",
              "p50_ms": 0.344, "p99_ms": 12.345, "gsps_served": 91.234, "latency_parts": {str(i): 1.0 / 3 for i in range(80)}}
    full = dict(head, roofline=dict(stage, traffic=590123456.0),
                stages={"fir": stage}, forms={w: {n: form for n in names} for w in ("real_stream_r32_p1024_m16",
                                                                                    "wide_dynamic_range_c64_p4096_m8")},
                fir_only={"gsps": 700.12, "kernel_ms": 0.0921, "hbm_gbs": 5812.3, "hbm_frac": 0.7265},
                ops={str(i): form for i in range(9)}, batched={"streams": 64, "fp32": form, "bf16x3": form, "fp32/factored": form},
                serving=[served] * 10, cpu_context={str(i): 1.5 for i in range(90)},
                cpu_baseline={"value": 0.035123, "unit": "GSamples/s", "cores": 16, "kind": "oracle", "sample": "y" * 400})
    line = json.dumps(bench.summary(full))
    assert len(json.dumps(full)) > 16000 and len(line) < bench.LINE_BYTES
    got = json.loads(line)
    assert {k: got[k] for k in head} == head
    assert got["roofline"]["achieved"] == 101.23 and got["forms"]["real_stream_r32_p1024_m16"]["fp8"]["gsps"] == 123456.789
    assert got["roofline"]["traffic"] == 590123456.0
