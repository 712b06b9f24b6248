"""GPU kernels at the edges of their tiles and of the rules that choose between them,
against NumPy in FP64.  Every test prints its case before touching the GPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1609_03488_amd")


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _conv_solver(n, k, prec, engine):
    rng = np.random.default_rng(n + k)
    taps = rng.standard_normal(k)
    op = P.Operator(n + k - 1, n).add_conv(0, 0, taps, n, 0.75)
    st = P.Settings.make(precision=prec, normalize=0, conv_mfma=engine)
    return taps, P.Solver(op, n + k - 1, [], st), rng


# one output, less than a wave, tile edges of both forms (FP64: 128 / 256 outputs,
# FP32: 256 / 512), a step of 16 taps with and without remainders, two passes of
# 2048 taps, and both sides of the 512 tiles where the wide form takes over
@pytest.mark.parametrize("n,k", [(1, 1), (60, 3), (128, 16), (257, 17), (500, 20), (513, 36), (2500, 2051),
                                 (131040, 33), (131300, 33), (262100, 45), (262400, 40)])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32], ids=["fp64", "fp32"])
def test_direct_convolution_edges(n, k, prec):
    """|dev - ref| <= (k + 4) u sum_t |w_t||x_t| elementwise: k fused multiply-adds
    and the conversions of the operands, in the working precision."""
    print("[case] direct convolution", n, k, prec, flush=True)
    taps, s, rng = _conv_solver(n, k, prec, 0)
    x, y = rng.standard_normal(n), rng.standard_normal(n + k - 1)
    u = 2.0 ** -53 if prec == P.FP64 else 2.0 ** -24
    a, at = np.abs(taps), 0.75 * taps
    err = np.abs(s.apply(x) - np.convolve(at, x))
    assert np.all(err <= (k + 4) * u * 0.75 * np.convolve(a, np.abs(x)))
    err = np.abs(s.apply(y, transpose=True) - np.correlate(y, at, "valid"))
    assert np.all(err <= (k + 4) * u * 0.75 * np.correlate(np.abs(y), a, "valid"))
