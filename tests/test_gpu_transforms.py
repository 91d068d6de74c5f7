"""Spectra at the sizes where the work of the transforms' blocks is divided
differently: one thread a line and fewer (4), one wavefront a line (128), two
(256), four (512 in the plane), fewer histograms than wavefronts (1024), and a
last block whose lines run out (odd numbers of N/2 + 1 columns)."""
import numpy as np
import pytest

from paper_0712_0813_amd import ce
from oracle import spectrum
from _parity import Case

pytestmark = pytest.mark.gpu

SIZES = [(3, 4, ce.CE_FP64), (3, 16, ce.CE_FP32), (3, 128, ce.CE_FP32), (3, 256, ce.CE_FP32),
         (2, 4, ce.CE_FP32), (2, 128, ce.CE_FP64), (2, 512, ce.CE_FP32), (2, 1024, ce.CE_FP32)]


@pytest.mark.parametrize("dims,N,precision", SIZES)
def test_spectrum_of_read_fields(dims, N, precision):
    case = Case(f"{dims}d_{N}", dims, N, 1, 0.15 * N, 0.01, seed=71)
    phi, phid = case.inputs()
    with case.sim(precision) as s:
        s.load(phi, phid)
        s.step(2)
        f, fd = s.read()
        pf, pd, cnt = s.spectrum(0)
        again = s.spectrum(0)
    for got, want in zip((pf, pd), (f[0], fd[0])):
        power, count = spectrum(want)
        assert np.array_equal(cnt, count)
        # FP64 transforms on both sides: rounding of each bin and of the
        # largest mode, the background
        assert np.all(np.abs(got - power) <= 1e-12 * np.abs(power) + 1e-14 * power.sum())
    assert all(np.array_equal(a, b) for a, b in zip((pf, pd, cnt), again))
