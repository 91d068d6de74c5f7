"""Default launches of medium cubes, whose tiles are all resident at once:
chunks that do not divide the edge, two or two and a half tiles a compute
unit.  Against the direct pass, which knows no tiles: the same arithmetic at
every site, sums in another order.  A mean that rounds differently moves a
deviation by a rounding of its FP32 drift at most, 2^-24 a step."""
import numpy as np
import pytest

from paper_0712_0813_amd import ce

pytestmark = pytest.mark.gpu

STEPS = 3


@pytest.mark.parametrize("N,nf,precision", [(160, 1, ce.CE_FP32), (192, 2, ce.CE_FP32), (192, 1, ce.CE_FP64),
                                            (224, 1, ce.CE_FP32), (256, 2, ce.CE_FP32), (256, 2, ce.CE_FP64)])
def test_default_launch_against_direct(N, nf, precision):
    rng = np.random.default_rng(N)
    wave = [np.cos(2 * np.pi * rng.integers(1, 9) * np.arange(N) / N) for _ in range(3 * nf)]
    phi = np.stack([(1.0 if i == 0 else 0.0) + 1e-3 * wave[3 * i][:, None, None] * wave[3 * i + 1][:, None]
                    * wave[3 * i + 2] for i in range(nf)])
    out = []
    for direct in (False, True):
        with ce.Simulation(3, N, nf, 0.15 * N, 0.01, G=[0.0, 100.0][:nf], expansion=True, kappa=2.94,
                           precision=precision) as s:
            if direct:
                s.set_launch(ce.CE_KERNEL_DIRECT, 0, 0, 0, 0, 0)
            else:
                assert s.get_launch().as_tuple()[0] == ce.CE_KERNEL_TILED3D
            s.load(phi, 0.1 * phi)
            s.step(STEPS)
            f, fd = s.read()
            out.append((f, fd, s.energies().as_dict(nf)))
    tol = STEPS * 2.0 ** -24 if precision == ce.CE_FP32 else 1e-14
    (f, fd, e), (g, gd, h) = out
    assert np.max(np.abs(f - g)) <= tol
    # the derivative takes its own rounding and dt times the force of such a
    # difference, 4 dims / dx^2 and the couplings at most
    assert np.max(np.abs(fd - gd)) <= tol * (1 + 0.01 * (12 / 0.15 ** 2 + 103))
    for k in ("kin", "grad", "pot", "rho", "a", "mean", "mean_sq"):
        for x, y in zip(np.atleast_1d(e[k]), np.atleast_1d(h[k])):
            assert abs(x - y) <= 1e-6 * abs(y) + 1e-14, k
