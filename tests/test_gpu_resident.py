"""Steps taken by a resident pass (a run of steps in one launch, the state kept
on the chip) are bitwise the steps of plain launches: fields, derivatives and
every step's diagnostics, whatever way a call is cut into launches.  Sizes are
the smallest of each dimension, one block and its neighbours by one quad,
ragged last blocks, several launch blocks per resident block, and the largest
that stay resident.  The steps themselves are compared with the oracle in the
parity tests, through the same default path.
"""
import numpy as np
import pytest

from paper_0712_0813_amd import ce
from paper_0712_0813_amd.workloads import DEFAULT_KAPPA

pytestmark = pytest.mark.gpu

POLY = ((0.25, (4, 0, 0)), (20.0, (2, 2, 0)), (0.02, (6, 0, 0)), (0.1, (0, 2, 0)))
T3, S2 = ce.CE_KERNEL_TILED3D, ce.CE_KERNEL_STREAM2D
# dims, N, fields, launch (None: the library's)
SIZES = [
    (1, 4, 1, None), (1, 64, 3, None), (1, 1024, 2, None), (1, 1028, 2, None), (1, 5000, 1, None), (1, 65536, 2, None),
    (2, 4, 2, None), (2, 32, 2, None), (2, 36, 3, None), (2, 300, 3, None), (2, 500, 2, None), (2, 864, 1, None), (2, 1000, 1, None),
    (3, 4, 1, None), (3, 8, 2, None), (3, 16, 2, None), (3, 20, 3, None), (3, 32, 2, None), (3, 48, 2, None),
    # units: one and several per row, one wave of four at work, 1 to 16 rows
    (2, 256, 2, (S2, 4, 64, 256, 1, 0)), (2, 256, 3, (S2, 4, 64, 256, 8, 0)), (2, 256, 1, (S2, 4, 64, 256, 16, 4)),
    (2, 512, 2, (S2, 4, 64, 256, 2, 0)), (2, 768, 2, (S2, 4, 64, 256, 4, 0)), (2, 1024, 1, (S2, 4, 64, 256, 16, 0)),
    (2, 1024, 2, (S2, 4, 64, 256, 4, 0)),
    # tiles: whole rows and columns, several tiles per direction, 1 to 8 planes
    (3, 32, 2, (T3, 4, 8, 256, 1, 0)), (3, 32, 3, (T3, 4, 8, 256, 4, 8)), (3, 64, 2, (T3, 4, 16, 256, 1, 0)),
    (3, 64, 3, (T3, 4, 16, 256, 2, 0)), (3, 64, 1, (T3, 4, 8, 256, 8, 7)), (3, 64, 2, (T3, 4, 8, 256, 4, 0)),
    (3, 96, 2, (T3, 4, 8, 256, 8, 0)), (3, 128, 2, (T3, 4, 16, 256, 8, 0)), (3, 128, 1, (T3, 4, 8, 256, 8, 0)),
    # two blocks of the direct launch as one; ragged tiles
    (3, 68, 2, None), (3, 80, 1, None), (3, 84, 3, None), (3, 92, 2, None), (3, 124, 1, None),
    (3, 60, 1, None), (3, 100, 2, None),
]


def _run(dims, N, nf, launch, precision, poly, plain, calls):
    rng = np.random.default_rng(N * 10 + dims)
    shape = (nf,) + (N,) * dims
    phi = 1e-3 * rng.standard_normal(shape)
    phi[0] += 1.0
    phid = 1e-3 * rng.standard_normal(shape)
    kw = dict(lam=0.0, terms=[(c, e[:nf] + (0,) * (3 - nf)) for c, e in POLY]) if poly else \
        dict(G=(0.0, 100.0, 30.0)[:nf], mu2=(0.1, 0.0, 0.0), expansion=True, kappa=DEFAULT_KAPPA)
    with ce.Simulation(dims, N, nf, N * 0.15, 0.01, precision=precision, **kw) as s:
        if launch is not None:
            s.set_launch(*launch)
        if plain:
            s.set_step_block(0)
        s.load(phi, phid)
        for n in calls:
            s.step(n)
        f, fd = s.read()
        log = [e.as_dict(nf) for e in s.energy_log(sum(calls) + 1)]
    return f, fd, log


@pytest.mark.parametrize("model", ["quartic", "poly"])
@pytest.mark.parametrize("precision", [ce.CE_FP32, ce.CE_FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "d%d_n%d_f%d%s" % (s[:3] + ("" if s[3] is None else "_z%d" % s[3][4],)))
def test_resident_steps_are_the_plain_steps_bitwise(size, precision, model):
    args = size + (precision, model == "poly")
    f0, fd0, log0 = _run(*args, plain=True, calls=(17,))
    f, fd, log = _run(*args, plain=False, calls=(5, 1, 4, 7))
    assert np.array_equal(f, f0) and np.array_equal(fd, fd0)
    assert log == log0


def test_long_calls_are_cut_into_several_launches():
    # more steps than one resident launch takes, and an odd remainder
    args = (3, 16, 2, None, ce.CE_FP32, False)
    f0, fd0, log0 = _run(*args, plain=True, calls=(521,))
    f, fd, log = _run(*args, plain=False, calls=(521,))
    assert np.array_equal(f, f0) and np.array_equal(fd, fd0)
    assert log == log0
