"""Members of a pool that a second thread admits to run in tall blocks, each
working several tiles or groups of units in turn: bitwise the lone runs with one
block for each, as in a pool of one thread."""
import threading

import numpy as np
import pytest

from paper_0712_0813_amd import ce
from paper_0712_0813_amd.workloads import DEFAULT_KAPPA

pytestmark = pytest.mark.gpu

POLY = ((0.25, (4, 0, 0)), (20.0, (2, 2, 0)), (0.02, (6, 0, 0)))
# dims, N, fields, precision, polynomial model: columns of 1 to 16 tiles, two
# columns a lattice and many, groups that are a multiple of eight and not, units
# of one row and of several a segment
MEMBERS = [(3, 32, 2, 0, False), (3, 64, 2, 0, True), (3, 64, 3, 0, False), (3, 96, 1, 0, False), (3, 128, 2, 0, False),
           (2, 256, 2, 0, False), (2, 512, 1, 0, True), (2, 768, 2, 0, False), (2, 1024, 3, 0, False),
           (2, 512, 2, 1, False), (3, 64, 2, 1, False), (3, 100, 1, 0, False)]


def _params(dims, N, nf, precision, poly):
    kw = dict(lam=0.0, terms=[(c, e) for c, e in POLY if not any(e[nf:])]) if poly else \
        dict(G=(0.0, 100.0, 30.0)[:nf], expansion=True, kappa=DEFAULT_KAPPA)
    return ce.make_params(dims, N, nf, N * 0.15, 0.01, precision=precision, **kw), kw


def _fields(dims, N, nf):
    rng = np.random.default_rng(N * 10 + dims)
    phi = 1e-3 * rng.standard_normal((nf,) + (N,) * dims)
    phi[0] += 1.0
    return phi, 1e-3 * rng.standard_normal(phi.shape)


@pytest.mark.parametrize("member", MEMBERS, ids=lambda m: "d%d_n%d_f%d_p%d%s" % (m[:4] + ("_poly" if m[4] else "",)))
def test_members_in_tall_blocks_are_lone_runs_bitwise(member):
    dims, N, nf, precision, poly = member
    p, kw = _params(*member)
    phi, phid = _fields(dims, N, nf)
    steps, ids = (9, 14), []
    with ce.Pool(8 << 30) as pool:
        th = threading.Thread(target=lambda: ids.extend(pool.admit(p, phi, phid, n) for n in steps))
        th.start()
        th.join()
        assert len(ids) == len(steps)
        while pool.info().active > 0:
            pool.run_block(5)
        got = [pool.poll(j)[1].as_dict(nf) for j in ids], [pool.retire(j) for j in ids]
    for n, e, (f, fd) in zip(steps, *got):
        with ce.Simulation(dims, N, nf, N * 0.15, 0.01, precision=precision, **kw) as s:
            s.set_launch(*ce.ce_pool_launch_for(p).as_tuple())
            s.set_step_block(0)
            s.load(phi, phid)
            s.step(n)
            g, gd = s.read()
            assert np.array_equal(f, g) and np.array_equal(fd, gd)
            assert e == s.energies().as_dict(nf)
