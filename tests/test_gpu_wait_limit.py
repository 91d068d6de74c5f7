"""Launches that keep a lattice on the chip and find no room to start (wait
limit 0: they never do) leave the state as it was: every way of asking for the
simulation then gives bitwise what plain launches give, whatever was queued
behind the launch, and a pool's members likewise."""
import numpy as np
import pytest

from paper_0712_0813_amd import ce
from paper_0712_0813_amd.workloads import DEFAULT_KAPPA

pytestmark = pytest.mark.gpu

T3, S2 = ce.CE_KERNEL_TILED3D, ce.CE_KERNEL_STREAM2D
CALLS = (7, 1, 2, 40, 1)
# dims, N, fields, launch (None: the library's): direct (with threads that have
# no site; several launch blocks as one), tiles (fewer blocks than tiles; blocks
# without a tile), ragged tiles, units (waves without a unit), a single block
SIZES = [(1, 1028, 1, None), (2, 300, 2, None), (3, 32, 2, None), (3, 80, 1, None), (3, 64, 2, None),
         (3, 64, 1, (T3, 4, 8, 256, 8, 7)), (3, 32, 2, (T3, 4, 8, 256, 4, 64)), (3, 100, 1, None),
         (2, 256, 2, (S2, 4, 64, 256, 8, 0)), (2, 768, 1, (S2, 4, 64, 256, 16, 0)), (1, 64, 2, None)]


def _kw(nf, precision):
    return dict(G=(0.0, 100.0, 30.0)[:nf], expansion=True, kappa=DEFAULT_KAPPA, precision=precision)


def _fields(dims, N, nf):
    rng = np.random.default_rng(N * 10 + dims)
    phi = 1e-3 * rng.standard_normal((nf,) + (N,) * dims)
    phi[0] += 1.0
    return phi, 1e-3 * rng.standard_normal(phi.shape)


def _sim(dims, N, nf, launch, precision):
    s = ce.Simulation(dims, N, nf, N * 0.15, 0.01, **_kw(nf, precision))
    if launch is not None:
        s.set_launch(*launch)
    return s


def _ask(s, how, nf):
    if how == "read":
        return s.read()
    if how == "sites":
        return s.read_sites(nf - 1, np.arange(5, dtype=np.int64))
    if how == "spectrum":
        return s.spectrum(0)
    if how == "image":
        return (np.array(s.save_image()),)
    if how == "log":
        return (np.array([list(e.as_dict(nf)["mean"]) for e in s.energy_log(9)]),)
    if how == "sync":
        s.sync()
    if how == "time":
        s.time_steps(6)
    return s.read()


@pytest.mark.parametrize("precision", [ce.CE_FP32, ce.CE_FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "d%d_n%d_f%d%s" % (s[:3] + ("" if s[3] is None else "_z%d" % s[3][4],)))
def test_launch_without_room_changes_no_result(size, precision):
    dims, N, nf, launch = size
    phi, phid = _fields(dims, N, nf)
    got = []
    for plain in (True, False):
        with _sim(dims, N, nf, launch, precision) as s:
            if plain:
                s.set_step_block(0)
            else:
                s.set_wait_limit(0.0)
            s.load(phi, phid)
            for n in CALLS:
                s.step(n)
            f, fd = s.read()
            for n in CALLS:   # plain launches by now
                s.step(n)
            log = [e.as_dict(nf) for e in s.energy_log(2 * sum(CALLS) + 1)]
            s.set_launch(*s.get_launch().as_tuple())   # the waiting launches again
            s.set_wait_limit(200.0)
            s.step(21)
            got.append((f, fd, log) + s.read() + (s.energies().as_dict(nf),))
    for a, b in zip(*got):
        assert np.array_equal(a, b) if isinstance(a, np.ndarray) else a == b


@pytest.mark.parametrize("how", ["read", "sites", "spectrum", "image", "log", "sync", "time", "restored"])
def test_every_way_of_asking_takes_the_missing_steps(how):
    phi, phid = _fields(3, 32, 2)
    got = []
    for plain in (True, False):
        with _sim(3, 32, 2, None, ce.CE_FP32) as s:
            s.load(phi, phid)
            image = s.save_image()
            s.set_step_block(0 if plain else 32)
            if not plain:
                s.set_wait_limit(0.0)
            s.step(13)
            if how == "restored":   # what was halted is replaced
                s.restore_image(image)
                s.step(3)
            got.append(_ask(s, how, 2))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_pool_without_room_changes_no_result():
    mix = [(3, 64, 2, 31), (3, 64, 2, 50), (3, 64, 2, 50), (2, 256, 1, 44), (2, 256, 1, 50), (1, 256, 2, 40)]
    with ce.Pool(8 << 30) as pool:
        pool.set_wait_limit(0.0)
        ids = []
        for dims, N, nf, steps in mix:
            phi, phid = _fields(dims, N, nf)
            ids.append(pool.admit(ce.make_params(dims, N, nf, N * 0.15, 0.01, **_kw(nf, ce.CE_FP32)), phi, phid, steps))
        pool.set_quota(ids[1], 3)
        pool.set_quota(ids[2], 0)
        pool.run_block(10)
        pool.run_block(10)
        mid = pool.poll(ids[1])[1]
        assert mid.step == 6
        pool.set_quota(ids[1], -1)
        pool.set_quota(ids[2], -1)
        while pool.info().active > 0:
            pool.run_block(10)
        res = []
        for j, (_, _, nf, steps) in zip(ids, mix):
            done, e = pool.poll(j)
            assert done and e.step == steps
            res.append(pool.retire(j) + (e.as_dict(nf),))
    for (dims, N, nf, steps), r in zip(mix, res):
        p = ce.make_params(dims, N, nf, N * 0.15, 0.01, **_kw(nf, ce.CE_FP32))
        with _sim(dims, N, nf, ce.ce_pool_launch_for(p).as_tuple(), ce.CE_FP32) as s:
            s.set_step_block(0)
            s.load(*_fields(dims, N, nf))
            s.step(steps)
            assert all(np.array_equal(a, b) for a, b in zip(s.read(), r))
            assert s.energies().as_dict(nf) == r[2]
