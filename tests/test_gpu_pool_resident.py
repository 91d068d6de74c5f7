"""Pool classes that stay on the chip for a block of steps: more members than are
worked at once, members that end inside a block, wait or are limited, classes
side by side, memory taken over from earlier members and simulations, and lone
runs on streams of their own.  Always bitwise the plain launches' results."""
import threading

import numpy as np
import pytest

from paper_0712_0813_amd import ce
from paper_0712_0813_amd.workloads import DEFAULT_KAPPA

pytestmark = pytest.mark.gpu


def _kw(nf):
    return dict(G=(0.0, 100.0, 30.0)[:nf], expansion=True, kappa=DEFAULT_KAPPA)


def _params(dims, N, nf):
    return ce.make_params(dims, N, nf, N * 0.15, 0.01, **_kw(nf))


def _fields(dims, N, nf, seed):
    rng = np.random.default_rng(1000 * seed + N)
    phi = 1e-3 * rng.standard_normal((nf,) + (N,) * dims)
    phi[0] += 1.0 + 0.01 * seed
    return phi, 1e-3 * rng.standard_normal(phi.shape)


def _plain(dims, N, nf, seed, steps):
    """Plain launches with the member launch; `steps` increasing counts to report at."""
    out, at = {}, 0
    with ce.Simulation(dims, N, nf, N * 0.15, 0.01, **_kw(nf)) as s:
        s.set_launch(*ce.ce_pool_launch_for(_params(dims, N, nf)).as_tuple())
        s.set_step_block(0)
        s.load(*_fields(dims, N, nf, seed))
        for n in sorted(set(steps)):
            s.step(n - at)
            at = n
            out[n] = s.read() + (s.energies().as_dict(nf),)
    return out


def _same(got, want):
    return np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]) and got[2] == want[2]


# dims, N, fields, members: two and a half rounds of eight (or of four, of
# sixteen groups of units); members of a round share their inputs with those of
# the others, so few lone runs check them all
@pytest.mark.parametrize("dims,N,nf,members", [(3, 64, 2, 20), (3, 64, 3, 10), (3, 32, 1, 160), (2, 512, 2, 40),
                                               (2, 512, 3, 20), (2, 1024, 2, 10)])
def test_class_of_more_members_than_are_worked_at_once(dims, N, nf, members):
    kinds = 3
    steps = [9, 23, 30]          # within the first block, the third, at the end of the third
    inputs = [_fields(dims, N, nf, k) for k in range(kinds)]
    p = _params(dims, N, nf)
    with ce.Pool(64 << 30) as pool:
        ids = [pool.admit(p, *inputs[m % kinds], steps[(m // kinds) % 3]) for m in range(members)]
        paused, limited = ids[members // 2], ids[-1]
        pool.set_quota(paused, 0)
        pool.set_quota(limited, 4)
        pool.run_block(10)
        assert pool.resident_classes() == 1
        assert pool.steps_left(paused) == steps[(members // 2 // kinds) % 3]
        pool.run_block(10)
        pool.set_quota(paused, -1)
        pool.set_quota(limited, -1)
        while pool.info().active > 0:
            pool.run_block(10)
        got = []
        for j in ids:
            done, e = pool.poll(j)
            assert done
            got.append(pool.retire(j) + (e.as_dict(nf),))
    want = [_plain(dims, N, nf, k, steps) for k in range(kinds)]
    for m, g in enumerate(got):
        assert _same(g, want[m % kinds][steps[(m // kinds) % 3]]), m


def test_resident_classes_side_by_side_and_members_one_after_the_other():
    # two resident classes and a batched one; retired members' memory is taken
    # over by the next
    mix = [(3, 64, 2, 6), (2, 512, 1, 10), (1, 1024, 2, 2)]
    with ce.Pool(64 << 30) as pool:
        for turn in range(2):
            ids = [(d, N, nf, pool.admit(_params(d, N, nf), *_fields(d, N, nf, turn), 25))
                   for d, N, nf, count in mix for _ in range(count)]
            pool.run_block(16)
            assert pool.resident_classes() == 2
            pool.run_block(16)
            want = {(d, N, nf): _plain(d, N, nf, turn, [25])[25] for d, N, nf, _ in mix}
            for d, N, nf, j in ids:
                e = pool.poll(j)[1].as_dict(nf)
                assert _same(pool.retire(j) + (e,), want[d, N, nf])


def test_no_class_is_resident_once_a_second_thread_has_admitted():
    with ce.Pool(8 << 30) as pool:
        a = pool.admit(_params(3, 64, 2), *_fields(3, 64, 2, 0), 20)
        pool.run_block(10)
        assert pool.resident_classes() == 1
        b = []
        th = threading.Thread(target=lambda: b.append(pool.admit(_params(3, 64, 2), *_fields(3, 64, 2, 1), 20)))
        th.start()
        th.join()
        while pool.info().active > 0:
            pool.run_block(10)
            assert pool.resident_classes() == 0
        for seed, j in ((0, a), (1, b[0])):
            e = pool.poll(j)[1].as_dict(2)
            assert _same(pool.retire(j) + (e,), _plain(3, 64, 2, seed, [20])[20])


def _lone(dims, N, nf, seed, calls, stream=None):
    s = ce.Simulation(dims, N, nf, N * 0.15, 0.01, stream=stream, **_kw(nf))
    s.set_launch(*ce.ce_pool_launch_for(_params(dims, N, nf)).as_tuple())
    s.load(*_fields(dims, N, nf, seed))
    return s


def test_lone_runs_interleaved_on_their_own_streams():
    want = {seed: _plain(3, 64, 2, seed, [60])[60] for seed in (0, 1)}
    sims = [_lone(3, 64, 2, seed, None) for seed in (0, 1)]   # a stream each, made by the library
    try:
        for _ in range(3):
            for s in sims:
                s.step(20)
        for seed, s in enumerate(sims):
            assert _same(s.read() + (s.energies().as_dict(2),), want[seed])
    finally:
        for s in sims:
            s.close()


def test_memory_of_a_destroyed_run_is_as_good_as_new():
    for seed in (0, 1, 0):
        with _lone(3, 64, 2, seed, None) as s:
            s.step(25)
            assert _same(s.read() + (s.energies().as_dict(2),), _plain(3, 64, 2, seed, [25])[25])


def test_steps_captured_from_a_stream_are_plain_launches():
    import torch
    want = _plain(3, 64, 2, 0, [4, 14, 34])
    st = torch.cuda.Stream()
    with _lone(3, 64, 2, 0, None, stream=st.cuda_stream) as s:
        s.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            s.step(4)                    # queued by the replay only
        with torch.cuda.stream(st):
            graph.replay()
        s.sync()
        assert _same(s.read() + (s.energies().as_dict(2),), want[4])
        s.step(10)
        assert _same(s.read() + (s.energies().as_dict(2),), want[14])
        s.step(20)
        assert _same(s.read() + (s.energies().as_dict(2),), want[34])
