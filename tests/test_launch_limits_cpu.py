"""Cooperative launches that are refused, and how long one may last; from the
host code on a stand-in for the HIP runtime."""
import pytest

import _hoststub


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _hoststub.build(tmp_path_factory.mktemp("stub"))


def test_refused_launches_become_plain_ones(lib):
    _hoststub.run(lib, """
        with sim(3, 64, 2) as s:
            s.set_step_block(1000)
            s.step(10)
            lib.stub_reset()
            lib.stub_fail(COOP.encode(), 1)
            s.step(300)
            assert (calls(COOP), calls(KERNEL)) == (1, 300) and s.step_count == 310
            s.step(100)
            assert (calls(COOP), calls(KERNEL)) == (1, 400)
            s.set_launch(*s.get_launch().as_tuple())      # planned again
            s.step(100)
            assert (calls(COOP), calls(KERNEL)) == (2, 400)
        with ce.Pool(8 << 30) as pool:
            j = [pool.admit_generated(params(3, 64, 2), SPEC, 1000) for _ in range(8)]
            pool.run_block(10)
            lib.stub_reset()
            lib.stub_fail(COOP.encode(), 1)
            pool.run_block(20)
            assert (calls(COOP), calls(KERNEL)) == (1, 20) and pool.steps_left(j[0]) == 970
            pool.run_block(20)
            assert calls(COOP) == 1
    """)


@pytest.mark.parametrize("members,k,launches", [(8, 50, 1), (8, 4096, 16), (64, 256, 1), (256, 50, 1), (256, 300, 5)])
def test_a_pool_launch_lasts_some_milliseconds(lib, members, k, launches):
    # 2048 steps of a tile, 256 steps: eight 64^3 members are worked at once
    _hoststub.run(lib, f"""
        with ce.Pool(64 << 30) as pool:
            for _ in range({members}):
                j = pool.admit_generated(params(3, 64, 2), SPEC, 10000)
            lib.stub_reset()
            pool.run_block({k})
            assert (calls(COOP), calls(KERNEL)) == ({launches}, 0), (calls(COOP), calls(KERNEL))
            assert pool.steps_left(j) == 10000 - {k}
    """)


def test_batched_classes_are_replayed_beside_resident_ones(lib):
    # 8 x 64^3 stays on the chip for a block; two lines and a 48^3 cube are
    # batched, as a graph from the composition's second block on
    _hoststub.run(lib, """
        with ce.Pool(8 << 30) as pool:
            for _ in range(8):
                j = pool.admit_generated(params(3, 64, 2), SPEC, 10000)
            for p in (params(1, 1024, 1), params(1, 1024, 2)):
                pool.admit_generated(p, SPEC, 10000)
            lib.stub_reset()
            pool.run_block(16)
            assert (calls(COOP), calls(KERNEL), calls("hipGraphLaunch")) == (1, 32, 0)
            for n in range(2, 5):
                pool.run_block(16)
                assert (calls(COOP), calls(KERNEL), calls("hipGraphLaunch")) == (n, 64, n - 1)
            assert calls("hipGraphInstantiate") == 1
            pool.run_block(4)    # too few launches for a graph beside others
            assert (calls(COOP), calls(KERNEL), calls("hipGraphLaunch")) == (5, 72, 3)
            assert pool.steps_left(j) == 10000 - 68
    """)
