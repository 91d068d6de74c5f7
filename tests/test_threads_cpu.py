"""Which launches the library takes when several threads use it, from its host
code on a stand-in for the HIP runtime."""
import pytest

import _hoststub


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _hoststub.build(tmp_path_factory.mktemp("stub"))


def test_lone_run_is_cooperative_only_while_no_other_thread_is_in_the_library(lib):
    _hoststub.run(lib, """
        with sim(3, 64, 2) as a, sim(3, 64, 2) as b:
            a.set_step_block(1000), b.set_step_block(1000)   # no graphs: launches can be counted
            lib.stub_reset()
            a.step(100)
            assert calls(COOP) == 1 and calls(KERNEL) == 0
            lib.stub_hold(b"hipStreamSynchronize")
            th = threading.Thread(target=b.sync)
            th.start()
            lib.stub_wait_held(1)
            lib.stub_reset()
            a.step(100)
            assert calls(COOP) == 0 and calls(KERNEL) == 100
            lib.stub_release(b"hipStreamSynchronize")
            th.join()
            a.step(100)
            assert calls(COOP) == 1 and calls(KERNEL) == 100
            # many threads at once: no call of another beside a cooperative launch
            def work(s):
                for _ in range(20):
                    s.step(10)
                    s.sync()
            ts = [threading.Thread(target=work, args=(s,)) for s in (a, b)]
            for t in ts: t.start()
            for t in ts: t.join()
            assert lib.stub_beside_cooperative() == 0
    """)


def test_pool_block_is_cooperative_only_while_no_other_thread_is_in_the_library(lib):
    _hoststub.run(lib, """
        with ce.Pool(8 << 30) as pool, sim(3, 32, 1) as other:
            for _ in range(8):
                pool.admit_generated(params(3, 64, 2), SPEC, 1000)
            lib.stub_reset()
            pool.run_block(10)
            assert calls(COOP) == 1 and calls(KERNEL) == 0
            lib.stub_hold(b"hipMemcpy")
            th = threading.Thread(target=lambda: other.energies(allow_nonfinite=True))
            th.start()
            lib.stub_wait_held(1)
            lib.stub_reset()
            pool.run_block(10)
            assert calls(COOP) == 0 and calls(KERNEL) + calls("hipGraphLaunch") > 0
            lib.stub_release(b"hipMemcpy")
            th.join()
            lib.stub_reset()
            pool.run_block(10)
            assert calls(COOP) == 1
    """)


def test_second_thread_of_a_pool_waits_for_the_resident_block_in_flight(lib):
    _hoststub.run(lib, """
        with ce.Pool(8 << 30) as pool:
            for _ in range(8):
                pool.admit_generated(params(3, 64, 2), SPEC, 1000)
            pool.run_block(10)
            assert calls(COOP) == 1
            lib.stub_hold(b"hipEventSynchronize")    # the block runs
            done = []
            th = threading.Thread(target=lambda: done.append(pool.admit_generated(params(3, 64, 2), SPEC, 1000)))
            allocs = calls("hipMalloc")
            th.start()
            lib.stub_wait_held(1)
            assert not done and calls("hipMalloc") == allocs
            lib.stub_release(b"hipEventSynchronize")
            th.join()
            assert done
            lib.stub_reset()
            for _ in range(3):
                pool.run_block(10)
            assert calls(COOP) == 0
    """)


@pytest.mark.parametrize("dims,N,nf,blocks", [
    # blocks of a member: columns of up to 64 planes, units of up to 64 rows
    # (two blocks at least); smaller tilings keep what they have.  A launch of
    # more than eight is cut to a multiple of eight.
    (3, 64, 2, 4), (3, 64, 3, 4), (3, 32, 2, 1), (3, 128, 1, 32), (3, 96, 2, 16), (2, 256, 2, 2), (2, 512, 1, 4),
    (2, 1024, 2, 16), (3, 48, 2, 104), (1, 1024, 1, 1)])
def test_members_of_a_shared_pool_get_tall_blocks(lib, dims, N, nf, blocks):
    _hoststub.run(lib, f"""
        import numpy as np
        phi = np.zeros(({nf},) + ({N},) * {dims})
        with ce.Pool(8 << 30) as pool:
            th = threading.Thread(target=lambda: pool.admit(params({dims}, {N}, {nf}), phi, phi, 1000))
            th.start()
            th.join()
            lib.stub_reset()
            pool.run_block(1)
            assert calls(COOP) == 0 and calls(KERNEL) == 1
            assert lib.stub_blocks() == {blocks}, lib.stub_blocks()
    """)
