"""Device memory kept from destroyed simulations: kept only once the device is
idle, taken by the next of its size, bounded, and given back on request; from
the host code on a stand-in for the HIP runtime."""
import pytest

import _hoststub


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _hoststub.build(tmp_path_factory.mktemp("stub"))


def test_kept_memory(lib):
    _hoststub.run(lib, """
        def once(N):
            with sim(3, N, 1) as s:
                s.step(2)
        once(32)
        lib.stub_reset()
        once(32)
        assert (calls("hipMalloc"), calls("hipFree")) == (0, 0)
        assert calls("hipDeviceSynchronize") == 1
        # not idle: not kept
        lib.stub_fail(b"hipDeviceSynchronize", 1)
        once(32)
        assert calls("hipFree") == 1
        once(32)
        assert calls("hipMalloc") == 1
        # eight blocks at most
        for N in range(16, 56, 4):
            with ce.Simulation(3, N, 1, 0.15 * N, 0.01) as s:
                pass
        lib.stub_reset()
        ce.ce_release_memory()
        assert calls("hipFree") == 8
        ce.ce_release_memory()
        assert calls("hipFree") == 8
        once(32)
        assert calls("hipMalloc") == 1
    """)
