"""Which lattices step in resident launches and with which default tiling, where
plain launches or another tiling are measured to be faster; from the host code
on a stand-in for the HIP runtime."""
import pytest

import _hoststub

POLY = "dict(lam=0.0, terms=[(0.25, (4, 0, 0)), (20.0, (2, 2, 0))])"
QUARTIC = "dict(G=(0.0, 1.0, 1.0))"


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _hoststub.build(tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("dims,N,nf,fp64,model,resident,planes", [
    # three FP64 fields: few blocks of whole planes only, units below four rows
    (3, 8, 3, True, QUARTIC, True, 0), (3, 12, 3, True, QUARTIC, False, 0), (3, 16, 3, True, POLY, True, 0),
    (3, 32, 3, True, QUARTIC, False, 0), (3, 48, 3, True, POLY, False, 0), (3, 48, 2, True, QUARTIC, True, 0),
    (2, 512, 3, True, QUARTIC, True, 1), (2, 768, 3, True, QUARTIC, False, 4), (2, 768, 2, True, POLY, True, 4),
    # the polynomial model: three FP32 fields in units of eight, units of sixteen
    (2, 1024, 3, False, POLY, True, 4), (2, 1280, 3, False, POLY, False, 8), (2, 1280, 3, False, QUARTIC, True, 8),
    (2, 1536, 2, False, POLY, False, 8), (2, 1536, 2, False, QUARTIC, True, 16), (2, 2048, 2, False, POLY, True, 16),
    # planes of an FP64 tile
    (3, 64, 1, True, QUARTIC, True, 2), (3, 64, 2, True, QUARTIC, True, 2), (3, 64, 2, True, POLY, True, 1),
    (3, 64, 3, True, QUARTIC, True, 1), (3, 64, 2, False, QUARTIC, True, 1)])
def test_resident_launches_and_default_tilings(lib, dims, N, nf, fp64, model, resident, planes):
    _hoststub.run(lib, f"""
        import numpy as np
        phi = np.zeros(({nf},) + ({N},) * {dims})
        with ce.Simulation({dims}, {N}, {nf}, 0.15 * {N}, 0.01, precision={int(fp64)}, **{model}) as s:
            assert s.get_launch().planes == {planes}, s.get_launch().as_tuple()
            s.load(phi, phi)
            s.set_step_block(1000)
            lib.stub_reset()
            s.step(40)
            one = 1 if {dims} == 3 and {N} == 8 else 0    # a single block: an ordinary launch
            assert (calls(COOP), calls(KERNEL)) == ((1 - one, one) if {resident} else (0, 40)), (calls(COOP), calls(KERNEL))
    """)


@pytest.mark.parametrize("dims,N,nf,members,model,resident", [
    # 64 groups a 1024^2 member, 32 tiles a 64^3 one: four and eight at once
    (2, 1024, 2, 4, POLY, True), (2, 1024, 2, 5, POLY, False), (2, 1024, 2, 16, QUARTIC, True), (2, 512, 3, 8, POLY, True),
    (3, 64, 2, 8, POLY, True), (3, 64, 2, 9, POLY, False), (3, 64, 2, 64, QUARTIC, True)])
def test_resident_class_of_a_pool(lib, dims, N, nf, members, model, resident):
    _hoststub.run(lib, f"""
        import numpy as np
        phi = np.zeros(({nf},) + ({N},) * {dims})
        with ce.Pool(8 << 30) as pool:
            for _ in range({members}):
                pool.admit(params({dims}, {N}, {nf}, **{model}), phi, phi, 100)
            lib.stub_reset()
            pool.run_block(10)
            assert (calls(COOP), calls(KERNEL)) == ((1, 0) if {resident} else (0, 10)), (calls(COOP), calls(KERNEL))
    """)
