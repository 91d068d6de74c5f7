"""The tuner times runs of any length, longer than a step block too; from the
host code on a stand-in for the HIP runtime."""
import pytest

import _hoststub


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _hoststub.build(tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("steps,warmup,final", [(8, 3, 40), (5000, 3, 40), (8, 4096, 9001), (1, 0, 1)])
def test_tuner_takes_any_number_of_steps(lib, tmp_path, steps, warmup, final):
    _hoststub.run(lib, f"""
        from paper_0712_0813_amd import autotune
        autotune._ARCH = "gfx950"
        autotune.gpu_arch = lambda: "gfx950"
        autotune.candidates = lambda dims, N: [(ce.CE_KERNEL_DIRECT, 0, 0, 0, 0, g) for g in (0, 7)]
        taken = []
        step, time_steps = ce.Simulation.step, ce.Simulation.time_steps
        ce.Simulation.step = lambda s, n: (taken.append(n), step(s, n))
        ce.Simulation.time_steps = lambda s, n: (taken.append(n), time_steps(s, n))[1]
        e = autotune.tune(3, 16, 1, steps={steps}, warmup={warmup}, final_steps={final},
                          cache_path={str(tmp_path / "c.json")!r})
        assert e["screened"] == 2 and e["finalists"] == 2
        assert sum(taken) == 2 * ({warmup} + {steps}) + 2 * ({warmup} + 2 * {final})
        assert calls("hipGraphInstantiate") == 0
    """)
