"""The launch the server gives its members: the tuner's where it is tall enough."""
import pytest

from paper_0712_0813_amd import autotune, ce, serve
from paper_0712_0813_amd.workloads import ensemble_512x64

T3, S2 = ce.CE_KERNEL_TILED3D, ce.CE_KERNEL_STREAM2D


@pytest.mark.parametrize("dims,N,cached,want", [
    (3, 64, None, (T3, 4, 16, 256, 64, 4)),
    (3, 64, (T3, 4, 16, 256, 8, 32), (T3, 4, 16, 256, 64, 4)),        # finer: not beside other threads
    (3, 64, (T3, 4, 8, 256, 64, 4), (T3, 4, 8, 256, 64, 4)),          # as tall, another shape
    (3, 256, (T3, 4, 64, 512, 128, 64), (T3, 4, 64, 512, 128, 64)),
    (3, 64, (ce.CE_KERNEL_DIRECT, 0, 0, 0, 0, 256), (T3, 4, 16, 256, 64, 4)),
    (2, 1024, (S2, 4, 64, 256, 16, 64), (S2, 4, 64, 256, 64, 16)),
    (2, 1024, (S2, 4, 64, 256, 64, 16), (S2, 4, 64, 256, 64, 16)),
    (3, 96, (T3, 4, 8, 256, 8, 108), None), (1, 256, None, None)])
def test_tuned_member_launch(monkeypatch, dims, N, cached, want):
    monkeypatch.setattr(autotune, "lookup", lambda *a, **k: cached)
    lat = ensemble_512x64(count=1, steps=1)[0].with_(dims=dims, N=N)
    assert serve.tuned_member_launch(lat) == want
