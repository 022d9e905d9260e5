"""Two-step passes over columns with many sources (keys read 64 at a time) against the split pass, bit for bit: fewer
and more sources in a row of columns than one read takes, several at one node (they add in their order), FP32 and FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("count", [4, 5, 63, 64, 65, 200])
def test_many_sources(count, precision):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    nx, ny, nz, n = 70, 14, 13, 10
    out = []
    for variant in (fdtd.KERNEL_SPLIT, fdtd.KERNEL_TB2):
        rng = np.random.default_rng(count)
        g = fdtd.Grid(nx, ny, nz, 0.5, max_steps=n, precision=precision, npml=2)
        for q in range(count):
            i, j, k = (4, 5, 6) if q % 9 == 0 else (int(rng.integers(3, 66)), 5, int(rng.integers(3, 10)))
            g.add_source(int(rng.integers(0, 3)), i, j, k, rng.standard_normal(n))
        pid = g.add_probe(0, 2, 4, 5, 6)
        g.set_kernel(variant, 0, 0)
        g.step(n)
        out.append([g.get_field(c) for c in range(6)] + [g.probe(pid)])
    assert np.abs(out[0][-1]).max() > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)
