"""Two-step passes of grids with more probes than a pass records itself (2048) against the split pass, bit for bit:
single values, lines of fewer and more terms than a wave's 64 and a block's 256 threads, loops; either side of the line;
FP32 and FP64, Debye media, and the same grid in a batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, NY, NZ, N = 300, 14, 13, 7


def _grid(fd, count, precision, npml, debye):
    rng = np.random.default_rng(count)
    g = fd.Grid(NX, NY, NZ, 0.5, max_steps=N, precision=precision, npml=npml)
    if debye:
        cm = np.zeros(g.shape, np.uint8)
        cm[: NZ // 2] = 1
        g.set_materials(cm, [(1, 0, 1), (9, 0.01, 1)])
        g.set_debye([1e-9, 2e-8, 3e-7], [[0, 0, 0], [4, 5, 6]])
    g.add_source(2, 40, 6, 6, rng.standard_normal(N))
    g.add_source(0, 200, 7, 5, rng.standard_normal(N))
    ids = []
    for q in range(count):
        j, k = int(rng.integers(1, NY - 1)), int(rng.integers(1, NZ - 1))
        if q % 50 == 0:
            ids.append(g.add_probe(1, 0, 1, j, k, (298, 257, 256, 65, 64, 63)[q // 50 % 6]))
        elif q % 50 == 1:
            ids.append(g.add_probe(2, q % 3, int(rng.integers(2, NX - 2)), j, k))
        else:
            ids.append(g.add_probe(0, q % 3, int(rng.integers(1, NX - 1)), j, k))
    return g, ids


@pytest.mark.parametrize("count,precision,npml,debye", [
    (2048, 32, 2, False), (2049, 32, 2, False), (2049, 32, 0, False), (2049, 64, 2, False), (2049, 32, 2, True)])
def test_many_probes(count, precision, npml, debye):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    out = []
    for variant, ty in ((fdtd.KERNEL_SPLIT, 0), (fdtd.KERNEL_TB2, 0), (fdtd.KERNEL_TB2, 4), (fdtd.KERNEL_TB2, 12)):
        if debye and ty:
            continue
        g, ids = _grid(fdtd, count, precision, npml, debye)
        g.set_kernel(variant, ty, 0)
        g.step(4)
        g.step(3)
        out.append(np.stack([g.probe(i) for i in ids]))
        g.close()
    if not debye:
        g, ids = _grid(fdtd, count, precision, npml, False)
        b = fdtd.Batch([g], tile=(60, 8, 16))
        b.run(N)
        out.append(np.stack([b.probe(0, i) for i in ids]))
    assert np.abs(out[0]).max() > 0
    for o in out[1:]:
        assert np.array_equal(out[0], o)
