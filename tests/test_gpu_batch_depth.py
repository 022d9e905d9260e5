"""Two-step passes of batches against the same grids alone, bit for bit, where the tiles' depth is not what was asked
for: few grids (chunks shallower than tile_z), tile_z past the 64 planes that the depth model looks at, grids of a few
planes, and tile lists shorter than, equal to and longer than a round of an XCD's runs (8 x 17 tiles)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIMS = [(61, 19, 70), (60, 8, 5), (33, 40, 129), (121, 9, 66), (20, 57, 64)]


def _grid(fd, d, n, precision):
    rng = np.random.default_rng(sum(d))
    g = fd.Grid(*d, 0.5, max_steps=n, npml=2, precision=precision)
    cm = rng.integers(0, 2, size=g.shape).astype(np.uint8)
    g.set_materials(cm, [(1, 0, 1), (7, 0.02, 1)])
    g.add_source(2, d[0] // 2, d[1] // 2, d[2] // 2, rng.standard_normal(n))
    return g, [g.add_probe(0, 2, d[0] // 2 + 1, d[1] // 2, d[2] // 2), g.add_probe(1, 0, 2, 4, 2, d[0] - 5)]


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("count,tile_z", [(1, 16), (1, 4096), (5, 16), (5, 65), (5, 128), (15, 24), (15, 64)])
def test_depth_of_batch_tiles(count, tile_z, precision):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    n = 7
    dims = [DIMS[q % len(DIMS)] for q in range(count)]
    both = [_grid(fdtd, d, n, precision) for d in dims]
    b = fdtd.Batch([g for g, _ in both], tile=(60, 8, tile_z))
    b.run(4)
    b.run(3)
    for q, d in enumerate(dims[:len(DIMS)]):
        g, ids = _grid(fdtd, d, n, precision)
        g.set_kernel(fdtd.KERNEL_SPLIT, 0, 0)
        g.step(n)
        for c in range(6):
            assert np.array_equal(g.get_field(c), both[q][0].get_field(c)), (d, c)
        for i, j in zip(ids, both[q][1]):
            assert np.array_equal(g.probe(i), b.probe(q, j)), d
        assert np.abs(g.probe(ids[0])).max() > 0
        g.close()
