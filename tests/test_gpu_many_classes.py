"""Two-step passes of grids with more than 256 coefficient classes: against the split pass, bit for bit, on either side of
what the tiles' tables in LDS hold (768 and 2,048 classes), alone and in a batch; and the time against the split pass where
they are the default (0.7 of its time with 1,300 classes on 203 x 157 x 131, 0.93 to 0.97 with 17,000; with the tables in
memory 1.45 and 1.8).  Bounds lie between."""
import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu

DIMS, N = (125, 29, 23), 7


def _grid(fd, classes, npml, precision):
    """Every lumped resistor of a value of its own is a class more."""
    def make(extra):
        sc = S.random_case(*DIMS, npml, seed=classes, nsteps=N, n_mats=3)
        sc.cell_mat[:] = 0
        sc.cell_mat[:9] = 1
        sc.wires = []
        taken = {s[1:4] for s in sc.sources}
        nodes = [(i, j, k) for k in range(2, DIMS[2] - 2) for j in range(2, DIMS[1] - 2) for i in range(2, DIMS[0] - 2)]
        nodes = [n for n in nodes if n not in taken]
        rng = np.random.default_rng(1)
        sc.lumped = [(0, q % 3, *nodes[p], 50.0 + q) for q, p in enumerate(rng.permutation(len(nodes))[:extra])]
        g = fd.Grid.from_params(sc.params(), precision=precision)
        ids = S.apply(sc, g)
        g.finalize()
        return g, ids
    g, ids = make(0)
    g, ids = make(classes - g.num_classes)
    assert g.num_classes == classes
    return g, ids


def _out(g, ids):
    return [g.get_field(c) for c in range(6)] + [g.probe(i) for i in ids]


@pytest.mark.parametrize("classes,npml,precision", [
    (257, 0, 32), (768, 0, 32), (769, 0, 32), (2048, 0, 32), (2049, 0, 32), (257, 5, 32), (2048, 5, 32), (2049, 5, 32),
    (257, 0, 64), (2049, 5, 64)])
def test_many_classes(classes, npml, precision):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    g, ids = _grid(fdtd, classes, npml, precision)
    g.set_kernel(fdtd.KERNEL_SPLIT, 0, 0)
    g.step(N)
    ref = _out(g, ids)
    assert max(np.abs(r).max() for r in ref) > 0
    for ty, tz in ((0, 0), (4, 5), (8, 1), (8, 23), (12, 7)):
        g, ids = _grid(fdtd, classes, npml, precision)
        g.set_kernel(fdtd.KERNEL_TB2, ty, tz)
        g.step(4)
        g.step(3)
        for a, b in zip(ref, _out(g, ids)):
            assert np.array_equal(a, b), (ty, tz)
    pairs = [_grid(fdtd, c, npml, precision) for c in (classes, 257)]
    b = fdtd.Batch([p[0] for p in pairs], tile=(60, 8, 32))
    b.run(N)
    out = [pairs[0][0].get_field(c) for c in range(6)] + [b.probe(0, i) for i in pairs[0][1]]
    for a, o in zip(ref, out):
        assert np.array_equal(a, o)


@pytest.mark.parametrize("mu,bound", [(0.0, 0.9), (0.1, 1.2)])
def test_default_pass_with_many_classes(mu, bound):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    sc = S.config2(203, 157, 131, npml=8, wire_cells=8, n_steps=800, e_probe_offsets=(4,))
    sc.cell_mat[:] = np.random.default_rng(1).integers(0, 4, size=sc.cell_mat.shape).astype(np.uint8)
    sc.materials = [(1.0 + 0.1 * q, 1e-3, 1.0 + mu * q) for q in range(4)]
    g = fdtd.Grid.from_params(sc.params(), precision=32)
    S.apply(sc, g)

    def us(variant):
        g.set_kernel(variant, 0, 0)
        g.step(20)
        best = float("inf")
        for _ in range(4):
            g.timing(True)
            g.kernel_time()
            g.step(60)
            ms, n = g.kernel_time()
            g.timing(False)
            best = min(best, 1e3 * ms / n)
        return best

    split, auto = us(fdtd.KERNEL_SPLIT), us(fdtd.KERNEL_AUTO)
    print(f"{g.num_classes} classes: split {split:.1f}, default {auto:.1f} us a step", flush=True)
    assert auto < bound * split
