"""The one-launch two-step pass against the split pass, bit for bit, at the
sizes where its tiles can go wrong: grids just under, at and past one 60-wide
tile and one row of 4, 8 or 12, chunks of one plane up to the whole height,
grids of two planes, CPML thicknesses that leave tiles clear of some, all or
no slabs, 1- and 2-byte class ids, odd step counts, and steps cut into calls
(the probes of a call's last step are recorded by a launch of their own)."""
import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu

CASES = [  # dims, npml, precision, materials, (tile_y, tile_z) shapes
    ((59, 13, 9), 0, 32, 4, [(0, 0), (4, 1), (8, 3), (12, 9)]),
    ((60, 12, 11), 3, 32, 4, [(0, 0), (4, 2), (8, 1), (12, 5)]),
    ((61, 17, 12), 0, 32, 4, [(0, 0), (4, 5), (8, 12), (12, 1)]),
    ((64, 25, 10), 3, 64, 4, [(0, 0), (4, 3), (8, 10), (12, 2)]),
    ((9, 8, 8), 0, 32, 3, [(0, 0), (8, 2), (12, 1)]),
    ((121, 40, 23), 2, 32, 4, [(0, 0), (4, 7), (8, 6), (12, 23)]),   # tiles clear of every slab
    ((200, 52, 30), 4, 64, 4, [(0, 0), (8, 7)]),
    ((130, 37, 20), 4, 32, 40, [(0, 0), (8, 5), (12, 20)]),          # 2-byte class ids
    ((70, 21, 18), 0, 64, 40, [(0, 0), (8, 4)]),
]


@pytest.fixture(scope="module")
def fd():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    fdtd.lib()
    return fdtd


def _run(fd, sc, precision, variant, ty, tz, chunks):
    g = fd.Grid.from_params(sc.params(), precision=precision)
    ids = S.apply(sc, g)
    g.set_kernel(variant, ty, tz)
    for n in chunks:
        g.step(n)
    return [g.get_field(c) for c in range(6)] + [g.probe(i) for i in ids], g.num_classes


@pytest.mark.parametrize("dims,npml,precision,mats,shapes", CASES,
                         ids=[f"{d[0]}x{d[1]}x{d[2]}p{p}f{q}m{m}" for d, p, q, m, _ in CASES])
def test_two_step_launch_equals_the_split_pass(fd, dims, npml, precision, mats, shapes):
    sc = S.random_case(*dims, npml, seed=31 + dims[0], nsteps=24, n_mats=2 if mats == 40 else mats)
    if mats < 6:   # layers: few classes; cells drawn one by one: thousands
        sc.cell_mat[:] = (np.arange(dims[2]) * mats // dims[2]).astype(np.uint8)[:, None, None]
    ref, ncls = _run(fd, sc, precision, fd.KERNEL_SPLIT, 0, 0, (24,))
    assert (ncls > 256) == (mats == 40)
    assert max(np.abs(r).max() for r in ref) > 0
    for q, (ty, tz) in enumerate(shapes):
        variant = fd.KERNEL_AUTO if ty == 0 else fd.KERNEL_TB2
        got, _ = _run(fd, sc, precision, variant, ty, tz, ((24,), (2, 7, 1, 14), (11, 13))[q % 3])
        for a, b in zip(ref, got):
            assert np.array_equal(a, b), (dims, ty, tz)


@pytest.mark.parametrize("precision", [32, 64])
def test_two_planes(fd, precision):
    """Grids two cells high: every plane of a tile's pipeline but two lies outside."""
    g0, g1 = (fd.Grid(20, 11, 2, 0.5, max_steps=9, precision=precision) for _ in range(2))
    amps = np.sin(np.arange(9.0))
    out = []
    for g, variant in ((g0, fd.KERNEL_SPLIT), (g1, fd.KERNEL_AUTO)):
        g.add_source(2, 9, 5, 1, amps)
        pid = g.add_probe(0, 2, 8, 5, 1)
        g.set_kernel(variant)
        g.step(9)
        out.append([g.get_field(c) for c in range(6)] + [g.probe(pid)])
    assert np.abs(out[0][-1]).max() > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)
