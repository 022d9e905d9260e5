"""An oblique wire (a source at every edge it touches) and many ideal sources in a grid of more coefficient classes than the
two-step tiles' tables hold: against the split pass, bit for bit, and the time of the wire's sources in the two-step pass
(at most 45 us a step more than without the wire; reading all sources of a column in every plane took 70)."""
import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu


def _grid(fd, dims, npml, precision, steps, wire, sources=0):
    sc = S.random_case(*dims, npml, seed=9, nsteps=steps, n_mats=4)
    rng = np.random.default_rng(2)
    for q in range(sources):  # along one column, and spread
        k = 1 + q % (dims[2] - 2)
        i, j = (dims[0] // 2, dims[1] // 2 + 1) if q % 2 else (int(rng.integers(1, dims[0] - 1)), int(rng.integers(1, dims[1] - 1)))
        sc.sources.append((q % 3, i, j, k, rng.standard_normal(steps)))
    sc.wires = []
    g = fd.Grid.from_params(sc.params(), precision=precision)
    ids = S.apply(sc, g)
    if wire:
        m = npml + 1.3
        g.add_oblique_wire([m, m + 0.4, m + 0.2], [m + 9.0, m + 10.0, m + 11.0], 0.004, 0, sc.sources[0][4], 2)
    g.finalize()
    return g, ids


@pytest.mark.parametrize("npml,precision,wire", [(0, 32, True), (6, 32, True), (6, 32, False), (0, 64, False), (6, 64, True)])
def test_sources(npml, precision, wire):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    ref = None
    for variant, ty, tz in ((fdtd.KERNEL_SPLIT, 0, 0), (fdtd.KERNEL_TB2, 0, 0), (fdtd.KERNEL_TB2, 8, 31), (fdtd.KERNEL_TB2, 4, 3)):
        g, ids = _grid(fdtd, (42, 36, 61), npml, precision, 9, wire, 120)
        assert g.num_classes > 2048
        g.set_kernel(variant, ty, tz)
        g.step(6)
        g.step(3)
        out = [g.get_field(c) for c in range(6)] + [g.probe(i) for i in ids]
        if ref is None:
            ref = out
            assert max(np.abs(r).max() for r in ref) > 0
        for a, b in zip(ref, out):
            assert np.array_equal(a, b), (variant, ty, tz)


def test_time_of_a_wire():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    us = []
    for wire in (False, True):
        g, _ = _grid(fdtd, (42, 36, 61), 10, 32, 1000, wire)
        g.set_kernel(fdtd.KERNEL_TB2, 4, 16)
        g.set_graph(20)
        g.step(40)
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            g.step(100)
            b.record()
            b.synchronize()
            best = min(best, 10.0 * a.elapsed_time(b))
        us.append(best)
    print(f"{g.num_classes} classes: {us[0]:.1f} us a step, with a wire {us[1]:.1f}", flush=True)
    assert us[1] < us[0] + 45.0
