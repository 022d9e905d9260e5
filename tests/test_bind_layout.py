"""A refused binding leaves the context as it was: the layout (with its two sets of pole currents) before a binding, the
whole run after one, and the static array with the context that holds it."""
import ctypes as C

import numpy as np
import pytest

from paper_2207_06908_amd import fdtd
from paper_2207_06908_amd import scenarios as S

TAU = [1e-10, 9e-10, 8e-9, 7e-8]
DIMS = (100, 75, 75)
ONE_SET = 3 * 4 * 100 * 75 * 75 * 4  # bytes
STATIC = 64 << 20  # FDTD_STATIC_BYTES


def _grid(nsteps=24):
    """A grid whose workspace fits the static array with one set of currents only."""
    sc = S.random_case(*DIMS, 0, seed=8, nsteps=nsteps, n_mats=2)
    sc.cell_mat[:] = 0
    sc.cell_mat[:40] = 1
    sc.debye = (TAU, np.array([[0.0] * 4, [3.0] * 4]))
    g = fdtd.Grid.from_params(sc.params(), precision=32)
    ids = S.apply(sc, g)
    n = g.workspace_bytes()
    assert n - ONE_SET < STATIC < n
    return g, ids, n


def test_a_refused_address_keeps_both_sets():
    g, _, n = _grid()
    bind = fdtd.lib().fdtd_bind_workspace
    for size in (n - ONE_SET, n):  # misaligned: refused on the host, the memory is not looked at
        assert bind(g._h, C.c_void_p(0x10008), size) == -5
        assert g.workspace_bytes() == n
    assert bind(g._h, C.c_void_p(0x10000), n - ONE_SET - 256) == -5
    assert g.workspace_bytes() == n


def test_a_static_binding_without_a_gpu_keeps_both_sets():
    import torch
    if torch.cuda.is_available():
        pytest.skip("needs a machine without a GPU")
    g, _, n = _grid()
    assert fdtd.lib().fdtd_bind_static(g._h) == -6
    assert g.workspace_bytes() == n


@pytest.mark.gpu
def test_a_bound_context_is_not_laid_out_again():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    out = []
    for again in (False, True):
        g, ids, n = _grid()
        g.set_kernel(fdtd.KERNEL_TB2)
        g.set_graph(8)
        g.step(10)
        if again:
            assert fdtd.lib().fdtd_bind_static(g._h) == -3
            assert g.workspace_bytes() == n
        g.step(14)
        out.append([g.probe(i) for i in ids] + [g.get_field(c) for c in range(6)])
        g.close()
    assert max(np.abs(a).max() for a in out[0]) > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.gpu
def test_the_array_stays_with_its_holder():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    bind = fdtd.lib().fdtd_bind_static
    held = fdtd.Grid(20, 20, 20, 0.5, max_steps=4)
    held.bind_static()
    assert bind(held._h) == -3
    g, ids, n = _grid()
    assert bind(g._h) == -3            # the array is still held
    assert g.workspace_bytes() == n    # and the full size is asked for
    g.step(8)                          # an ordinary binding
    held.close()
    assert np.isfinite(g.probe(ids[0])).all()
    g.close()
