"""Coefficient classes of layered and blocky media, where whole planes and rows of class ids are copies of the ones
before: fields against the FP64 oracle, element by element (1e-11 of the largest value, FP64 kernels)."""
import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu

NX, NY, NZ = 13, 11, 12


def _media(name, rng):
    cm = np.zeros((NZ, NY, NX), np.uint8)
    if name == "layers":
        cm[:] = (np.arange(NZ) // 3)[:, None, None]
    elif name == "rows":
        cm[:] = (np.arange(NY) // 3)[None, :, None]
    elif name == "columns":
        cm[:] = (np.arange(NX) // 4)[None, None, :]
    elif name == "blocks":
        cm[:] = rng.integers(0, 4, (4, 4, 4)).repeat(3, 0).repeat(3, 1).repeat(4, 2)[:NZ, :NY, :NX]
    elif name == "cells":  # single cells that differ, at the ends of runs of equal planes and rows
        for k, j, i in ((0, 0, 0), (NZ - 1, NY - 1, NX - 1), (4, 0, 5), (7, NY - 1, 0), (8, 5, NX - 1), (5, 5, 5)):
            cm[k, j, i] = 1 + (i + j + k) % 3
    return cm


@pytest.mark.parametrize("name", ["uniform", "layers", "rows", "columns", "blocks", "cells"])
def test_block_media_against_the_oracle(oracle_mod, name):
    from paper_2207_06908_amd import fdtd
    sc = S.random_case(NX, NY, NZ, 0, seed=5, nsteps=16, n_mats=4)
    sc.cell_mat[:] = _media(name, np.random.default_rng(9))
    o = oracle_mod.Oracle.from_params(sc.params())
    S.apply(sc, o)
    g = fdtd.Grid.from_params(sc.params(), precision=64)
    S.apply(sc, g)
    o.step(sc.n_steps)
    g.step(sc.n_steps)
    for c in range(6):
        ref, got = o.get_field(c), g.get_field(c)
        assert np.abs(ref).max() > 0
        assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max(), c
