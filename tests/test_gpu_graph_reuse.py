"""Captured graphs are kept for every pairing of sets they start from: calls that leave the field sets flipped (an odd
number of passes beside the replay) cost the host no more than calls that do not.  Capturing
and instantiating 200 steps again in every call takes the host four to six times as long; the bound is 3."""
import time

import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu
G, CALLS = 200, 15


@pytest.mark.parametrize("kind", ["tb2", "fused", "fused_debye", "tb2_debye"])
def test_flipped_sets_keep_their_graphs(kind):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd

    def host_us(extra):
        sc = S.random_case(30, 26, 24, 0, seed=4, nsteps=CALLS * (G + 4), n_mats=1)
        if kind.endswith("debye"):
            sc.debye = ([1e-9], np.full((1, 1), 3.0))
        g = fdtd.Grid.from_params(sc.params(), precision=32)
        S.apply(sc, g)
        g.set_kernel(fdtd.KERNEL_TB2 if kind.startswith("tb2") else fdtd.KERNEL_FUSED)
        g.set_graph(G)
        us = []
        for _ in range(CALLS):
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.step(G + extra)
            us.append((time.perf_counter() - t) * 1e6)
        return float(np.median(us[4:]))

    even = host_us(4 if kind.startswith("tb2") else 2)
    odd = host_us(2 if kind.startswith("tb2") else 1)
    print(f"{kind}: {odd:.0f} us of host time a call with flipped sets, {even:.0f} without", flush=True)
    assert odd < 3 * even
