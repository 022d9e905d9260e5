"""The default pass of grids in Debye media with more probes than a two-step pass records itself: as fast as the split
pass where that is the faster one (4,000 single values on 38 x 115 x 30: 1.13 of its time in two-step passes; lines of 35
terms 1.3), the two-step pass where its probes cost less (50,000 values: 0.6).  Bounds: times vary by a few
percent; blind to its probes the default took 1.9, 2.7 and 3.5 times as long."""
import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,lines,bound", [(4000, False, 1.15), (20000, True, 1.15), (50000, False, 0.85)])
def test_default_pass_with_many_probes(count, lines, bound):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    dims = (38, 115, 30)
    sc = S.random_case(*dims, 10, seed=5, nsteps=1500, n_mats=4)
    sc.cell_mat[:] = (np.arange(dims[2]) * 4 // dims[2]).astype(np.uint8)[:, None, None]
    rng = np.random.default_rng(3)
    sc.debye = ([1e-10, 9e-10, 8e-9, 7e-8], np.array([[0.0] * 4, [20.0] * 4] * 2))
    for q in range(count):
        i, j, k = (int(rng.integers(2, d - 2)) for d in dims)
        sc.probes.append((f"p{q}", 1, 0, 1, j, k, 35) if lines else (f"p{q}", 0, q % 3, i, j, k, 1))
    g = fdtd.Grid.from_params(sc.params(), precision=32)
    S.apply(sc, g)
    g.set_graph(20)

    def us(variant):
        g.set_kernel(variant, 0, 0)
        g.step(40)
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            g.step(100)
            b.record()
            b.synchronize()
            best = min(best, 10.0 * a.elapsed_time(b))
        return best

    split, auto = us(fdtd.KERNEL_SPLIT), us(fdtd.KERNEL_AUTO)
    print(f"{count} probes: split {split:.1f}, default {auto:.1f} us a step", flush=True)
    assert auto < bound * split
