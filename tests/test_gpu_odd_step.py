"""The single step after two-step passes, by the split or the fused pass as the grid's size has it, against the split
pass alone, bit for bit: FP64 grids without a CPML on either side of the line (6 x 2^20 nodes)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(186, 184, 183), (189, 184, 183)])
def test_odd_step_fp64(dims):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    assert (dims[0] * dims[1] * dims[2] < 6 << 20) == (dims[0] == 186)
    out = []
    for variant in (fdtd.KERNEL_SPLIT, fdtd.KERNEL_AUTO):
        g = fdtd.Grid(*dims, 0.5, max_steps=4, precision=64)
        g.add_source(2, 90, 91, 92, np.array([1.0, -2.0, 3.0, 0.5]))
        pid = g.add_probe(0, 2, 91, 91, 92)
        g.set_kernel(variant, 0, 0)
        g.step(3)
        g.step(1)
        out.append([g.get_field(c) for c in (0, 2, 4)] + [g.probe(pid)])
        g.close()
    assert np.abs(out[0][-1]).max() > 0
    for a, b in zip(*out):
        assert np.array_equal(a, b)
