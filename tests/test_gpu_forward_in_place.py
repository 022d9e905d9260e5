"""sur_forward with inputs inside the memory of its outputs: each chunk's inputs are read before its outputs are written,
so the answers are those of separate buffers, bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,at", [(1, 0), (65, 3), (4096, 0), (5000, "end")])
def test_forward_in_place(rows, at):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import sur
    widths = [5, 512, 512, 256]
    e = sur.Ensemble(widths, 1, 8192)
    e.init_params(0, 7)
    x = torch.rand(rows, 5, generator=torch.Generator().manual_seed(rows)).cuda()
    ref = e.forward(0, x)
    y = torch.zeros(rows * 256, device="cuda")
    first = y.numel() - x.numel() if at == "end" else at
    y[first:first + x.numel()] = x.flatten()
    got = e.forward(0, y[first:first + x.numel()].view(rows, 5), out=y.view(rows, 256))
    assert torch.equal(ref, got)
    assert float(ref.abs().max()) > 0
