"""Fused inference against one product launch per layer: every block shape, ragged rows and widths.

Both paths take the K steps of each accumulator in the same order with the same instruction and share the epilogue's
arithmetic, so they agree bit for bit: no tolerance."""
import pytest

pytestmark = pytest.mark.gpu


# rows around the block shapes' limits (16-row blocks up to 256 of them, 32-row ones up to 512, then 64-row ones)
@pytest.mark.parametrize("widths,nets,rows", [
    ([5, 512, 512, 512, 512, 256], 4, (1, 15, 17, 1024, 1025, 4096, 4097, 4160)),
    ([5, 512, 512, 512, 512, 256], 1, (33, 4096, 4099, 16384, 16387)),
    ([32, 64, 320, 192], 1, (1, 63, 4097, 16400)),
    ([1, 128, 64], 3, (2, 1400, 5500)),
    ([7, 64], 1, (5, 5000, 17000)),
])
def test_blocks_match_layers(widths, nets, rows):
    import torch
    from paper_2207_06908_amd.sur import Ensemble
    ens = Ensemble(widths, n_nets=nets, max_rows=16448)
    for q in range(nets):
        ens.init_params(q, 11 + q)
    gen = torch.Generator().manual_seed(len(widths))
    for n in rows:
        x = (torch.rand(n, widths[0], generator=gen) * 3 - 1.5).cuda()
        got = {}
        for fused in (0, 1):
            ens.set_kernel(fused)
            buf = torch.full((n * widths[-1] + 2,), float("nan"), device="cuda")
            # outputs that start off a 16-byte boundary, and a guard value past the end
            y = ens.forward(nets - 1, x, out=buf[1:1 + n * widths[-1]].view(n, widths[-1]))
            ym, sp, ids, cnt = ens.infer_route(x, 0.02)
            assert torch.isnan(buf[0]) and torch.isnan(buf[-1])
            got[fused] = (y.clone(), ym, sp, ids[:int(cnt.item())])
        for a, b in zip(got[0], got[1]):
            assert torch.equal(a, b), (widths, n)
        assert torch.equal(ens.forward(nets - 1, x), got[1][0])
