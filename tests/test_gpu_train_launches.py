"""A training step in two launches against one product launch per layer.

Both take the K steps of each accumulator and every sum in the same order, so losses, gradients, parameters and the
bfloat16 copies (seen through a later forward pass) agree bit for bit: no tolerance."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,batches", [
    ([5, 512, 512, 512, 512, 256], (1, 64, 65, 256, 1000)),
    ([8, 320, 64, 192, 128], (63, 96, 4096, 4200)),
    ([32, 128, 64], (17, 130)),
    ([3, 64], (5, 200)),
    ([4, 64, 64, 64, 64, 64, 64, 64], (40, 129)),
])
def test_two_launches_match_layers(widths, batches):
    import numpy as np
    import torch
    from paper_2207_06908_amd.sur import Ensemble
    gen = torch.Generator().manual_seed(sum(widths))
    for n in batches:
        x = (torch.rand(n + 50, widths[0], generator=gen) * 2 - 1).cuda()
        t = torch.randn(n + 50, widths[-1], generator=gen).cuda()
        rows = torch.randperm(n + 50, generator=gen)[:n].to(torch.int32).cuda()
        got = {}
        for fused in (0, 1):
            ens = Ensemble(widths, n_nets=2, max_rows=4224)
            for q in range(2):
                ens.init_params(q, 5 + q)
            ens.set_kernel(fused)
            out = [ens.train_step(1, x, t, rows=rows, update=False).clone(), ens.get_grads(1)]
            for k in range(3):
                out.append(ens.train_step(1, x, t, rows=rows if k else None, batch=n, lr=3e-3).clone())
            out += [ens.get_grads(1), ens.get_params(1), ens.get_params(0)]
            ens.set_kernel(0)
            out += [ens.forward(q, x) for q in range(2)]
            got[fused] = [o if isinstance(o, np.ndarray) else o.cpu().numpy() for o in out]
        assert all(np.isfinite(a).all() for a in got[1])
        for i, (a, b) in enumerate(zip(got[0], got[1])):
            assert np.array_equal(a, b), (widths, n, i)
