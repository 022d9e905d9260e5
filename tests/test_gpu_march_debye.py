"""The two-step pass in Debye media against the split pass, bit for bit: one to four poles, tiles clear of some, all or
no CPML slabs, chunks of one plane up to the whole height, steps cut into odd calls, captured graphs and one-step
passes in between (they flip the field sets but not the currents')."""
import numpy as np
import pytest

from paper_2207_06908_amd import scenarios as S

pytestmark = pytest.mark.gpu

TAU = [1e-10, 9e-10, 8e-9, 7e-8]


@pytest.mark.parametrize("dims,npml,poles,tile_z", [
    ((59, 13, 9), 0, 1, (0, 1, 9)),
    ((61, 17, 12), 3, 2, (0, 5, 1)),
    ((121, 40, 23), 2, 4, (0, 7, 23)),
    ((200, 52, 30), 4, 3, (0, 2, 11)),
    ((17, 16, 16), 0, 4, (0, 2, 3)),
])
def test_two_step_debye_equals_the_split_pass(dims, npml, poles, tile_z):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2207_06908_amd import fdtd
    rng = np.random.default_rng(dims[0])

    def run(plan):
        sc = S.random_case(*dims, npml, seed=17 + dims[0], nsteps=40, n_mats=4)
        sc.cell_mat[:] = (np.arange(dims[2]) * 4 // dims[2]).astype(np.uint8)[:, None, None]  # layers: few classes
        sc.debye = (TAU[:poles], de)
        g = fdtd.Grid.from_params(sc.params(), precision=32)
        ids = S.apply(sc, g)
        assert g.num_classes <= 256
        for variant, tz, graph, n in plan:
            g.set_kernel(variant, 0, tz)
            g.set_graph(graph)
            g.step(n)
        return [g.get_field(c) for c in range(6)] + [g.probe(i) for i in ids]

    de = rng.uniform(0.5, 30.0, size=(4, poles))
    de[::2] = 0.0
    ref = run([(fdtd.KERNEL_SPLIT, 0, 0, 40)])
    assert max(np.abs(r).max() for r in ref) > 0
    plans = [[(fdtd.KERNEL_AUTO, tz, 0, 40)] for tz in tile_z]
    plans.append([(fdtd.KERNEL_TB2, tile_z[1], 0, 3), (fdtd.KERNEL_SPLIT, 0, 0, 2), (fdtd.KERNEL_FUSED, 0, 0, 3),
                  (fdtd.KERNEL_AUTO, 0, 4, 9), (fdtd.KERNEL_FUSED, 0, 0, 1), (fdtd.KERNEL_AUTO, 0, 4, 12),
                  (fdtd.KERNEL_AUTO, 0, 8, 10)])
    for plan in plans:
        for a, b in zip(ref, run(plan)):
            assert np.array_equal(a, b), plan


def test_debye_without_room_for_a_second_set():
    """A workspace too small for the second set of currents still binds, and the split pass gives the same bits; a
    smaller one does not."""
    import ctypes as C
    import torch
    from paper_2207_06908_amd import fdtd
    de = np.full((2, 4), 3.0)
    de[0] = 0.0
    out = []
    for short in (False, True, "static"):
        sc = S.random_case(100, 75, 75, 0, seed=8, nsteps=7, n_mats=2)
        sc.cell_mat[:] = 0
        sc.cell_mat[:40] = 1
        sc.debye = (TAU, de)
        g = fdtd.Grid.from_params(sc.params(), precision=32)
        ids = S.apply(sc, g)
        if short:
            n = g.workspace_bytes()
            less = 3 * 4 * 100 * 75 * 75 * 4
            assert n - less < 64 << 20 < n
            if short == "static":
                g.bind_static()
            else:
                buf = torch.empty(n - less, dtype=torch.uint8, device="cuda")
                bind = fdtd.lib().fdtd_bind_workspace
                assert bind(g._h, C.c_void_p(buf.data_ptr()), n - less - 256) == -5
                assert bind(g._h, C.c_void_p(buf.data_ptr()), n - less) == 0
                g._ws = buf
        g.step(sc.n_steps)
        out.append([g.get_field(c) for c in range(6)] + [g.probe(i) for i in ids])
        g.close()
    assert max(np.abs(r).max() for r in out[0]) > 0
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
