"""States at the edge of what a kernel's scale, counters or tables are laid out for: every particle
at one corner, in one cell, leaving its tile at once, or moved by the caller between two calls."""
import numpy as np
import pytest

from _state import periodic_diff, random_state, rel_inf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ppm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1211_4575_amd import pp
    pp.lib()
    return pp


@pytest.mark.parametrize("n,O,per_tile", [((16, 16, 16), 3, 1024), ((16, 16, 16), 2, 1024), ((24, 24, 1), 3, 2048),
                                          ((12, 8, 20), 3, 1000)])
def test_charge_of_a_cluster_that_splits_over_its_tiles(ppm, orc, n, O, per_tile):
    """Particles at the corner of a tile that one push shares out among the tiles around it, while
    each of them still charges the node they started from: the charge density after the push, with
    the sort's order pending, and with it applied.  Contributions are rounded to 2^-(50 - 13 - 2) of
    the largest at worst, 2^13 of them to a node of 0.14 of that or more: 1e-10 of the largest node."""
    from paper_1211_4575_amd import inputs as I
    flat = n[2] == 1
    tile = (8, 8) if flat else (4, 4, 4)
    corner = np.array([t if O == 3 else t - 0.5 for t in tile] + ([0.25] if flat else []))
    signs = np.array(np.meshgrid(*[(-1, 1)] * len(tile))).reshape(len(tile), -1)
    u = np.repeat(0.05 * signs, per_tile, axis=1)
    u = np.concatenate([u, np.zeros((3 - len(tile), u.shape[1]))])
    pos = np.repeat(corner[:, None], u.shape[1], axis=1)
    cell, off = I.to_split(pos, n, origin=I.split_origin(O))
    sp = dict(q=1.0, m=1.0, w=1.0, cell=cell, off=off, u=u.astype(np.float32))
    kw = dict(n=n, dt=0.4, shape_order=O, field_order=2, relax_max_iter=100)
    run = ppm.Run(ppm.make_params(precision=ppm.PP_PREC_FP32_SPLIT, **kw), [sp])
    got = []
    for call in (run.gather_push_deposit, run.sort, lambda: None):
        call()
        got.append(run.diagnostics(ppm.PP_DIAG_RHO).gauss_max)  # E = 0: the largest charge density
        if call == run.sort:
            parts = run.particles(0)
    run.close()
    rho = orc.deposit_rho(orc.make_params(**kw), 1.0, 1.0, I.from_split(parts["cell"], parts["pos"], n))
    assert np.max(np.abs(np.array(got) / np.max(rho) - 1.0)) < 1e-10, (got, np.max(rho))


@pytest.mark.parametrize("count,q", [(1, 1.0), (64, -0.5), (100, 1.0)])
def test_charge_of_a_single_cell(ppm, count, q):
    """A box of one cell, whose only node takes every particle's whole charge: density q w count, to the
    FP64 rounding of the weights (1e-12)."""
    rng = np.random.default_rng(4)
    sp = dict(q=q, m=1.0, w=1.0, cell=np.zeros(count, np.int32), off=rng.uniform(0, 1, (3, count)).astype(np.float32),
              u=np.zeros((3, count), np.float32))
    for background in (0.0, -q * count):
        run = ppm.Run(ppm.make_params((1, 1, 1), dt=0.4, shape_order=3, field_order=2, rho_background=background,
                                      precision=ppm.PP_PREC_FP32_SPLIT), [sp])
        for call in (lambda: None, run.gather_push_deposit, run.sort):
            call()
            d = run.diagnostics(ppm.PP_DIAG_RHO)
            assert abs(d.gauss_max - abs(q * count + background)) < 1e-12 * abs(q) * count
        run.close()
