"""Paths of the library that take the same call by different kernels, against each other and the
oracle, at the sizes where they can differ."""
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


def _by_id(parts):
    order = np.argsort(parts["id"])
    return {k: v[..., order] for k, v in parts.items()}


# grid, shape order, current scheme: cubic and flat tiles, ragged edges, thin and single-cell
# axes (runtime-shaped tiles; 70x2x2 has more halo than the tiled kernel's LDS)
FP64_TILE_CASES = [((9, 8, 5), 3, 0), ((9, 8, 5), 2, 1), ((17, 9, 1), 3, 0), ((17, 9, 1), 2, 0), ((70, 1, 1), 3, 1),
                   ((5, 3, 2), 2, 0), ((5, 3, 2), 3, 1), ((70, 2, 2), 3, 0), ((40, 24, 36), 3, 0)]


@pytest.mark.parametrize("n,O,current", FP64_TILE_CASES)
def test_fp64_sorted_push_equals_unsorted_push(ppm, orc, n, O, current):
    """A push of freshly sorted particles (tile by tile) against one of the same particles left
    unsorted; some particles start at the edges of the box, outside it (also by more than a
    period) and many in one cell.  FP64 sums in another order: 1e-12 of the largest value."""
    species, E, B = random_state(orc, n, 6, seed=31, uth=0.4)
    N = np.array(n, dtype=np.float64)
    pos = species[0]["pos"]
    edge = [np.zeros(3), N - 1e-9, N - 0.5, 0.5 * N, 2.3 * N, -0.2 * N, -1.4 * N]
    for i, x in enumerate(edge):
        pos[:, i] = x
    pos[:, 20:min(120, pos.shape[1])] = 0.37 * N[:, None]
    kw = dict(n=n, dt=0.35, shape_order=O, field_order=2, current_scheme=current, relax_max_iter=100)
    out = []
    for sort in (True, False):
        run = ppm.Run(ppm.make_params(precision=ppm.PP_PREC_FP64, **kw), species, E=E, B=B)
        run.gather_push_deposit()
        if sort:
            run.sort()
        run.gather_push_deposit()
        out.append((run.fields()[2], [_by_id(run.particles(s)) for s in range(len(species))], run.diagnostics().flags))
        run.close()
    (J1, p1, f1), (J2, p2, f2) = out
    assert f1 == f2 == 0
    assert rel_inf(J1, J2) < 1e-12
    for a, b in zip(p1, p2):
        assert np.max(np.abs(periodic_diff(a["pos"], b["pos"], n))) < 1e-12
        assert rel_inf(a["u"], b["u"]) < 1e-12


@pytest.mark.parametrize("n,order", [((33, 9, 5), 6), ((5, 40, 33), 6), ((31, 8, 1), 4), ((7, 3, 2), 6), ((1, 1, 64), 2),
                                     ((64, 17, 34), 2)])
def test_field_step_matches_oracle_for_any_sweep_count(ppm, orc, n, order):
    """The field step alone (no particles) at the edges of its 32x8 columns, over time steps whose
    relaxation takes one, an odd and an even number of sweeps (they use the arrays differently).
    Both sides relax to 1e-14, in FP64: 1e-12 of the largest value."""
    species, E, B = random_state(orc, n, 1, seed=17)
    seen = set()
    for dt in (1e-8, 0.05, 0.1, 0.2, 0.3, 0.4):
        kw = dict(n=n, dt=dt, shape_order=3, field_order=order, relax_tol=1e-14, relax_max_iter=200)
        ref = orc.Run(orc.make_params(**kw), [], E=E, B=B)
        run = ppm.Run(ppm.make_params(precision=ppm.PP_PREC_FP64, **kw), [], E=E, B=B)
        for _ in range(2):
            ref.step()
            run.field_step()
        Eg, Bg, _ = run.fields()
        sweeps = run.diagnostics(ppm.PP_DIAG_FIELDS).relax_iters
        seen.add(1 if sweeps == 1 else 2 + sweeps % 2)
        assert rel_inf(Eg, ref.E) < 1e-12 and rel_inf(Bg, ref.B) < 1e-12, (dt, sweeps)
        run.close()
    assert seen == {1, 2, 3} or max(n) == 1


@pytest.mark.parametrize("n,O", [((9, 8, 5), 3), ((17, 9, 1), 2), ((64, 1, 1), 3), ((18, 2, 2), 2), ((3, 5, 8), 3)])
def test_species_sorted_one_by_one_and_together(ppm, orc, n, O):
    """Three species, one of them empty and one with 700 particles in a cell, sorted together, one
    by one, and one of them twice: the current of the next push is an exact sum over the same
    particles, so it has to come out bit for bit the same."""
    species, E, B = random_state(orc, n, 5, seed=3, uth=0.4, nspecies=3, pair=False)
    species[1] = dict(species[1], pos=np.zeros((3, 0)), u=np.zeros((3, 0)))
    many = 0.4 * np.array(n)[:, None] + np.random.default_rng(1).uniform(0, 0.3, (3, 700))
    species[2] = dict(species[2], pos=np.concatenate([species[2]["pos"], many], 1),
                      u=np.concatenate([species[2]["u"], np.full((3, 700), 0.1)], 1))
    from paper_1211_4575_amd import inputs as I
    split = []
    for s in species:
        cell, off = I.to_split(s["pos"], n, origin=I.split_origin(O))
        split.append(dict(q=s["q"], m=s["m"], w=s["w"], cell=cell, off=off, u=s["u"].astype(np.float32)))
    kw = dict(n=n, dt=0.35, shape_order=O, field_order=4, relax_max_iter=100, precision=ppm.PP_PREC_FP32_SPLIT)
    out = []
    for order in ((-1,), (2, 0, 1), (2, -1), (0, 0, -1)):
        run = ppm.Run(ppm.make_params(**kw), split, E=E, B=B)
        for _ in range(3):
            run.gather_push_deposit()
            for s in order:
                run.sort(s)
        run.gather_push_deposit()
        assert run.diagnostics().flags == 0
        assert [len(np.unique(run.particles(s)["id"])) for s in range(3)] == [s["u"].shape[1] for s in split]
        out.append(run.fields()[2])
        run.close()
    for J in out[1:]:
        assert np.array_equal(J, out[0])


@pytest.mark.parametrize("n,O", [((9, 8, 5), 3), ((17, 9, 1), 2), ((64, 1, 1), 3), ((70, 2, 2), 3), ((3, 5, 8), 2)])
def test_fp64_sort_orders(ppm, orc, n, O):
    """Pushes with and without sorts between them, in several orders (the sort after a tiled push
    takes its counts and ranks, the others count again): the same particles, J and cell order as
    sorting every time; each sum is FP64 in another order, 1e-12 of the largest value."""
    species, E, B = random_state(orc, n, 5, seed=8, uth=0.4, nspecies=2, pair=False)
    many = 0.4 * np.array(n)[:, None] + np.random.default_rng(1).uniform(0, 0.3, (3, 5000))
    species[1] = dict(species[1], pos=np.concatenate([species[1]["pos"], many], 1),
                      u=np.concatenate([species[1]["u"], np.full((3, 5000), 0.1)], 1))
    species[0]["pos"][:, 0] = 1.7 * np.array(n)  # a period outside
    species[0]["u"][:, 1] = np.nan  # flagged and left as it is
    kw = dict(n=n, dt=0.35, shape_order=O, field_order=4, relax_max_iter=100, precision=ppm.PP_PREC_FP64)
    out = []
    for sorts in ((-1,), (0, 1), (1, -1), (), (0,), "every second step"):
        run = ppm.Run(ppm.make_params(**kw), species, E=E, B=B)
        for i in range(4):
            run.gather_push_deposit()
            for s in (sorts if sorts != "every second step" else ((-1, -1) if i % 2 else ())):
                run.sort(s)
        run.gather_push_deposit()
        flags = run.diagnostics().flags
        run.sort()
        parts = [run.particles(s) for s in range(2)]
        out.append((run.fields()[2], [_by_id(p) for p in parts], flags))
        # in cell order, the cells tile by tile (sides of a tile: powers of two, 64 cells)
        t = [1, 1, 1]
        while np.prod(t) < 64 and any(t[d] < n[d] for d in range(3)):
            t[min((d for d in range(3) if t[d] < n[d]), key=lambda d: t[d])] *= 2
        nt = [-(-n[d] // t[d]) for d in range(3)]
        for p in parts:
            c = np.floor(p["pos"] + 0.5).astype(int)
            c = np.where(c >= np.array(n)[:, None], c - np.array(n)[:, None], c)
            tile = c[0] // t[0] + nt[0] * (c[1] // t[1] + nt[1] * (c[2] // t[2]))
            key = tile * 64 + c[0] % t[0] + t[0] * (c[1] % t[1] + t[1] * (c[2] % t[2]))
            assert np.all(np.diff(key) >= 0)
        run.close()
    for J, parts, flags in out[1:]:
        assert flags == out[0][2] == ppm.PP_FLAG_NONFINITE
        assert rel_inf(J, out[0][0]) < 1e-12
        for a, b in zip(parts, out[0][1]):
            assert np.max(np.abs(periodic_diff(a["pos"], b["pos"], n))) < 1e-12
            assert np.array_equal(np.isnan(a["u"]), np.isnan(b["u"]))
            assert np.nanmax(np.abs(a["u"] - b["u"])) < 1e-12


@pytest.mark.parametrize("n,O", [((9, 10, 7), 3), ((13, 4, 16), 2), ((24, 23, 24), 3), ((22, 24, 21), 2), ((28, 26, 27), 3)])
def test_split_push_for_every_box_size_equals_batched(ppm, orc, n, O):
    """Boxes of up to 256, 512 and 768 tiles and species take workgroups of different sizes, a batch
    always the paired ones: the same particles and exact sums, so bit for bit the same."""
    import torch
    from paper_1211_4575_amd import inputs as I
    species, E, B = random_state(orc, n, 3, seed=12, uth=0.4)
    many = 0.4 * np.array(n)[:, None] + np.random.default_rng(1).uniform(0, 0.3, (3, 1300))
    split = []
    for s in species:
        cell, off = I.to_split(np.concatenate([s["pos"], many], 1), n, origin=I.split_origin(O))
        u = np.concatenate([s["u"], np.full((3, 1300), 0.1)], 1).astype(np.float32)
        split.append(dict(q=s["q"], m=s["m"], w=s["w"], cell=cell, off=off, u=u))
    kw = dict(n=n, dt=0.35, shape_order=O, field_order=4, relax_max_iter=100, precision=ppm.PP_PREC_FP32_SPLIT)
    out = []
    for batched in (False, True):
        run = ppm.Run(ppm.make_params(**kw), split, E=E, B=B)
        if batched:
            batch = ppm.pp_batch_create(1, torch.cuda.current_stream().cuda_stream)
            ppm.pp_batch_add(batch, run.handle)
            for _ in range(4):
                ppm.pp_batch_step(batch)
            ppm.pp_batch_remove(batch, run.handle)
            ppm.pp_batch_destroy(batch)
        else:
            for _ in range(4):
                run.step()
        assert run.diagnostics().flags == 0
        out.append((run.fields(), [_by_id(run.particles(s)) for s in range(2)]))
        run.close()
    (f1, p1), (f2, p2) = out
    for a, b in zip(f1, f2):
        assert np.array_equal(a, b)
    for a, b in zip(p1, p2):
        assert all(np.array_equal(a[k], b[k]) for k in a)


@pytest.mark.parametrize("n,order", [((33, 9, 350), 6), ((70, 17, 180), 4), ((32, 8, 1400), 2)])
def test_field_step_of_boxes_marched_in_planes(ppm, orc, n, order):
    """The field step where a block takes several planes, with numbers of tiles that the XCDs do not
    divide evenly.  Both sides relax to 1e-14, in FP64: 1e-12 of the largest value."""
    _, E, B = random_state(orc, n, 1, seed=19)
    kw = dict(n=n, dt=0.3, shape_order=3, field_order=order, relax_tol=1e-14, relax_max_iter=200)
    ref = orc.Run(orc.make_params(**kw), [], E=E, B=B)
    run = ppm.Run(ppm.make_params(precision=ppm.PP_PREC_FP64, **kw), [], E=E, B=B)
    for _ in range(2):
        ref.step()
        run.field_step()
    Eg, Bg, _ = run.fields()
    assert rel_inf(Eg, ref.E) < 1e-12 and rel_inf(Bg, ref.B) < 1e-12
    run.close()


@pytest.mark.parametrize("precision", ["split", "fp64"])
@pytest.mark.parametrize("count", [4608, 4609, 65534, 65536])
def test_sort_of_a_tile_at_the_sizes_of_its_lds_image(ppm, orc, precision, count):
    """A box of one tile: the sort loses no particle, and the next current is the same for the
    particles in another order (the split form; bit for bit, in fixed point) or left unsorted (FP64
    may be; 1e-12 of the largest value for sums in another order)."""
    from paper_1211_4575_amd import inputs as I
    n = (4, 4, 4)
    rng = np.random.default_rng(2)
    _, E, B = random_state(orc, n, 1, seed=5)
    s = dict(q=-1.0, m=1.0, w=1.0 / count, pos=rng.uniform(0, 4, (3, count)), u=rng.normal(0, 0.3, (3, count)))
    split = precision == "split"
    if split:
        cell, off = I.to_split(s["pos"], n, origin=I.split_origin(3))
        s = dict(q=-1.0, m=1.0, w=1.0 / count, cell=cell, off=off, u=s["u"].astype(np.float32))
    kw = dict(n=n, dt=0.35, shape_order=3, field_order=2, relax_max_iter=100,
              precision=ppm.PP_PREC_FP32_SPLIT if split else ppm.PP_PREC_FP64)
    out = []
    for first in (True, False):
        if split and not first:
            s = dict(s, **{k: np.ascontiguousarray(s[k][..., ::-1]) for k in ("cell", "off", "u")})
        run = ppm.Run(ppm.make_params(**kw), [s], E=E, B=B)
        run.gather_push_deposit()
        if split or first:
            run.sort()
        run.gather_push_deposit()
        assert run.diagnostics().flags == 0
        assert np.array_equal(np.sort(run.particles(0)["id"]), np.arange(count))
        out.append(run.fields()[2])
        run.close()
    assert np.array_equal(*out) if split else rel_inf(*out) < 1e-12


@pytest.mark.parametrize("current", [0, 1])
@pytest.mark.parametrize("n,O", [((24, 16, 1), 3), ((9, 17, 1), 2), ((13, 11, 1), 3)])
def test_flat_tiles_match_oracle(ppm, orc, n, O, current):
    """The current of 8x8x1 tiles, whose z nodes share their additions, over three steps of particles
    that cross faces along z too.  FP32 weights and offsets: 1e-5 in the L2 norm."""
    from paper_1211_4575_amd import inputs as I
    species, E, B = random_state(orc, n, 5, seed=23, uth=0.7)
    split, ref_species = [], []
    for s in species:
        cell, off = I.to_split(s["pos"], n, origin=I.split_origin(O))
        u = s["u"].astype(np.float32)
        split.append(dict(q=s["q"], m=s["m"], w=s["w"], cell=cell, off=off, u=u))
        ref_species.append(dict(s, pos=I.from_split(cell, off, n), u=u.astype(np.float64)))
    kw = dict(n=n, dt=0.45, shape_order=O, field_order=4, relax_tol=1e-14, relax_max_iter=200)
    ref = orc.Run(orc.make_params(current_scheme=current, **kw), ref_species, E=E, B=B)
    run = ppm.Run(ppm.make_params(precision=ppm.PP_PREC_FP32_SPLIT, current_scheme=current, **kw), split, E=E, B=B)
    for _ in range(3):
        ref.step()
        run.step()
        J = run.fields()[2]
        assert np.linalg.norm(J - ref.J) < 1e-5 * np.linalg.norm(ref.J)
    assert run.diagnostics().flags == 0
    run.close()


@pytest.mark.parametrize("order", [2, 4, 6])
def test_field_step_of_a_box_past_the_caches_equals_batched(ppm, order):
    """A box whose arrays stream past the caches when it is stepped alone, not in a batch: bit for bit
    the same fields."""
    import torch
    n = (164, 161, 160)
    gen = torch.Generator(device="cuda").manual_seed(4)
    E0, B0 = (torch.randn(3, n[2], n[1], n[0], dtype=torch.float64, device="cuda", generator=gen) for _ in range(2))
    kw = dict(n=n, dt=0.35, shape_order=2, field_order=order, relax_tol=1e-8, relax_max_iter=100,
              precision=ppm.PP_PREC_FP32_SPLIT)
    species = [dict(q=-1.0, m=1.0, w=0.1, cell=np.arange(64, dtype=np.int32), off=np.zeros((3, 64), np.float32),
                    u=np.full((3, 64), 0.1, np.float32))]
    out = []
    for batched in (False, True):
        run = ppm.Run(ppm.make_params(**kw), species)
        run.E.copy_(E0)
        run.B.copy_(B0)
        if batched:
            batch = ppm.pp_batch_create(1, torch.cuda.current_stream().cuda_stream)
            ppm.pp_batch_add(batch, run.handle)
            for _ in range(2):
                ppm.pp_batch_step(batch)
            ppm.pp_batch_remove(batch, run.handle)
            ppm.pp_batch_destroy(batch)
        else:
            for _ in range(2):
                run.step()
        torch.cuda.synchronize()
        out.append((run.E.clone(), run.B.clone()))
        run.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
