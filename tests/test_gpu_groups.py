"""Grouped FP64 evaluation: far copies of 64-element groups by multipole
expansions, near ones element by element, in units of several sizes.

Bound against the oracle: 1e-10 pointwise on non-negligible points, the FP64
evaluation's own (the expansions are truncated below 3e-12 of a group's summed
absolute charge over distance, the closed forms round at 1e-11 of an element's
field).  Everything that only regroups the work is held to equal bits.
"""
import numpy as np
import pytest

import oracle
from synth import Images, gem_cell, gem_eval_points

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nb():
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    import paper_2606_24154_amd as nb
    return nb


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", dtype=torch.float64)


def evaluate(nb, geom, sigma, pts, precision=0):
    dp = nb.DevicePanels.from_geometry(geom, "cuda:0")
    out = nb.eval_points(dp, dev(sigma), *[dev(pts[:, k]) for k in range(3)], precision=precision)
    return torch.stack(out, 1).cpu().numpy()


def geometry(copies):
    """A ragged mesh (1242 elements: 19 groups and 26 elements over) with 121
    copies, with more copies than one list of near ones holds (169), with
    reflections, or with enough groups for a second level of expansions."""
    g = gem_cell(k=17, nr=2, n_images=5)
    if copies == "121":
        return g
    if copies == "levels":  # 16 816 elements, 263 groups: expansions of 4 and of 16 groups
        return gem_cell(k=120, nr=7, n_images=3)
    if copies == "none":  # one copy: no grouping
        return g.with_images(Images(a1=g.images.a1, a2=g.images.a2))
    im = g.images
    if copies == "169":
        return g.with_images(Images(a1=im.a1, a2=im.a2, n1=6, n2=6))
    return g.with_images(Images(a1=im.a1, a2=im.a2, n1=2, n2=3, mirror_mask=5,
                                mirror_pos=np.array([-2e-4, 0.0, -1.5e-3]),
                                mirror_parity=np.array([1, 1, -1], np.int32)))


def points(geom, m, seed=5):
    """Field-map points, and among them points in the hole and a few element
    sizes above the copper, where groups of the own cell are near."""
    p = gem_eval_points(geom, m, seed)
    rng = np.random.default_rng(seed)
    c = 0.5 * (geom.images.a1 + geom.images.a2)
    near = p[::3]
    near[:] = c + rng.normal(size=near.shape) * np.array([12e-6, 12e-6, 30e-6])
    return p


@pytest.mark.parametrize("copies", ["121", "169", "mirror", "levels"])
def test_grouped_eval_against_oracle(nb, copies):
    g = geometry(copies)
    rng = np.random.default_rng(7)
    sigma = 1e-5 * np.where(g.value > 0, 1.0, -1.0) * (0.5 + rng.random(g.n))
    p = points(g, 61)
    ref = oracle.eval_points(g, sigma, p)
    got = evaluate(nb, g, sigma, p)
    ap = np.abs(ref[:, 0])
    en = np.linalg.norm(ref[:, 1:], axis=1)
    s, t = ap >= 1e-3 * ap.max(), en >= 1e-3 * en.max()
    assert np.max(np.abs(got[s, 0] - ref[s, 0]) / ap[s]) <= 1e-10
    assert np.max(np.linalg.norm(got[t, 1:] - ref[t, 1:], axis=1) / en[t]) <= 1e-10


@pytest.mark.parametrize("copies, precision", [("121", 0), ("169", 0), ("mirror", 0), ("none", 0), ("levels", 0),
                                               ("121", 1), ("mirror", 1), ("none", 1)])
def test_unit_sizes_give_equal_bits(nb, copies, precision):
    """Calls of 1 to 530 000 points take units from lattice rows and runs
    of 8 elements (16-element runs where nothing is grouped) to whole segments,
    unordered, small-sorted and radix-sorted."""
    g = geometry(copies)
    if copies == "none":  # an odd start of the runs of pairs
        g = g.subset(np.arange(1, g.n))
    rng = np.random.default_rng(8)
    sigma = 1e-5 * rng.standard_normal(g.n)
    p = points(g, 530_000)
    full = evaluate(nb, g, sigma, p, precision)
    for m in (1, 63, 64, 65, 700, 4096, 4097, 40_000):
        at = rng.choice(len(p), m, replace=False)
        assert np.array_equal(evaluate(nb, g, sigma, p[at], precision), full[at]), m


@pytest.mark.parametrize("precision", [0, 1])
def test_fewer_points_at_a_time_give_equal_bits(nb, precision):
    """67 216 elements without copies are one segment of 1051 groups: the unit
    sums of 20 000 points are taken a few thousand points at a time."""
    g = gem_cell(k=360, nr=10, n_images=1)
    g = g.with_images(Images(a1=g.images.a1, a2=g.images.a2))
    sigma = 1e-5 * np.random.default_rng(11).standard_normal((3, g.n))
    p = points(g, 20_000)
    dp = nb.DevicePanels.from_geometry(g, "cuda:0")
    out = nb.eval_points_multi(dp, dev(sigma), *[dev(p[:, k]) for k in range(3)], precision=precision)
    out = torch.stack(out, 2).cpu().numpy()
    at = np.arange(7, len(p), 33)
    for k in range(3):
        assert np.array_equal(evaluate(nb, g, sigma[k], p[at], precision), out[k][at]), k
    assert np.array_equal(evaluate(nb, g, sigma[1], p, precision), out[1])


def test_units_within_the_fixed_scratch(nb):
    """The allocation-free evaluation takes the finer units that its scratch has
    room for: rows of expansions, expansions, and whole segments."""
    ses = nb.Session(nb.DevicePanels.from_geometry(geometry("121"), "cuda:0"))
    p = points(geometry("121"), 70_000)
    for m in (64, 1000, 6000, 20_000, 70_000):
        q = [dev(p[:m, k]) for k in range(3)]
        out = [torch.empty_like(q[0]) for _ in range(4)]
        ses.eval_points_noalloc(*q, out)
        for a, b in zip(out, ses.eval_points(*q)):
            assert torch.equal(a, b), m
    ses.close()


def test_lattice_of_several_lists(nb):
    """441 copies, listed 128 at a time: all are near the group that spans the foil
    and the drift plane, a few rows of them the others."""
    g = geometry("121")
    g = g.with_images(Images(a1=g.images.a1, a2=g.images.a2, n1=10, n2=10))
    sigma = 1e-5 * (0.5 + np.random.default_rng(12).random(g.n))
    p = points(g, 270_000)
    full = evaluate(nb, g, sigma, p)
    ref = oracle.eval_points(g, sigma, p[:40])
    assert np.max(np.abs(full[:40, 0] / ref[:, 0] - 1)) <= 1e-10
    en = np.linalg.norm(ref[:, 1:], axis=1)
    t = en >= 1e-3 * en.max()
    assert np.max(np.linalg.norm(full[:40, 1:] - ref[:, 1:], axis=1)[t] / en[t]) <= 1e-10
    rng = np.random.default_rng(13)
    for m in (1, 64, 700, 4097):
        at = rng.choice(len(p), m, replace=False)
        assert np.array_equal(evaluate(nb, g, sigma, p[at]), full[at]), m


@pytest.mark.parametrize("ncol", [2, 3, 5])
def test_columns_equal_single_evaluations(nb, ncol):
    g = geometry("121")
    sigma = 1e-5 * np.random.default_rng(9).standard_normal((ncol, g.n))
    p = points(g, 777)
    dp = nb.DevicePanels.from_geometry(g, "cuda:0")
    out = torch.stack(nb.eval_points_multi(dp, dev(sigma), *[dev(p[:, k]) for k in range(3)]), 2).cpu().numpy()
    for k in range(ncol):
        assert np.array_equal(out[k], evaluate(nb, g, sigma[k], p)), k


def test_density_that_is_not_finite(nb):
    """A group with such a density is evaluated element by element: infinite
    results keep their sign instead of turning into NaN in an expansion."""
    g = geometry("121")
    sigma = np.full(g.n, 1e-6)
    sigma[100] = np.inf
    got = evaluate(nb, g, sigma, points(g, 200))
    assert np.all(got[:, 0] == np.inf)
    assert np.all(np.isinf(got[:, 1:]))
    sigma[100] = np.nan
    assert np.all(np.isnan(evaluate(nb, g, sigma, points(g, 200))))


@pytest.mark.parametrize("copies", ["121", "169", "levels"])
@pytest.mark.parametrize("bad", [(0,), (1,), (0, 2), (2, 3)])
def test_columns_with_densities_that_are_not_finite(nb, copies, bad):
    """Which copies of a group are near differs by column where a density is not
    finite: the finite columns and the others each equal their single evaluation."""
    g = geometry(copies)
    sigma = 1e-5 * np.random.default_rng(10).standard_normal((4, g.n))
    for k, v in zip(bad, (np.nan, -np.inf)):
        sigma[k, 100 + 300 * k] = v
    p = points(g, 131)
    dp = nb.DevicePanels.from_geometry(g, "cuda:0")
    out = torch.stack(nb.eval_points_multi(dp, dev(sigma), *[dev(p[:, k]) for k in range(3)]), 2).cpu().numpy()
    for k in range(4):
        assert np.isfinite(out[k]).all() == (k not in bad)
        assert np.array_equal(out[k], evaluate(nb, g, sigma[k], p), equal_nan=True), k


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("copies", ["121", "none"])
def test_server_units_give_equal_bits(nb, copies, precision):
    """A launch of few items runs as groups or 16-element runs, one of many as
    whole items: a short request alone, and the same points at the head of one
    that fills several rounds, agree with the session's evaluation."""
    g = geometry(copies)
    if copies == "121":  # a mesh of 7 groups, or the long request takes seconds
        g = gem_cell(k=8, nr=2, n_images=6)
    ses = nb.Session(nb.DevicePanels.from_geometry(g, "cuda:0"), precision=precision)
    srv = nb.Server([ses], hbm_budget=1 << 30)
    p = np.ascontiguousarray(points(g, 64 * 9000 if copies == "none" else 64 * 8300))
    for m in (1, 64, 100, len(p)):
        q = np.ascontiguousarray(p[:m])
        got = srv.wait(srv.submit(0, q))[0]
        ref = torch.stack(ses.eval_points(*[dev(q[:, k]) for k in range(3)]), 1).cpu().numpy()
        assert np.array_equal(np.stack([got[k] for k in ("phi", "ex", "ey", "ez")], 1), ref)
    srv.close()
    ses.close()
