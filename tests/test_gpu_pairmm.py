"""Pair sums with several right-hand sides on the matrix cores.

Every tile of right-hand sides (the edges of 16, 32 and 64), each formulation,
problems of unequal wavenumbers and bodies that leave partial target blocks,
against the oracle; targets near a body; density scales and non-finite
densities.

Bounds.  FP32: the phase carries FP32 rounding of the distance difference
(up to about 5e-7 of a row's sum), the split factors 2^-22, so 2e-6 in the
2-norm and 4e-6 of the largest entry.  Near targets: r^2 is formed against
|D|^2, so its relative error is (D / r)^2 2^-24, 36 x 6e-8 at D = 0.6 and
r = 0.1, up to 2.5 of which enters 1 / r^2 and the factor (i - 1 / kr): 6e-6.
FP64: 1e-12 of the norm and of the largest entry (coordinates of size 20 in
phases k r of size 100 and sums of a few thousand terms, each 2^-53).
"""
import numpy as np
import pytest

from oracle import geometry as geo
from oracle import pairsum as opair
from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)
FORMS = {"double": qax.QAX_DOUBLE_LAYER, "combined": qax.QAX_COMBINED_FIELD, "single": qax.QAX_SINGLE_LAYER}


def scenario():
    # two problems; bodies of 16 x 10 = 160, 16 x 6 = 96, 32 x 12 = 384 ... nodes
    s = sc.random_mixed(n_bodies=7, side=10.0, k=3.0, seed=11)
    b = s.bodies.copy()
    b["n_theta"] = [10, 6, 12, 18, 4, 22, 14]
    b["problem"][4:] = 1
    return sc.Scenario("mm", b, np.array([3.0, 6.5]), s.dirs)


def densities(n, nrhs, seed=3):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((n, nrhs)) + 1j * rng.standard_normal((n, nrhs))


def oracle_sum(s, mu, form):
    d = geo.discretize(s)
    if form == "combined":               # eta = k of each problem
        out = np.zeros_like(mu)
        for p, k in enumerate(s.k):
            tg = np.nonzero(d.problem == p)[0]
            out[tg] = opair.pair_sum(d, s.k, mu, targets=tg, eta=float(k))
        return out
    return opair.pair_sum(d, s.k, mu, single=form == "single")


def run(P, prec, mu):
    nrhs = mu.shape[1]
    out = P.vec(nrhs)
    qax.qax_pair_sum(P.h, prec, torch.from_numpy(np.ascontiguousarray(mu.ravel())).to(DEV), out, nrhs)
    return out.cpu().numpy().reshape(-1, nrhs)


def close(got, want, norm, big):
    assert np.linalg.norm(got - want) < norm * np.linalg.norm(want)
    assert np.abs(got - want).max() < big * np.abs(want).max()


@pytest.mark.parametrize("form", sorted(FORMS))
def test_every_tile_of_right_hand_sides(form):
    s = scenario()
    mu = densities(s.n_unknowns(), 70)
    want = oracle_sum(s, mu, form)
    with qax.Problem(s, formulation=FORMS[form]) as P:
        for nrhs in (2, 16, 17, 32, 33, 64, 65, 70):
            close(run(P, qax.QAX_MIXED, mu[:, :nrhs]), want[:, :nrhs], 2e-6, 4e-6)
        for nrhs in (2, 3, 4, 5, 8, 9, 16, 17, 24, 25, 32, 33, 70):
            close(run(P, qax.QAX_FP64, mu[:, :nrhs]), want[:, :nrhs], 1e-12, 1e-12)


@pytest.mark.parametrize("nrhs", [3, 20, 40])
def test_near_targets(nrhs):
    # two spheres of radius 0.5 that all but touch (gap 0.1), a third far off
    b = sc.make_bodies(3)
    for i, x in enumerate((0.0, 1.1, 9.0)):
        sc._fill(b[i], sc.SPHERE, 0.5, 0.5, 0.0, 2, 24, 0.3 * i, 0.1, (x, 0.0, 0.0))
    s = sc.Scenario("near", b, np.array([2.0]), sc.paper_direction())
    mu = densities(s.n_unknowns(), nrhs)
    want = oracle_sum(s, mu, "double")
    with qax.Problem(s) as P:
        close(run(P, qax.QAX_MIXED, mu), want, 6e-6, 6e-6)
        close(run(P, qax.QAX_FP64, mu), want, 1e-12, 1e-12)


@pytest.mark.parametrize("nrhs", [5, 30, 50])
def test_density_scales(nrhs):
    # powers of two per column pass through exactly; a zero column stays zero;
    # a column that is not finite spoils no other column
    s = scenario()
    mu = densities(s.n_unknowns(), nrhs)
    with qax.Problem(s) as P:
        plain = run(P, qax.QAX_MIXED, mu)
        f = 2.0 ** np.linspace(-200, 200, nrhs).round()
        f[2] = 0.0
        assert np.array_equal(run(P, qax.QAX_MIXED, mu * f), plain * f)
        bad = mu.copy()
        bad[5, 1], bad[9, 3] = np.inf, np.nan
        got = run(P, qax.QAX_MIXED, bad)
        keep = [c for c in range(nrhs) if c not in (1, 3)]
        assert np.array_equal(got[:, keep], plain[:, keep])
        seen = geo.discretize(s).body != 0      # targets off the body of the bad nodes, in its problem
        seen &= geo.discretize(s).problem == 0
        assert not np.isfinite(got[seen][:, [1, 3]]).any()


def test_small_wavenumber_falls_back():
    # k = 0 and a k far below the kernels' range keep the per-target kernel
    s = sc.tiny(n_bodies=3, n_panels=1, n_theta=8, k=1e-9, spacing=2.5)
    for k in (0.0, 1e-9):
        t = sc.Scenario("k", s.bodies, np.array([k]), s.dirs)
        mu = densities(t.n_unknowns(), 4)
        with qax.Problem(t) as P:
            close(run(P, qax.QAX_MIXED, mu), oracle_sum(t, mu, "double"), 2e-6, 4e-6)
            close(run(P, qax.QAX_FP64, mu), oracle_sum(t, mu, "double"), 1e-12, 1e-12)


def field_reference(s, x, mu, problem, form, far):
    """Near field at x, or far field in directions x, of one problem in plain numpy."""
    d = geo.discretize(s)
    m = d.problem == problem
    k, y, aw, v = float(s.k[problem]), d.pos[m], d.aw[m], mu[m]
    w = np.linalg.norm(aw, axis=1)
    if far:
        e = np.exp(-1j * k * (x @ y.T))
        f = w if form == "single" else -1j * k * (x @ aw.T) - (1j * k * w if form == "combined" else 0.0)
        return (e * f) @ v / (4 * np.pi)
    dx = y[None] - x[:, None]
    r = np.sqrt((dx * dx).sum(-1))
    e = np.exp(1j * k * r) / (4 * np.pi * r)
    f = w if form == "single" else (1j * k / r - 1 / r ** 2) * np.einsum("ijc,jc->ij", dx, aw)
    if form == "combined":
        f = f - 1j * k * w
    return (e * f) @ v


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("points", [1, 31, 65, 200])
def test_fields_every_tile(form, points):
    # odd numbers of targets (partial tiles, clamped rows), tiles of
    # right-hand sides; the far field with no, some and only paired directions
    s = scenario()
    mu = densities(s.n_unknowns(), 33)
    rng = np.random.default_rng(points)
    near = rng.uniform(-9.0, 9.0, (points, 3)) + np.array([0.0, 0.0, 25.0])
    dirs = rng.standard_normal((points, 3))
    dirs /= np.linalg.norm(dirs, axis=1)[:, None]
    with qax.Problem(s, formulation=FORMS[form]) as P:
        for nrhs in (1, 2, 4, 7, 9, 33):
            v = torch.from_numpy(np.ascontiguousarray(mu[:, :nrhs].ravel())).to(DEV)
            for p in range(2):
                u = torch.zeros(points * nrhs, dtype=torch.complex128, device=DEV)
                qax.qax_nearfield(P.h, v, near, u, nrhs, problem=p)
                close(u.cpu().numpy().reshape(points, nrhs),
                      field_reference(s, near, mu[:, :nrhs], p, form, False), 1e-12, 1e-12)
            for x in (dirs, np.concatenate([dirs, -dirs[::2]]), np.concatenate([-dirs, dirs, dirs])):
                n = x.shape[0]
                u = torch.zeros(2 * n * nrhs, dtype=torch.complex128, device=DEV)
                qax.qax_farfield(P.h, v, x, u, nrhs)
                got = u.cpu().numpy().reshape(2, n, nrhs)
                un = torch.zeros_like(u)
                qax.qax_farfield_noalloc(P.h, v, torch.from_numpy(x).to(DEV), un, nrhs)
                gn = un.cpu().numpy().reshape(2, n, nrhs)
                for p in range(2):
                    want = field_reference(s, x, mu[:, :nrhs], p, form, True)
                    close(got[p], want, 1e-12, 1e-12)
                    close(gn[p], want, 1e-12, 1e-12)
