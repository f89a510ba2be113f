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
