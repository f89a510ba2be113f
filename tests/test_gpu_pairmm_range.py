"""Range of the FP32 pair sum with several right-hand sides, whose factors are
split in two FP16 parts: bodies far apart in radii at small k r, densities that
differ between bodies by more than FP16's range, values that are not finite.
Counts of right-hand sides 3, 20 and 40 take the three kernels (16, 32, 64 a tile).

Bound of every row and column, of the sum of the sizes of its terms: an entry of the
kernel matrix takes about ten FP32 roundings (2^-24 each) and the hardware's sine
and cosine, the split 2^-22 a factor, 1e-6 together; 2e-6 where the phases reach
k r = 50 (the rounding of the distance differences).
"""
import numpy as np
import pytest

from oracle import geometry as geo
from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)
FORMS = {"double": qax.QAX_DOUBLE_LAYER, "combined": qax.QAX_COMBINED_FIELD, "single": qax.QAX_SINGLE_LAYER}
COUNTS = (3, 20, 40)


def spheres(k, specs):
    """specs: (radius, azimuths, centre) per sphere."""
    b = sc.make_bodies(len(specs))
    for i, (a, nth, x) in enumerate(specs):
        sc._fill(b[i], sc.SPHERE, a, a, 0.0, 1, nth, 0.3 * i, 0.1, x)
    return sc.Scenario("range", b, np.array([k]), sc.paper_direction())


def densities(n, nrhs):
    rng = np.random.default_rng(6)
    return rng.standard_normal((n, nrhs)) + 1j * rng.standard_normal((n, nrhs))


def matrix(s, form="double"):
    """The inter-body kernel matrix (zero within a body), in plain numpy."""
    d, k = geo.discretize(s), float(s.k[0])
    e = d.pos[None] - d.pos[:, None]
    same = d.body[:, None] == d.body[None]
    r = np.where(same, 1.0, np.sqrt((e * e).sum(-1)))
    w = np.linalg.norm(d.aw, axis=1)[None]
    f = w if form == "single" else (1j * k / r - 1 / r ** 2) * (e * d.aw[None]).sum(-1)
    if form == "combined":
        f = f - 1j * k * w
    return np.where(same, 0.0, f * np.exp(1j * k * r) / (4 * np.pi * r)), d


def run(P, mu):
    out = P.vec(mu.shape[1])
    qax.qax_pair_sum(P.h, qax.QAX_MIXED, torch.from_numpy(np.ascontiguousarray(mu.ravel())).to(DEV), out, mu.shape[1])
    return out.cpu().numpy().reshape(mu.shape)


def close(got, K, mu, tol, rows=slice(None)):
    err, size = np.abs(got - K @ mu)[rows], (np.abs(K) @ np.abs(mu))[rows]
    assert (err <= tol * size).all(), (err / np.maximum(size, 1e-300)).max()


@pytest.mark.parametrize("nrhs", COUNTS)
@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("dist,k", [(300.0, 0.01), (1e3, 0.01), (1e3, 1e-3), (1e4, 1e-3), (1e4, 1e-4), (1e5, 1e-6)])
def test_bodies_far_apart(dist, k, form, nrhs):
    # two a few radii apart, one far off: targets of every scale in a tile's bodies
    s = spheres(k, [(1.0, 20, (0.0, 0.0, 0.0)), (0.5, 14, (0.8 * dist, 0.0, 0.6 * dist)), (0.7, 10, (3.0, 1.0, 0.0))])
    mu = densities(s.n_unknowns(), nrhs)
    K, d = matrix(s, form)
    with qax.Problem(s, formulation=FORMS[form]) as P:
        close(run(P, mu), K, mu, 1e-6)
        for b in range(3):                  # one body's sources at a time
            one = np.where((d.body == b)[:, None], mu, 0.0)
            close(run(P, one), K, one, 1e-6)


@pytest.mark.parametrize("nrhs", COUNTS)
@pytest.mark.parametrize("span", [60, 450])
def test_densities_apart_between_bodies(span, nrhs):
    # 2^-span ... 2^span from body to body and per column: rows that see the small ones only
    s = spheres(3.0, [(0.5, 12, (0.0, 0.0, 0.0)), (0.5, 8, (2.0, 0.0, 0.0)), (0.4, 10, (0.0, 9.0, 0.0))])
    K, d = matrix(s)
    mu = densities(s.n_unknowns(), nrhs)
    e = np.random.default_rng(1).integers(-span, span + 1, (3, nrhs))
    mu = mu * (2.0 ** e)[d.body]
    with qax.Problem(s) as P:
        close(run(P, mu), K, mu, 2e-6)
        for keep in ((0, 1), (1, 2), (0, 2)):      # two bodies: each sees the other alone
            two = np.where(np.isin(d.body, keep)[:, None], mu, 0.0)
            close(run(P, two), K, two, 2e-6)


@pytest.mark.parametrize("nrhs", COUNTS)
@pytest.mark.parametrize("bad", [np.inf, np.nan, complex(1.0, -np.inf)])
def test_nodes_of_a_bad_density_body_keep_their_sums(bad, nrhs):
    # a density that is not finite reaches every row of the other bodies and
    # none of its own body's
    s = spheres(3.0, [(1.0, 12, (0.0, 0.0, 0.0)), (1.0, 8, (3.0, 0.0, 0.0)), (0.8, 10, (0.0, 6.0, 0.0))])
    K, d = matrix(s)
    mu = densities(s.n_unknowns(), nrhs)
    own = d.body == 1
    spoilt = mu.copy()
    spoilt[np.nonzero(own)[0][7], 1] = bad
    with qax.Problem(s) as P:
        got = run(P, spoilt)
    close(got, K, mu, 2e-6, own)
    keep = [c for c in range(nrhs) if c != 1]
    close(got[:, keep], K, mu[:, keep], 2e-6)
    assert not np.isfinite(got[~own][:, 1]).any()
