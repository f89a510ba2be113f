"""FP64 sums at phases k r beyond 2^31 / (512 / 2 pi) = 2.6e7, where a 32-bit
count of 512ths of a revolution ends: near fields far off the bodies, pair
sums of bodies many wavelengths apart and far fields of bodies far from the
origin, against extended precision on the library's own nodes.

Tolerance: the kernels form r with a relative error of at most 4 x 2^-53
(differences, squares, inverse root, product), which turns the phase of every term by
k r times that; twice that, plus 1e-13 for the rest, of the sum of the terms' sizes.
The reciprocal sums (one right-hand side) scale the positions by k first and
round the phase again, the far field its three products: 8 and 6 x 2^-53.
"""
import numpy as np
import pytest

from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)
FORMS = {"double": qax.QAX_DOUBLE_LAYER, "combined": qax.QAX_COMBINED_FIELD, "single": qax.QAX_SINGLE_LAYER}
PHASES = [2.5e7, 2.7e7, 1.0e8, 1.0e9]     # the first is below the limit


def spheres(k, centres):
    b = sc.make_bodies(len(centres))
    for i, x in enumerate(centres):
        sc._fill(b[i], sc.SPHERE, 0.5, 0.5, 0.0, 1, 8, 0.3 * i, 0.1, x)
    return sc.Scenario("phase", b, np.array([k]), sc.paper_direction())


def nodes(P):
    pos = torch.zeros((P.N, 3), dtype=torch.float64, device=DEV)
    aw = torch.zeros_like(pos)
    qax.qax_nodes(P.h, pos, aw)
    return pos.cpu().numpy(), aw.cpu().numpy()


def reference(x, y, aw, mu, k, form, skip=None):
    """The sums and the sums of the terms' sizes in extended precision."""
    ld = np.longdouble
    two_pi = 2 * ld("3.14159265358979323846264338327950288")
    d = y[None].astype(ld) - x[:, None].astype(ld)
    r = np.sqrt((d * d).sum(-1))
    if skip is not None:
        r = np.where(skip, ld(1), r)
    ph = ld(k) * r
    ph = (ph - two_pi * np.round(ph / two_pi)).astype(float)
    e = np.exp(1j * ph) / (4 * np.pi * r.astype(float))
    w = np.linalg.norm(aw, axis=1)[None]
    if form == "single":
        f = w * e
    else:
        f = (1j * k / r - 1 / r ** 2).astype(complex) * (d * aw[None].astype(ld)).sum(-1).astype(float) * e
        if form == "combined":
            f = f - 1j * k * w * e
    if skip is not None:
        f = np.where(skip, 0.0, f)
    return f @ mu, np.abs(f) @ np.abs(mu)


def densities(n, nrhs):
    rng = np.random.default_rng(4)
    return rng.standard_normal((n, nrhs)) + 1j * rng.standard_normal((n, nrhs))


def dev(v):
    return torch.from_numpy(np.ascontiguousarray(v.ravel())).to(DEV)


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("kr", PHASES)
def test_near_field_far_off(kr, form):
    k = 4.0
    u = np.random.default_rng(2).standard_normal((40, 3))
    x = u / np.linalg.norm(u, axis=1)[:, None] * (kr / k)
    with qax.Problem(spheres(k, [(0.0, 0.0, 0.0), (3.0, 0.0, 0.0)]), formulation=FORMS[form]) as P:
        y, aw = nodes(P)
        for nrhs in (1, 8):
            mu = densities(P.N, nrhs)
            out = torch.zeros(x.shape[0] * nrhs, dtype=torch.complex128, device=DEV)
            qax.qax_nearfield(P.h, dev(mu), x, out, nrhs)
            want, size = reference(x, y, aw, mu, k, form)
            tol = (8 * 2.0 ** -53 * kr * 1.01 + 1e-13) * size
            assert (np.abs(out.cpu().numpy().reshape(-1, nrhs) - want) <= tol).all()


def pair_sums(kr, form, counts, roundings=4):
    k = 1.0e6
    with qax.Problem(spheres(k, [(0.0, 0.0, 0.0), (0.6 * kr / k, 0.8 * kr / k, 0.0)]), formulation=FORMS[form]) as P:
        y, aw = nodes(P)
        body = np.arange(P.N) >= P.offsets[1]
        for nrhs in counts:
            mu = densities(P.N, nrhs)
            out = P.vec(nrhs)
            qax.qax_pair_sum(P.h, qax.QAX_FP64, dev(mu), out, nrhs)
            want, size = reference(y, y, aw, mu, k, form, skip=body[:, None] == body[None])
            tol = (2 * roundings * 2.0 ** -53 * kr * 1.1 + 1e-13) * size
            assert (np.abs(out.cpu().numpy().reshape(-1, nrhs) - want) <= tol).all()


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("kr", PHASES)
def test_pair_sum_several_rhs(kr, form):
    pair_sums(kr, form, (2, 4, 9))


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("kr", PHASES)
def test_pair_sum_one_rhs(kr, form):
    pair_sums(kr, form, (1,), roundings=8)


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("kr", PHASES)
def test_far_field(kr, form):
    k, ld = 4.0, np.longdouble
    c = np.array([0.48, 0.6, 0.64]) * kr / k
    rng = np.random.default_rng(3)
    x = rng.standard_normal((40, 3))
    x /= np.linalg.norm(x, axis=1)[:, None]
    x = np.concatenate([x, -x[:10], [c / np.linalg.norm(c)]])
    with qax.Problem(spheres(k, [tuple(c), tuple(c + 3.0)]), formulation=FORMS[form]) as P:
        y, aw = nodes(P)
        ph = -ld(k) * (x.astype(ld) @ y.astype(ld).T)
        two_pi = 2 * ld("3.14159265358979323846264338327950288")
        e = np.exp(1j * (ph - two_pi * np.round(ph / two_pi)).astype(float)) / (4 * np.pi)
        w = np.linalg.norm(aw, axis=1)[None]
        f = e * (w if form == "single" else -1j * k * (x @ aw.T) - (1j * k * w if form == "combined" else 0.0))
        for nrhs in (1, 8):
            mu = densities(P.N, nrhs)
            out = torch.zeros(x.shape[0] * nrhs, dtype=torch.complex128, device=DEV)
            qax.qax_farfield(P.h, dev(mu), x, out, nrhs)
            tol = (12 * 2.0 ** -53 * kr * 1.01 + 1e-13) * (np.abs(f) @ np.abs(mu))
            assert (np.abs(out.cpu().numpy().reshape(-1, nrhs) - f @ mu) <= tol).all()
