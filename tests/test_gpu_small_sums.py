"""Sums with several right-hand sides too small to fill the chip split their
sources further: a few hundred nodes (four workgroups if each takes all sources)
take no longer than ten times the pairs, and right, down to one source chunk per
workgroup."""

import numpy as np
import pytest

from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)


def scene(bodies, n_theta):
    b = sc.make_bodies(bodies)
    for i in range(bodies):
        b[i]["shape"], b[i]["a"], b[i]["c"], b[i]["kappa"] = sc.SPHEROID, 0.5, 0.8, 0.2
        b[i]["n_panels"], b[i]["n_theta"] = 1, n_theta
        b[i]["cx"], b[i]["cy"], b[i]["cz"] = 2.4 * (i % 3), 2.4 * (i // 3 % 3), 2.4 * (i // 9)
    return sc.Scenario("small", b, np.array([2.0]), sc.paper_direction())


def density(n, nrhs):
    rng = np.random.default_rng(nrhs)
    return rng.standard_normal((n, nrhs)) + 1j * rng.standard_normal((n, nrhs))


def fastest(P, nrhs):
    mu, out = torch.from_numpy(density(P.N, nrhs).reshape(-1)).to(DEV), P.vec(nrhs)
    ts = []
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            qax.qax_pair_sum(P.h, qax.QAX_FP64, mu, out, nrhs)
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b))
    return min(ts)


def test_fewer_pairs_take_no_longer():
    # 480 and 1536 nodes, 64 right-hand sides: 187 us against 116 with eight source
    # chunks or more per workgroup, 39 against 72 split further
    with qax.Problem(scene(5, 6)) as small, qax.Problem(scene(12, 8)) as large:
        # (a fifth more allowed: a slow host's launches can bound both)
        assert fastest(small, 64) < 1.2 * fastest(large, 64)


@pytest.mark.parametrize("bodies,n_theta", [(2, 4), (3, 6), (5, 6), (12, 8)])    # 4, 9, 15 and 48 source chunks
@pytest.mark.parametrize("nrhs", [2, 8, 33])
def test_split_sums(bodies, n_theta, nrhs):
    """Against one right-hand side at a time: FP64 sums of N terms, FP32 ones to 1e-5 of the column."""
    with qax.Problem(scene(bodies, n_theta)) as P:
        mu = density(P.N, nrhs)
        out, one = P.vec(nrhs), P.vec()
        for prec, tol in ((qax.QAX_FP64, 1e-13), (qax.QAX_MIXED, 1e-5)):
            qax.qax_pair_sum(P.h, prec, torch.from_numpy(mu.reshape(-1)).to(DEV), out, nrhs)
            got = out.cpu().numpy().reshape(P.N, nrhs)
            for r in range(nrhs):
                qax.qax_pair_sum(P.h, qax.QAX_FP64, torch.from_numpy(mu[:, r].copy()).to(DEV), one)
                want = one.cpu().numpy()
                assert np.linalg.norm(got[:, r] - want) <= tol * np.linalg.norm(want), (prec, r)
        # evaluation points and far-field directions
        X = np.random.default_rng(1).standard_normal((40, 3))
        X /= np.linalg.norm(X, axis=1, keepdims=True)
        pts = 40.0 * X
        m = torch.from_numpy(mu.reshape(-1)).to(DEV)
        u, f = (torch.zeros(40 * nrhs, dtype=torch.complex128, device=DEV) for _ in range(2))
        qax.qax_nearfield(P.h, m, pts, u, nrhs)
        qax.qax_farfield(P.h, m, X, f, nrhs)
        u1, f1 = (torch.zeros(40, dtype=torch.complex128, device=DEV) for _ in range(2))
        for r in range(nrhs):
            m = torch.from_numpy(mu[:, r].copy()).to(DEV)
            qax.qax_nearfield(P.h, m, pts, u1)
            qax.qax_farfield(P.h, m, X, f1)
            for a, b in ((u, u1), (f, f1)):
                assert (a.reshape(40, nrhs)[:, r] - b).norm() <= 1e-13 * b.norm(), r
