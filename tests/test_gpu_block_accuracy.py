"""The FP64 block product with two and three right-hand sides adds its rows in
64 lanes and then a tree, as with one: a row of order n is a chain of
L = 2 ceil(n / 64) products, six sums across the lanes and the store's one.
The matrix cores' single chain of 2 n products would lift the residual that a
badly conditioned solve can reach.

Bound: a rounding is off by at most u = 2^-53 of its partial sum, u / sqrt(3) in
the mean square; independent roundings of partial sums no larger in the mean
than the row's sum add to u sqrt((L + 7) / 3) of it, over all rows together.
The reference is summed in extended precision.
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


@pytest.mark.parametrize("panels,n_theta", [(1, 8), (2, 10), (2, 32), (2, 64)])      # orders 128, 320, 1024, 2048
def test_chain_of_64_lanes(panels, n_theta):
    b = sc.make_bodies(1)
    b[0]["shape"], b[0]["a"], b[0]["c"], b[0]["kappa"] = sc.SPHEROID, 0.5, 1.0, 0.25
    b[0]["n_panels"], b[0]["n_theta"] = panels, n_theta
    with qax.Problem(sc.Scenario("one", b, np.array([3.0]), sc.paper_direction())) as P:
        qax.qax_assemble_self(P.h)
        n = P.N
        bound = 2.0 ** -53 * np.sqrt((2 * -(-n // 64) + 7) / 3.0)
        for inverse in (0, 1):
            t = torch.zeros(n * n, dtype=torch.complex128, device=DEV)
            qax.qax_self_block(P.h, 0, t, inverse=bool(inverse))
            M = t.cpu().numpy().reshape(n, n)
            Mr, Mi = M.real.astype(np.longdouble), M.imag.astype(np.longdouble)
            for nrhs in (2, 3):
                rng = np.random.default_rng(nrhs)
                v = rng.standard_normal((n, nrhs)) + 1j * rng.standard_normal((n, nrhs))
                vr, vi = v.real.astype(np.longdouble), v.imag.astype(np.longdouble)
                wr, wi = Mr @ vr - Mi @ vi, Mr @ vi + Mi @ vr
                out = P.vec(nrhs)
                qax.qax_block_apply(P.h, inverse, qax.QAX_FP64, torch.from_numpy(v.reshape(-1)).to(DEV), out, nrhs)
                o = out.cpu().numpy().reshape(n, nrhs)
                err = np.sqrt(float(((o.real - wr) ** 2 + (o.imag - wi) ** 2).sum() / (wr ** 2 + wi ** 2).sum()))
                assert err <= bound, (inverse, nrhs, err, bound)


@pytest.mark.parametrize("bodies", [400, 600])       # 25600 rows of order 64, and the 38400 that take the matrix cores
def test_many_short_fp32_blocks(bodies):
    """Both routes of the FP32 product against one right-hand side at a time: sums of the same
    rounded entries in FP64, 2 n eps |M| |v| off either way (rows' sums of |M| |v| by Cauchy and Schwarz)."""
    b = sc.make_bodies(bodies)
    for i in range(bodies):
        b[i]["shape"], b[i]["a"], b[i]["c"], b[i]["kappa"] = sc.SPHEROID, 0.5, 0.8, 0.2
        b[i]["n_panels"], b[i]["n_theta"] = 1, 4
        b[i]["cx"], b[i]["cy"] = 3.0 * (i % 25), 3.0 * (i // 25)
    with qax.Problem(sc.Scenario("short", b, np.array([2.0]), sc.paper_direction())) as P:
        qax.qax_assemble_self(P.h)
        n = P.N // bodies
        t = torch.zeros(n * n, dtype=torch.complex128, device=DEV)
        for inverse in (0, 1):
            qax.qax_self_block(P.h, 0, t, inverse=bool(inverse))
            rows = np.linalg.norm(t.cpu().numpy().reshape(n, n), axis=1).max()
            for nrhs in (2, 3):
                rng = np.random.default_rng(nrhs)
                v = rng.standard_normal((P.N, nrhs)) + 1j * rng.standard_normal((P.N, nrhs))
                out, one = P.vec(nrhs), P.vec()
                qax.qax_block_apply(P.h, inverse, qax.QAX_MIXED, torch.from_numpy(v.reshape(-1)).to(DEV), out, nrhs)
                got = out.cpu().numpy().reshape(bodies, n, nrhs)
                for r in range(nrhs):
                    qax.qax_block_apply(P.h, inverse, qax.QAX_MIXED, torch.from_numpy(v[:, r].copy()).to(DEV), one)
                    w = np.linalg.norm(v[:, r].reshape(bodies, n), axis=1)
                    bound = 4 * n * np.finfo(float).eps * rows * w
                    # the inverse of mirror-symmetric bodies goes through reduced blocks of other roundings
                    if inverse:
                        bound = bound + 4 * np.sqrt(n) * 2.0 ** -24 * rows * w
                    diff = np.abs(got[:, :, r] - one.cpu().numpy().reshape(bodies, n)).max(axis=1)
                    assert (diff <= bound).all(), (inverse, nrhs, r)
