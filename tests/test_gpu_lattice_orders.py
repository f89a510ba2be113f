"""The array apply with one right-hand side at block orders on both sides of
its products' splits (64 to 512: two rows per group of 16 or 32 lanes up to
256, one row per wavefront beyond) and at periods with every remainder of four
outputs, against the direct pair sum (FP64 1e-12, FP32 tables 1e-5, as the
array apply's other tests)."""

import numpy as np
import pytest

from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("dims", [(1, 2, 6), (5, 1, 2), (3, 4, 1)])
@pytest.mark.parametrize("npan,nth", [(1, 4), (1, 6), (1, 8), (1, 16), (1, 18), (2, 16)])
def test_orders_and_periods(dims, npan, nth):
    n = dims[0] * dims[1] * dims[2]
    b = sc.make_bodies(n)
    for i, (x, y, z) in enumerate(np.ndindex(*dims)):
        b[i]["shape"], b[i]["a"], b[i]["c"], b[i]["kappa"] = sc.SPHEROID, 0.5, 0.9, 0.2
        b[i]["n_panels"], b[i]["n_theta"], b[i]["theta1"] = npan, nth, 0.4
        b[i]["cx"], b[i]["cy"], b[i]["cz"] = 2.6 * x, 3.0 * y, 2.8 * z
    s = sc.Scenario("orders", b, np.array([1.5]), sc.paper_direction())
    rng = np.random.default_rng(nth)
    with qax.Problem(s) as P:
        mu = torch.from_numpy(rng.standard_normal(P.N) + 1j * rng.standard_normal(P.N)).to(DEV)
        want, got, got32 = P.vec(), P.vec(), P.vec()
        qax.qax_pair_sum(P.h, qax.QAX_FP64, mu, want)
        assert qax.qax_lattice(P.h) == dims
        qax.qax_pair_sum(P.h, qax.QAX_FP64, mu, got)
        qax.qax_pair_sum(P.h, qax.QAX_MIXED, mu, got32)
    assert (got - want).norm() < 1e-12 * want.norm()
    assert (got32 - want).norm() < 1e-5 * want.norm()
