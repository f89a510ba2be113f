"""Self-block rows at the azimuth counts and wavenumbers where the assembly
changes its ways: modes |m| <= N + 1 in half a wavefront (N + 1 < 32) or the
whole of it, the smallest and largest n_theta, transforms of 16 and 64 slots
or the plain inverse, few and many modes of the smooth factors (k = 0 none,
k = 9 most), forward and backward recurrences (rows next to a panel's
end and in its middle), one panel (the 64-node outer rule) and two.

Tolerance: the self-block entries' 1e-12 of the block's largest entry.
"""

import numpy as np
import pytest

from oracle import geometry as geo
from oracle import selfblock as oself
from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("npan,nth,k", [(1, 4, 2.0), (2, 16, 0.0), (2, 30, 9.0), (1, 60, 5.0), (2, 62, 9.0),
                                        (2, 64, 0.01)])
def test_rows_match_oracle(npan, nth, k):
    b = sc.make_bodies(2)
    for i in range(2):
        b[i]["shape"], b[i]["a"], b[i]["c"], b[i]["kappa"] = sc.SPHEROID, 0.5, 1.0, 0.25
        b[i]["n_panels"], b[i]["n_theta"], b[i]["cx"] = npan, nth, 4.0 * i
    s = sc.Scenario("assembly", b, np.array([k]), sc.paper_direction())
    body = geo.discretize(s).bodies[0]
    n = body.n
    rows = np.unique([nth // 4, 7 * nth + nth // 2, (16 * npan // 2 - 1) * nth + 1])
    want = oself.self_block(body, k, rows=rows)
    with qax.Problem(s) as P:
        qax.qax_assemble_self(P.h)
        t = torch.zeros(n * n, dtype=torch.complex128, device=DEV)
        qax.qax_self_block(P.h, 0, t)
        got = t.cpu().numpy().reshape(n, n)[rows]
    assert np.abs(got - want).max() < 1e-12 * np.abs(want).max()
