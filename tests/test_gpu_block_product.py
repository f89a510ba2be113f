"""The block-diagonal product with several right-hand sides at both sides of
its splits (8, 16, 24 and 32 right-hand sides a pass, more in several), blocks
of different orders in one launch (64 up, a last tile of 32 rows), against
numpy on the blocks the GPU assembled.

Tolerances: FP64 sums of n terms, 4 n eps |M| |v|; the FP32 matrices round each
entry by 2^-24 of itself once more, sums in FP64.
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
SIZES = [(1, 4), (1, 6), (2, 10), (1, 4), (2, 24)]     # orders 64, 96, 320, 64, 768


@pytest.fixture(scope="module")
def handle():
    b = sc.make_bodies(len(SIZES))
    for i, (npan, nth) in enumerate(SIZES):
        b[i]["shape"], b[i]["a"], b[i]["c"], b[i]["kappa"] = sc.SPHEROID, 0.5, 0.8 + 0.05 * i, 0.2
        b[i]["n_panels"], b[i]["n_theta"], b[i]["cx"] = npan, nth, 3.0 * i
    s = sc.Scenario("product", b, np.array([2.0]), sc.paper_direction())
    with qax.Problem(s) as P:
        qax.qax_assemble_self(P.h)
        off = [int(o) for o in P.offsets]
        mats = []
        for i in range(len(SIZES)):
            n = off[i + 1] - off[i]
            pair = []
            for inverse in (False, True):
                t = torch.zeros(n * n, dtype=torch.complex128, device=DEV)
                qax.qax_self_block(P.h, i, t, inverse=inverse)
                pair.append(t.cpu().numpy().reshape(n, n))
            mats.append(pair)
        yield P, off, mats


@pytest.mark.parametrize("nrhs", [2, 3, 8, 9, 17, 25, 33, 40, 64])
@pytest.mark.parametrize("inverse", [0, 1])
def test_product(handle, nrhs, inverse):
    P, off, mats = handle
    rng = np.random.default_rng(nrhs)
    v = rng.standard_normal((P.N, nrhs)) + 1j * rng.standard_normal((P.N, nrhs))
    vt = torch.from_numpy(v.reshape(-1)).to(DEV)
    eps = np.finfo(float).eps
    for prec, rounding in ((qax.QAX_FP64, 0.0), (qax.QAX_MIXED, 2.0 ** -24)):
        out = P.vec(nrhs)
        qax.qax_block_apply(P.h, inverse, prec, vt, out, nrhs)
        got = out.cpu().numpy().reshape(P.N, nrhs)
        for i, pair in enumerate(mats):
            sl = slice(off[i], off[i + 1])
            M, n = pair[inverse], off[i + 1] - off[i]
            bound = (rounding + 4 * n * eps) * (np.abs(M) @ np.abs(v[sl]))
            assert (np.abs(got[sl] - M @ v[sl]) <= bound).all(), (i, prec)
