"""FP64 inversion on the diagonal of blocks whose entries grow below a panel, by
factors between 1 and the limit of 8 beyond which interchanges take over: the
inverse against numpy's of the block that the GPU assembled.

The limits are per panel.  Tolerance: 64 eps cond(B) of the largest entry, as
for multipliers of order 1 (a growth of up to 8 in one of a few panels costs
less than the factor of 64 allows)."""
import numpy as np
import pytest

from paper_2606_31380_amd import scenarios as sc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_31380_amd import qax  # noqa: E402

DEV = torch.device("cuda", 0)
# bodies without mirror symmetry (one block, inverted as it is), far from resolved
CASES = [(sc.SPIRAL, 0.5, 1, 12, 60.0, qax.QAX_DOUBLE_LAYER), (sc.SPIRAL, 0.5, 2, 10, 30.0, qax.QAX_DOUBLE_LAYER),
         (sc.SPIRAL, 0.5, 1, 12, 120.0, qax.QAX_COMBINED_FIELD), (sc.CONCH, 0.6, 1, 12, 120.0, qax.QAX_COMBINED_FIELD),
         (sc.CONCH, 0.6, 2, 10, 40.0, qax.QAX_SINGLE_LAYER)]


def elimination(A, w=64):
    """The panels' elimination in numpy: the largest part of an entry below a panel,
    multiplier within a diagonal block, and cancellation of a pivot block's determinant."""
    A, n = A.copy(), A.shape[0]
    below = mult = det = 0.0
    for k in range(0, n, w):
        p = slice(k, min(k + w, n))
        D = A[p, p].copy()
        for t in range(0, D.shape[0], 2):
            q = D[t:t + 2, t:t + 2]
            det = max(det, abs(q[0, 0] * q[1, 1] / np.linalg.det(q)))
            m = D[t + 2:, t:t + 2] @ np.linalg.inv(q)
            mult = max(mult, np.abs(m).max(initial=0.0))
            D[t + 2:] -= m @ D[t:t + 2]
        Di = np.linalg.inv(A[p, p])
        G, W = A[:, p] @ Di, A[p].copy()
        g = G[p.stop:]
        below = max(below, np.abs(g.real).max(initial=0.0), np.abs(g.imag).max(initial=0.0))
        A -= G @ W
        A[p] = Di @ W
        A[:, p] = -G
        A[p, p] = Di
    return A, below, mult, det


@pytest.mark.parametrize("shape,a,panels,n_theta,k,form", CASES)
def test_growth_below_the_limit(shape, a, panels, n_theta, k, form):
    b = sc.make_bodies(1)
    b[0]["shape"], b[0]["a"], b[0]["c"], b[0]["n_panels"], b[0]["n_theta"] = shape, a, 1.0, panels, n_theta
    with qax.Problem(sc.Scenario("growth", b, np.array([k]), sc.paper_direction()), formulation=form) as P:
        qax.qax_assemble_self(P.h)
        mats = []
        for inverse in (False, True):
            t = torch.zeros(P.N * P.N, dtype=torch.complex128, device=DEV)
            qax.qax_self_block(P.h, 0, t, inverse=inverse)
            mats.append(t.cpu().numpy().reshape(P.N, P.N))
    B, got = mats
    _, below, mult, det = elimination(B)
    assert 1.0 < below < 8.0 and mult < 4.0 and det < 8.0      # stays on the diagonal, and grows
    want = np.linalg.inv(B)
    assert np.abs(got - want).max() <= 64 * np.finfo(float).eps * np.linalg.cond(B) * np.abs(want).max()
