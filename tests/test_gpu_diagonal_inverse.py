"""FP64 inversion of the self blocks by elimination on the diagonal, in panels
of 64 columns, and its return to interchanges: the inverse against numpy's of
the block that the GPU assembled.

Tolerance: elimination with multipliers of order 1 inverts B to a small
multiple of eps cond(B) |B^-1|; the factor is taken as 64.
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
PEANUT = (sc.PEANUT, 0.5, 0.3, 0.2)
SPHERE = (sc.SPHERE, 0.5, 0.5, 0.0)
SPHEROID = (sc.SPHEROID, 0.5, 1.0, 0.25)
CONCH = (sc.CONCH, 0.6, 1.0, 0.0)
SPIRAL = (sc.SPIRAL, 0.5, 1.0, 0.0)
QUASI = (sc.QUASI_ELLIPSOID, 0.5, 1.0, 0.0)

# orders inverted: (n_s / 2)(N + 1), (n_s / 2)(N - 1) of mirror-symmetric
# bodies, n_s 2 N of the others (n_s = 16 panels, 2 N azimuths)
CASES = {
    "below one panel": ([PEANUT + (1, 0, 4)], 2.0, qax.QAX_DOUBLE_LAYER),              # 24, 8
    "one panel exactly, 48": ([PEANUT + (1, 0, 14)], 2.0, qax.QAX_DOUBLE_LAYER),       # 64, 48
    "one panel and 8": ([SPHEROID + (1, 0, 16)], 3.0, qax.QAX_COMBINED_FIELD),         # 72, 56
    "one panel and 32, plain": ([SPIRAL + (1, 0, 6)], 2.0, qax.QAX_DOUBLE_LAYER),      # 96
    "panels exactly, plain": ([CONCH + (2, 0, 18)], 2.0, qax.QAX_COMBINED_FIELD),      # 576
    "orders apart in one batch": ([SPHERE + (1, 0, 6), PEANUT + (2, 1, 22), CONCH + (1, 0, 4), SPIRAL + (2, 0, 12)],
                                  3.0, qax.QAX_DOUBLE_LAYER),                       # 16 .. 384
    "unresolved": ([SPHERE + (2, 0, 16)], 20.0, qax.QAX_DOUBLE_LAYER),
    # far from resolved: three of the spheroid's four reduced blocks, some of
    # the quasi-ellipsoid's and the plain blocks of order 96 have multipliers
    # of 6 to 80, the others pass
    "some of each batch: interchanges": ([SPHEROID + (1, 0, 12), PEANUT + (1, 0, 12), QUASI + (1, 0, 16),
                                          SPHERE + (1, 0, 8), CONCH + (1, 0, 6), CONCH + (2, 0, 18),
                                          SPIRAL + (1, 0, 6)], 120.0, qax.QAX_DOUBLE_LAYER),
    "single layer": ([PEANUT + (2, 0, 16), CONCH + (1, 0, 8)], 3.0, qax.QAX_SINGLE_LAYER),
}


@pytest.mark.parametrize("name", list(CASES))
def test_inverse_matches_numpy(name):
    specs, k, form = CASES[name]
    b = sc.make_bodies(len(specs))
    for i, (shape, a, c, kap, npan, nref, nth) in enumerate(specs):
        b[i]["shape"], b[i]["a"], b[i]["c"], b[i]["kappa"] = shape, a, c, kap
        b[i]["n_panels"], b[i]["n_ref"], b[i]["n_theta"] = npan, nref, nth
        b[i]["theta1"], b[i]["theta2"], b[i]["cx"] = 0.4 * i, 0.7, 4.0 * i
    s = sc.Scenario("diagonal", b, np.array([k]), sc.paper_direction())
    with qax.Problem(s, formulation=form) as P:
        qax.qax_assemble_self(P.h)
        off = [int(o) for o in P.offsets]
        for i in range(len(specs)):
            n = off[i + 1] - off[i]
            mats = []
            for inverse in (False, True):
                t = torch.zeros(n * n, dtype=torch.complex128, device=DEV)
                qax.qax_self_block(P.h, i, t, inverse=inverse)
                mats.append(t.cpu().numpy().reshape(n, n))
            B, Bi = mats
            ref = np.linalg.inv(B)
            tol = 64 * np.finfo(float).eps * np.linalg.cond(B)
            assert np.abs(Bi - ref).max() <= tol * np.abs(ref).max(), (i, n)
