"""The triangular solves on the matrix cores at the edges of their 16-row tiles,
64-row blocks and size classes, with column counts around the eight of a
group, in both factor precisions, against the FP64 oracle.

The operator z I - A0 - exp(-z/2) A2 is sampled on a circle outside A0's
spectrum, so kappa(T(z_j)) is of the order of 10: FP64 solves are within
about n u kappa ~ 1e-12 of the oracle's, and 1e-10 is the parity bar of the
FP64 path; the mixed path stops at a normwise backward error of at most
1e-14, which kappa takes to 1e-13."""
import numpy as np
import pytest

import oracle
import workloads as wl
from workloads import Contour, Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nep():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_1910_11712_amd as P
    P.binding.lib()
    return P


@pytest.mark.parametrize("n,L", [(1, 1), (15, 7), (16, 8), (17, 9), (48, 3), (63, 1), (64, 16), (65, 5), (127, 8),
                                 (128, 2), (129, 17), (255, 8), (256, 9), (257, 1), (449, 12), (511, 8), (512, 15),
                                 (513, 8), (777, 11), (1000, 16), (1023, 1), (1024, 3), (1025, 5), (2049, 3)])
def test_solves_at_tile_edges(nep, n, L):
    rng = np.random.default_rng([n, L])
    A0 = (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2.0 * n)
    A2 = rng.standard_normal((n, n)) / np.sqrt(n)
    prob = Problem("rand", [A0, np.eye(n), A2],
                   [wl.fn_rational([-1.0]), wl.fn_rational([1.0, 0.0]), wl.fn_exp(alpha=-0.5)])
    con = Contour.circle(0.1 + 0.2j, 3.5)
    N, K = 4, 1
    V = wl.probes(n, L, 3)
    So = oracle.ciss_moments(prob, con, N, K, V)
    op = nep.SplitOperator.from_problem(prob)
    for prec in ("fp64", "mixed"):
        S, st = op.moments(con, nep.device_probes(V), N, L, K, prec=prec)
        S = nep.moments_to_numpy(S)
        assert st["n_fallback"] == 0 and st["n_unconverged"] == 0, st
        for p in range(So.shape[0]):
            e = np.linalg.norm(S[p] - So[p]) / np.linalg.norm(So[p])
            assert e <= 1e-10, (prec, p, e)
