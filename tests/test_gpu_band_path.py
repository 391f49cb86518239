"""Operators whose terms are all diagonal or narrow-banded (half-width at most
4) are factored, solved and refined over their band.  Edges of that path
against the FP64 oracle and against the dense path (the same operator with one
negligible entry outside every band, which keeps the dense factors): sizes
around the elimination window and the register buffers, every window width,
complex diagonal terms, odd probe counts, explicit points, eigenvalue counts,
exact zero pivots and batches that mix both paths."""
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


CON = Contour.circle(5.05, 0.7)


def _problem(n, lo, up, seed=0, dense_twin=False):
    """T(z) = B0 - z I + exp(-z) B1 + 0.1 D with complex diagonal D; weak
    diagonals in places, so that rows are exchanged."""
    rng = np.random.default_rng([n, lo, up, seed])

    def band(scale):
        A = np.zeros((n, n))
        for k in range(-lo, up + 1):
            i = np.arange(max(0, -k), min(n, n - k))
            A[i, i + k] = scale * rng.standard_normal(len(i))
        return A

    d = np.linspace(1.0, 10.0, n)
    d[rng.random(n) < 0.2] = 5.0
    B0, B1 = band(0.6) + np.diag(d), band(0.2)
    D = np.diag(rng.standard_normal(n) + 1j * rng.standard_normal(n))
    if dense_twin and n > 1:
        B0[0, n - 1] += 1e-30
    fns = [wl.fn_rational([1.0]), wl.fn_rational([-1.0, 0.0]), wl.fn_exp(alpha=-1.0), wl.fn_rational([0.1])]
    return Problem("band", [B0, np.eye(n), B1, D], fns)


def _moments(nep, p, N, L, K, prec, seed=5):
    op = nep.SplitOperator.from_problem(p)
    V = wl.probes(p.n, L, seed)
    S, st = op.moments(CON, nep.device_probes(V), N, L, K, prec=prec)
    return op, V, nep.moments_to_numpy(S), st


def _close(Sg, So, V, tol=1e-10):
    """Relative to the moments, or to the probes where the quadrature sum
    cancels (no eigenvalue inside)."""
    for q in range(So.shape[0]):
        err = np.linalg.norm(Sg[q] - So[q]) / max(np.linalg.norm(So[q]), 1e-2 * np.linalg.norm(V))
        assert err <= tol, (q, err)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("n,lo,up,N,L", [(1, 0, 0, 8, 1), (2, 1, 1, 8, 2), (5, 4, 4, 8, 1), (6, 2, 4, 8, 3),
                                         (33, 1, 1, 32, 5), (64, 1, 1, 66, 3), (65, 2, 1, 32, 8), (66, 3, 0, 32, 8),
                                         (97, 0, 0, 32, 7), (300, 4, 4, 32, 8), (301, 1, 1, 70, 9)])
def test_moments_match_oracle(nep, n, lo, up, N, L, prec):
    p = _problem(n, lo, up)
    op, V, Sg, st = _moments(nep, p, N, L, 2, prec)
    assert st["n_unconverged"] == 0 and st["singular_node"] < 0 and st["min_abs_pivot"] > 0.0, st
    if prec == "mixed":
        assert st["max_rel_residual"] <= 1e-14, st
    _close(Sg, oracle.ciss_moments(p, CON, N, 2, V), V)
    op.close()


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_further_probes_count_and_points(nep, prec):
    n, N, L, K = 130, 64, 4, 2
    p, twin = _problem(n, 2, 1, seed=3), _problem(n, 2, 1, seed=3, dense_twin=True)
    op, _, _, _ = _moments(nep, p, N, L, K, prec)
    opt, _, _, _ = _moments(nep, twin, N, L, K, prec)
    B = nep.binding
    V2 = wl.probes(n, L, 9)
    S2 = torch.empty((2 * K, L, n), dtype=torch.complex128, device="cuda")
    B.nep_ciss_moments_more(op.h, nep.device_probes(V2), S2)
    _close(nep.moments_to_numpy(S2), oracle.ciss_moments(p, CON, N, K, V2), V2)
    c, _, w = B.nep_ciss_count(op.h)
    ct, _, wt = B.nep_ciss_count(opt.h)
    assert c == ct and abs(w - wt) < 1e-3, (c, ct, w, wt)
    z = [4.1 + 0.3j, 6.0 - 0.2j, 5.5 + 1.0j]
    Y = torch.empty((3, L, n), dtype=torch.complex128, device="cuda")
    B.nep_solve_at(op.h, z, nep.device_probes(V2), Y, prec=prec)
    for k, zk in enumerate(z):
        T = sum(complex(f) * A for f, A in zip((1.0, -zk, np.exp(-zk), 0.1), p.mats))
        ref = np.linalg.solve(T, V2)
        got = Y[k].cpu().numpy().T
        assert np.linalg.norm(got - ref) <= 1e-11 * np.linalg.norm(ref), k
    op.close()
    opt.close()


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_zero_pivot_is_reported(nep, prec):
    A = np.diag([2.0, 0.0, 3.0, 1.0])
    A[0, 1] = 1.0  # column 1 is a multiple of column 0: the second pivot is exactly zero
    p = Problem("sing", [A], [wl.fn_rational([1.0])])
    with pytest.raises(nep.NepError) as ei:
        _moments(nep, p, 8, 2, 1, prec)
    assert ei.value.name == "NEP_ERR_SINGULAR"


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_batch_of_both_paths_equals_single_calls(nep, prec, graph):
    N, L, K = 32, 5, 2
    probs = [_problem(200, 1, 1), _problem(90, 2, 2, dense_twin=True), _problem(70, 4, 1),
             _problem(150, 1, 1, dense_twin=True), _problem(3, 1, 1)]
    ops, singles, Vs = [], [], []
    for k, p in enumerate(probs):
        op, V, Sg, _ = _moments(nep, p, N, L, K, prec, seed=k)
        ops.append(op)
        singles.append(Sg)
        Vs.append(nep.device_probes(V))
    Ss = [torch.zeros((2 * K, L, p.n), dtype=torch.complex128, device="cuda") for p in probs]
    B = nep.binding
    b = B.nep_batch_create([op.h for op in ops], [CON] * len(ops), B.opts_struct(N, L, K, prec), Vs, Ss,
                           use_graph=graph)
    for rep in range(3):
        for S in Ss:
            S.zero_()
        torch.cuda.synchronize()
        B.nep_batch_run(b, len(ops))
        for k in range(len(ops)):
            assert np.array_equal(nep.moments_to_numpy(Ss[k]), singles[k]), (rep, k)
    B.nep_batch_destroy(b)
    for op in ops:
        op.close()
