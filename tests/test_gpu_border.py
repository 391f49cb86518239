"""Operators of diagonal, banded (half-width 5 to 32) and low-rank terms: the
mixed path factors them as a bordered block-tridiagonal matrix and refines in
FP64.  Edges of that path (one to four chunks, ragged last block, no low-rank
term, ranks around the 32-column blocks, odd probe counts) against the FP64
oracle; further probes, counts and points against the dense path; a singular
chunk of a nonsingular matrix; batches against single calls."""
import numpy as np
import pytest
import scipy.linalg

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


def _problem(n, w, ranks, seed=0, dense_twin=False):
    """T(z) = B0 - z I + exp(-z) B1 + sum_k c_k(z) U_k V_k^T: non-symmetric
    bands with weak diagonals in places (rows are exchanged), non-symmetric
    low-rank terms."""
    rng = np.random.default_rng([n, w, seed])

    def band(scale):
        A = np.zeros((n, n))
        for k in range(-w, w + 1):
            i = np.arange(max(0, -k), min(n, n - k))
            A[i, i + k] = scale * rng.standard_normal(len(i))
        return A

    d = np.linspace(1.0, 10.0, n)
    d[rng.random(n) < 0.1] = 5.0
    mats = [band(0.5 / np.sqrt(w)) + np.diag(d), np.eye(n), band(0.2 / np.sqrt(w))]
    fns = [wl.fn_rational([1.0]), wl.fn_rational([-1.0, 0.0]), wl.fn_exp(alpha=-1.0)]
    for k, r in enumerate(ranks):
        mats.append(0.1 * rng.standard_normal((n, r)) @ rng.standard_normal((r, n)) / r)
        fns.append(wl.fn_rational([0.5, 1.0j]) if k == 0 else wl.fn_exp(alpha=0.1))
    if dense_twin:
        mats[0][0, n - 1] += 1e-30
    return Problem("bordered", mats, fns)


def _moments(nep, p, N, L, K=2, seed=5, **kw):
    op = nep.SplitOperator.from_problem(p)
    V = wl.probes(p.n, L, seed)
    S, st = op.moments(CON, nep.device_probes(V), N, L, K, prec="mixed", **kw)
    return op, V, nep.moments_to_numpy(S), st


def _close(Sg, So, V, tol=1e-10):
    for q in range(So.shape[0]):
        err = np.linalg.norm(Sg[q] - So[q]) / max(np.linalg.norm(So[q]), 1e-2 * np.linalg.norm(V))
        assert err <= tol, (q, err)


# n around whole blocks of 32 rows and around the sizes from which 2, 3 and 4 chunks are taken
@pytest.mark.parametrize("n,w,ranks,N,L", [(256, 5, [], 8, 1), (289, 32, [], 8, 33), (416, 6, [31], 8, 3),
                                           (640, 8, [33], 8, 8), (1024, 32, [], 4, 5), (1057, 17, [40, 24], 4, 8),
                                           (1550, 9, [20], 4, 7), (2049, 32, [64, 64], 4, 4)])
def test_moments_match_oracle(nep, n, w, ranks, N, L):
    p = _problem(n, w, ranks)
    op, V, Sg, st = _moments(nep, p, N, L)
    print(st)
    assert st["n_unconverged"] == 0 and st["n_fallback"] == 0 and st["min_abs_pivot"] > 0.0, st
    assert st["max_rel_residual"] <= 1e-14 and st["ms_lu"] > 0.0, st
    _close(Sg, oracle.ciss_moments(p, CON, N, 2, V), V)
    op.close()


def test_further_probes_count_and_points(nep):
    n, N, L, K = 1100, 64, 4, 2
    p, twin = _problem(n, 6, [33], seed=3), _problem(n, 6, [33], seed=3, dense_twin=True)
    op, _, _, st = _moments(nep, p, N, L)
    opt, _, _, _ = _moments(nep, twin, N, L)
    assert st["n_fallback"] == 0, st
    B = nep.binding
    c, _, w = B.nep_ciss_count(op.h)
    ct, _, wt = B.nep_ciss_count(opt.h)
    assert c == ct and abs(w - wt) < 1e-3, (c, ct, w, wt)
    Vd = nep.device_probes(wl.probes(n, L, 9))
    S2, St = (torch.empty((2 * K, L, n), dtype=torch.complex128, device="cuda") for _ in range(2))
    B.nep_ciss_moments_more(op.h, Vd, S2)
    B.nep_ciss_moments_more(opt.h, Vd, St)
    for q in range(2 * K):
        assert float(torch.linalg.norm(S2[q] - St[q])) <= 1e-10 * float(torch.linalg.norm(St[q]))
    z = [4.1 + 0.3j, 6.0 - 0.2j, 5.5 + 1.0j]
    Y, Yt = (torch.empty((3, L, n), dtype=torch.complex128, device="cuda") for _ in range(2))
    B.nep_solve_at(op.h, z, Vd, Y, prec="mixed")
    B.nep_solve_at(opt.h, z, Vd, Yt, prec="fp64")
    assert float(torch.linalg.norm(Y - Yt)) <= 1e-11 * float(torch.linalg.norm(Yt))
    op.close()
    opt.close()


def test_singular_chunk_falls_back(nep):
    """The banded part alone is singular at every node (a zero row), T is not."""
    n, N, L = 416, 8, 2
    rng = np.random.default_rng(4)
    p0 = _problem(n, 5, [])
    A = p0.mats[0].copy()
    A[100, :] = 0.0
    U, V = rng.standard_normal((n, 20)), rng.standard_normal((n, 20))
    U[100] = 3.0 * rng.standard_normal(20)
    p = Problem("chunk", [A, 0.1 * U @ V.T], [wl.fn_rational([1.0]), wl.fn_exp(alpha=-0.1)])
    op, Vp, Sg, st = _moments(nep, p, N, L)
    print(st)
    assert st["n_fallback"] == N and st["n_unconverged"] == 0 and st["singular_node"] < 0, st
    _close(Sg, oracle.ciss_moments(p, CON, N, 2, Vp), Vp)
    op.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batch_equals_single_calls(nep, graph):
    N, L, K = 8, 5, 2
    probs = [_problem(420, 7, [20]), _problem(150, 6, [], dense_twin=True), _problem(300, 1, []),
             _problem(1056, 32, []), _problem(700, 5, [10, 24])]
    ops, singles, Vs = [], [], []
    for k, p in enumerate(probs):
        op, V, Sg, st = _moments(nep, p, N, L, seed=k)
        assert st["n_fallback"] == 0, (k, st)
        ops.append(op)
        singles.append(Sg)
        Vs.append(nep.device_probes(V))
    Ss = [torch.zeros((2 * K, L, p.n), dtype=torch.complex128, device="cuda") for p in probs]
    B = nep.binding
    b = B.nep_batch_create([op.h for op in ops], [CON] * len(ops), B.opts_struct(N, L, K, "mixed"), Vs, Ss,
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


def _weak_chunk(eps, n=416, twin=False):
    """A - z D + W: row 100 of the banded part is eps times a random row at
    every z, and the low-rank term W makes T regular there."""
    rng = np.random.default_rng(4)
    A = _problem(n, 5, []).mats[0].copy()
    A[100] *= eps
    D = np.eye(n)
    D[100, 100] = 0.0
    U, V = rng.standard_normal((n, 20)), rng.standard_normal((n, 20))
    U[100] = 3.0 * rng.standard_normal(20)
    if twin:
        A[0, n - 1] += 1e-30
    return Problem("weak", [A, D, 0.1 * U @ V.T],
                   [wl.fn_rational([1.0]), wl.fn_rational([-1.0, 0.0]), wl.fn_rational([1.0])])


@pytest.mark.parametrize("eps", [0.0, 1e-9, 1e-7, 1e-4])
def test_count_behind_a_weak_chunk(nep, eps):
    """det T by the argument principle where a chunk is singular or nearly so: the eigenvalues of the pencil inside."""
    n, N, L = 416, 512, 2
    p = _weak_chunk(eps)
    lam = scipy.linalg.eigvals(p.mats[0] + p.mats[2], p.mats[1])
    inside = int(np.sum(np.abs(lam[np.isfinite(lam)] - 5.05) < 0.7))
    op, V, Sg, st = _moments(nep, p, N, L)
    print(st)
    assert st["n_unconverged"] == 0 and st["singular_node"] < 0 and st["min_abs_pivot"] > 0.0, st
    B = nep.binding
    c, step, w = B.nep_ciss_count(op.h)
    opt, _, _, stt = _moments(nep, _weak_chunk(eps, twin=True), N, L)
    assert stt["n_fallback"] == 0, stt
    ct, stept, wt = B.nep_ciss_count(opt.h)
    assert c == ct == inside and step < 3.0, (c, ct, inside, step, stept)
    # the determinants stay usable after further probes, on the same factors
    S2 = torch.empty((4, L, n), dtype=torch.complex128, device="cuda")
    B.nep_ciss_moments_more(op.h, nep.device_probes(wl.probes(n, L, 9)), S2)
    assert B.nep_ciss_count(op.h)[0] == inside
    op.close()
    opt.close()


def test_rejected_operator_keeps_dense_factors(nep):
    """The first call finds a chunk singular; the calls that follow on the same
    nodes solve with the dense factors at once, other nodes start anew."""
    n, N, L, K = 416, 16, 3, 2
    p = _weak_chunk(0.0)
    op, V, Sg, st = _moments(nep, p, N, L)
    assert st["n_fallback"] == N and st["n_unconverged"] == 0, st
    _close(Sg, oracle.ciss_moments(p, CON, N, K, V), V)
    V2 = wl.probes(n, L, 9)
    S2 = torch.zeros((2 * K, L, n), dtype=torch.complex128, device="cuda")
    st2 = nep.binding.nep_ciss_moments_more(op.h, nep.device_probes(V2), S2)
    assert st2["n_fallback"] == 0 and st2["n_unconverged"] == 0, st2
    _close(nep.moments_to_numpy(S2), oracle.ciss_moments(p, CON, N, K, V2), V2)
    S3, st3 = op.moments(CON, nep.device_probes(V2), N, L, K, prec="mixed")
    assert st3["n_fallback"] == 0 and st3["ms_lu"] > 0.0 and st3["min_abs_pivot"] > 0.0, st3
    assert torch.equal(S2, S3)
    con = Contour.circle(4.0, 0.5)
    S4, st4 = op.moments(con, nep.device_probes(V), N, L, K, prec="mixed")
    assert st4["n_fallback"] == N and st4["n_unconverged"] == 0, st4
    _close(nep.moments_to_numpy(S4), oracle.ciss_moments(p, con, N, K, V), V)
    z = [4.1 + 0.3j, 6.0 - 0.2j, 5.5 + 1.0j]
    Y = torch.empty((3, L, n), dtype=torch.complex128, device="cuda")
    nep.binding.nep_solve_at(op.h, z, nep.device_probes(V), Y, prec="mixed")
    for k, zk in enumerate(z):
        ref = np.linalg.solve(p.mats[0] - zk * p.mats[1] + p.mats[2], V)
        assert np.linalg.norm(Y[k].cpu().numpy().T - ref) <= 1e-10 * np.linalg.norm(ref)
    op.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batch_with_rejected_operators(nep, graph):
    """Two rejected operators beside dense ones of more and fewer rows, a band
    operator and a sound bordered one, in passes that follow each other."""
    N, L, K = 8, 5, 2
    probs = [_problem(500, 6, [], dense_twin=True), _weak_chunk(0.0), _problem(150, 6, [], dense_twin=True),
             _problem(300, 1, []), _weak_chunk(0.0, n=1040), _problem(420, 7, [20])]
    weak = [1, 4]
    ops = [nep.SplitOperator.from_problem(p) for p in probs]
    V = [wl.probes(p.n, L, k) for k, p in enumerate(probs)]
    So = [oracle.ciss_moments(p, CON, N, K, v) for p, v in zip(probs, V)]
    Vs = [nep.device_probes(v) for v in V]
    Ss = [torch.zeros((2 * K, L, p.n), dtype=torch.complex128, device="cuda") for p in probs]
    B = nep.binding
    b = B.nep_batch_create([op.h for op in ops], [CON] * len(ops), B.opts_struct(N, L, K, "mixed"), Vs, Ss,
                           use_graph=graph)
    for rep in range(4):
        for S in Ss:
            S.zero_()
        torch.cuda.synchronize()
        stats = B.nep_batch_run(b, len(ops))
        for k in range(len(ops)):
            assert stats[k]["n_fallback"] == (N if k in weak and rep == 0 else 0), (rep, k, stats[k])
            assert stats[k]["n_unconverged"] == 0 and stats[k]["min_abs_pivot"] > 0.0, (rep, k, stats[k])
            _close(nep.moments_to_numpy(Ss[k]), So[k], V[k])
    B.nep_batch_destroy(b)
    for op in ops:
        op.close()
