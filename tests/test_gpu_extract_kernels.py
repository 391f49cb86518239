"""The extraction's QR panels, device SVD and compact-WY product at the edges of
their row and column ranges (panels of 8 and 4 columns with one to four rows a thread and the path beyond
them, 63 to 80 columns around the device SVD's limit): moments of a known operator go in, eigenvalues, eigenvectors and
singular values are compared with the FP64 oracle's extraction of the same
moments."""
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


# (n, L, K): K n rows and K L columns of the block Hankel matrix
@pytest.mark.parametrize("n,L,K", [(40, 5, 1), (40, 4, 4), (127, 3, 4), (128, 4, 4), (129, 17, 1), (257, 2, 2),
                                   (512, 7, 2), (513, 9, 2), (1024, 16, 1), (1025, 9, 2), (700, 21, 3), (700, 16, 4),
                                   (700, 13, 5), (2050, 8, 2), (2100, 20, 4)])
def test_extraction_matches_oracle(nep, n, L, K):
    """A diagonal operator with a few eigenvalues inside: the moments are
    exact, S_p = sum over the eigenvalues, so the oracle's extraction is cheap
    at every size."""
    rng = np.random.default_rng([n, L, K])
    inside = min(3, K * L - 1)
    d = np.concatenate([[0.3 + 0.1j, -0.4j, -0.5 + 0.2j][:inside], 3.0 + rng.uniform(0.0, 4.0, n - inside)])
    con, N = Contour.circle(0.0, 1.0), 64
    p = Problem("diag", [np.diag(d), np.eye(n)], [wl.fn_rational([1.0]), wl.fn_rational([-1.0, 0.0])])
    V = wl.probes(n, L, 3)
    # exact discrete filter: sum_j w_j zeta_j^q / (d - z_j) for every diagonal entry
    z = np.exp(2j * np.pi * (np.arange(N) + 0.5) / N)
    S = np.stack([(np.sum((z / N) * z ** q / (d[:, None] - z), axis=1))[:, None] * V for q in range(2 * K)])
    op = nep.SplitOperator.from_problem(p)
    Sd = torch.from_numpy(np.ascontiguousarray(S.transpose(0, 2, 1))).to("cuda")
    r = op.extract(con, Sd, N, L, K, max_eigs=K * L, rank_tol=1e-10)
    ro = oracle.extract(p, con, S, K, rank_tol=1e-10)
    assert r["m"] == len(ro["lam"]), (r["m"], len(ro["lam"]))
    sv = np.linalg.svd(np.block([[S[a + b] for b in range(K)] for a in range(K)]), compute_uv=False)
    assert np.max(np.abs(r["sigma"] - sv)) <= 1e-13 * sv[0]
    got, ref = r["lam"][r["inside"]], d[:inside]
    assert len(got) == inside, r["lam"]
    for k in range(inside):
        q = int(np.argmin(np.abs(r["lam"] - ref[k])))
        assert abs(r["lam"][q] - ref[k]) <= 1e-12
        x = r["X"][:, q]
        assert abs(np.linalg.norm(x) - 1.0) <= 1e-13 and abs(x[k] - 1.0) <= 1e-11, (k, x[k])
        assert r["eta"][q] <= 1e-12
    op.close()


def _diag_moments(n, L, K, inside, con, N):
    """A diagonal operator with the given eigenvalues inside, probes and its moments through the exact discrete filter."""
    rng = np.random.default_rng([n, L, K])
    d = np.concatenate([inside, 3.0 + rng.uniform(0.0, 4.0, n - len(inside))])
    p = Problem("diag", [np.diag(d), np.eye(n)], [wl.fn_rational([1.0]), wl.fn_rational([-1.0, 0.0])])
    V = wl.probes(n, L, 3)
    z = np.exp(2j * np.pi * (np.arange(N) + 0.5) / N)
    S = np.stack([(np.sum((z / N) * z ** q / (d[:, None] - z), axis=1))[:, None] * V for q in range(2 * K)])
    return p, d, V, S


# K L = 256 and beyond: one and several 256-row blocks of the compact-WY product, ragged last blocks
@pytest.mark.parametrize("n,L,K", [(70, 64, 4), (70, 52, 5), (90, 64, 5), (70, 64, 8), (80, 57, 9)])
def test_extraction_of_many_columns(nep, n, L, K):
    con, N = Contour.circle(0.0, 1.0), 64
    p, d, V, S = _diag_moments(n, L, K, [0.3 + 0.1j, -0.4j, -0.5 + 0.2j, 0.1 - 0.1j], con, N)
    op = nep.SplitOperator.from_problem(p)
    Sd = torch.from_numpy(np.ascontiguousarray(S.transpose(0, 2, 1))).to("cuda")
    r = op.extract(con, Sd, N, L, K, max_eigs=K * L, rank_tol=1e-10)
    sv = np.linalg.svd(np.block([[S[a + b] for b in range(K)] for a in range(K)]), compute_uv=False)
    assert np.max(np.abs(r["sigma"] - sv)) <= 1e-13 * sv[0]
    assert np.count_nonzero(r["inside"]) == 4, r["lam"]
    for k in range(4):
        q = int(np.argmin(np.abs(r["lam"] - d[k])))
        x = r["X"][:, q]
        assert abs(r["lam"][q] - d[k]) <= 1e-12 and r["eta"][q] <= 1e-12
        assert abs(np.linalg.norm(x) - 1.0) <= 1e-13 and abs(x[k] - 1.0) <= 1e-11, (k, x[k])
    op.close()


def test_probe_augmentation_past_256_columns(nep):
    """200 eigenvalues inside saturate the first block's 160 columns; the
    second block's 320 resolve them."""
    n, L, K, N, tol = 260, 40, 4, 64, 1e-9
    con = Contour.circle(0.0, 1.0)
    rng = np.random.default_rng(2)
    inside = rng.uniform(0.1, 0.85, 200) * np.exp(2j * np.pi * rng.uniform(size=200))
    p, d, V, S = _diag_moments(n, 2 * L, K, inside, con, N)
    sv = np.linalg.svd(np.block([[S[a + b] for b in range(K)] for a in range(K)]), compute_uv=False)
    op = nep.SplitOperator.from_problem(p)
    X = torch.zeros((2 * K * L, n), dtype=torch.complex128, device="cuda")
    r = nep.binding.nep_eigs(op.h, con, nep.binding.opts_struct(N, L, K, "fp64"), nep.device_probes(V), 2 * L, X,
                             max_eigs=2 * K * L, rank_tol=tol)
    assert r["L_used"] == 2 * L and r["m"] == 200, (r["L_used"], r["m"])
    # a perturbation of the moments by rounding moves the eigenvalues by it over the smallest kept singular value,
    # times the condition of the (random, unstructured) projected eigenvectors, at most a few hundred
    bound = 1e3 * 2.3e-16 * sv[0] / sv[199]
    assert bound < 1e-7, bound
    for x in inside:
        assert np.min(np.abs(r["lam"] - x)) <= bound
    op.close()


def test_moments_that_hold_nan(nep):
    """Refused as moments without a rank, and no singular value is left over from the call before."""
    n, L, K, N = 40, 4, 4, 64
    con = Contour.circle(0.0, 1.0)
    p, d, V, S = _diag_moments(n, L, K, [0.3 + 0.1j], con, N)
    op = nep.SplitOperator.from_problem(p)
    B = nep.binding
    X = torch.zeros((K * L, n), dtype=torch.complex128, device="cuda")
    Sd = torch.from_numpy(np.ascontiguousarray(S.transpose(0, 2, 1))).to("cuda")
    opts = B.opts_struct(N, L, K, "mixed")
    good = B.nep_extract(op.h, con, opts, Sd, X, max_eigs=K * L)
    assert np.all(np.isfinite(good["sigma"]))
    Sd[1, 2, 7] = float("nan")
    with pytest.raises(B.NepError) as e:
        B.nep_extract(op.h, con, opts, Sd, X, max_eigs=K * L)
    assert e.value.m == 0
    assert np.all(np.isnan(e.value.sigma)), e.value.sigma
    op.close()
