"""How far the library's 64-bit sums are from the exact ones, against long
double (64-bit mantissa) references. All arithmetic is fp64, so what can be lost
is in the order of the sums: feedback, or a panel's product, accumulated term by
term onto a large value rounds at that value's magnitude in every term."""
import numpy as np
import pytest
from scipy.linalg import solve_triangular

import parity as pr
from paper_2607_27042_amd import workloads as wl

pytestmark = pytest.mark.gpu

# 2-norm of one rounding of normally distributed values, relative to theirs: an
# error of ulp / sqrt(12), and ulp^2 / value^2 is about 2^-104 / 2 on average
ROUNDING = 2.0 ** -52 * 0.5 ** 0.5 / 12 ** 0.5


def exact_y(X, Z, L, U):
    """Y = Z - E with L E U = Z - X, by substitution in long double."""
    E = Z.astype(np.longdouble) - X
    L, U = L.astype(np.longdouble), U.astype(np.longdouble)
    for i in range(E.shape[0]):
        E[i] -= L[i, :i] @ E[:i]
    for j in range(E.shape[1]):
        E[:, j] -= E[:, :j] @ U[:j, j]
    return Z - E


@pytest.mark.parametrize("m,n", [(64, 64), (200, 120), (96, 333)])
@pytest.mark.parametrize("reverse", [False, True])
def test_corrected_values(m, n, reverse):
    """An entry's value is rounded at its own magnitude when the tile's feedback
    is added to X, when its band's is, when its block's is, and by at most 15
    pushes inside its 4 x 4 block: 18 roundings. As many again are allowed for the
    feedback's own sums and for what earlier entries' errors bring."""
    p = wl.random_problem(m, n, 5, "f64", "general")
    res = pr.gpu_run(p, reverse=reverse)
    flip = (lambda a: a[::-1, ::-1]) if reverse else (lambda a: a)
    Y = exact_y(flip(p.X), flip(res["Z"]), res["L"], res["U"])
    err = float(np.linalg.norm((flip(res["Y"]) - Y).astype(np.float64)) / np.linalg.norm(Y.astype(np.float64)))
    print(f"Y {m}x{n} reverse={reverse}: {err:.3e}", flush=True)
    assert err <= 36 ** 0.5 * ROUNDING


def exact_feedback(S):
    """F unit lower with (S S^T)^{-1} = F Lambda F^T, in long double."""
    S = S[::-1].astype(np.longdouble)
    C, d = S @ S.T, S.shape[0]
    for j in range(d):  # Cholesky of the index-reversed Gram
        C[j:, j] -= C[j:, :j] @ C[j, :j]
        C[j:, j] /= np.sqrt(C[j, j])
    W = np.zeros_like(C)
    for i in range(d):
        W[i, :i] = -(C[i, :i] @ W[:i, :i])
        W[i, i] = 1
        W[i] /= C[i, i]
    return (W * C.diagonal()[:, None]).T[::-1, ::-1]


def lapack_feedback(S):
    S = S[::-1]
    C = np.linalg.cholesky(S @ S.T)
    W = solve_triangular(C, np.eye(len(C)), lower=True)
    return (W * C.diagonal()[:, None]).T[::-1, ::-1]


def test_factor_sums():
    """Factors of triangular bases, whose Grams vary most in magnitude: a panel's
    64 terms are summed from zero and leave the trailing block in one subtraction.
    LAPACK's route to the same factors is the yardstick: the library is 1.7 times as
    far from long double, and 2.7 times with every term subtracted from the trailing
    block by itself; the bound is their geometric mean."""
    d, ratio = 512, []
    for seed in (1, 2):
        rng = np.random.default_rng(seed)
        A = np.triu(rng.standard_normal((d, d)), 1) / d ** 0.5
        A[np.diag_indices(d)] = np.exp(rng.uniform(np.log(0.5), np.log(2.0), d))
        f = pr.binding.Factors.from_bases(pr.to_dev(A), pr.to_dev(A.T))
        L, U, _, _ = (t.cpu().numpy() for t in f.export())
        f.close()
        assert np.array_equal(L, U.T)  # the same Gram on both sides
        ref = exact_feedback(A.T)
        off = lambda x: float(np.linalg.norm((x - ref).astype(np.float64)))
        ratio.append(off(L) / off(lapack_feedback(A.T)))
    print("factor error over LAPACK's:", ratio, flush=True)
    assert np.mean(ratio) <= (1.7 * 2.7) ** 0.5
