"""How far the library's 64-bit sums are from the exact ones, against long
double (64-bit mantissa) references. All arithmetic is fp64, so what can be lost
is in the order of the sums: feedback, or a panel's product, accumulated term by
term onto a large value rounds at that value's magnitude in every term."""
import numpy as np
import pytest

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
