"""The tile sweep works on 4 x 4 blocks in bands of 16 rows; here are the
shapes where a block, a band or a tile ends, with factors far from the
identity, in both orders and types, and those where the width of the delivery
batches changes. The trajectory is replayed by the oracle
under the library's own factors: Z must match entry by entry, and Y, an fp64
sum of at most m + n products, must agree to 1e-9 (2e-6 of the largest value
where it leaves as fp32)."""
import numpy as np
import pytest

import oracle
import parity as pr
from paper_2607_27042_amd import workloads as wl

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 4), (5, 1), (4, 17), (16, 12), (17, 60), (49, 64), (64, 3), (64, 64), (61, 65),
          (65, 15), (80, 113), (128, 67), (131, 192), (193, 129)]


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("dtype,reverse", [("f64", False), ("f32", True)])
def test_block_edges(m, n, dtype, reverse):
    p = wl.random_problem(m, n, 31, dtype, "general", xscale=9.0)
    res = pr.gpu_run(p, reverse=reverse)
    flip = (lambda a: np.ascontiguousarray(a[::-1, ::-1])) if reverse else (lambda a: a)
    q = wl.Problem(p.name, flip(p.X), p.A, p.B, dtype)  # the problem the sweep runs forwards
    Z, Y = flip(res["Z"]), flip(res["Y"])
    Zo, Yo, c, hard = pr.replay(q, res["L"], res["U"], Z)
    pr.assert_replay_pass(q, c, hard, m * n)
    tol = 1e-9 if dtype == "f64" else 2e-6 * max(1.0, np.abs(Yo).max())
    assert np.abs(Y - Yo).max() <= tol
    X, A, B = p.widened()
    pr.assert_objective(p, res["obj"], oracle.objective(X, flip(Zo), A, B))


def test_delivery_widths_same_bits(monkeypatch):
    """The width decides which sources share a product, not the order of the sums."""
    p = wl.random_problem(1000, 700, 32, "f64", "general")
    ref = pr.gpu_run(p)
    for width in (1, 2, 3, 4, 5, 7):
        monkeypatch.setenv("GPTQ2D_BATCH", str(width))
        res = pr.gpu_run(p)
        assert np.array_equal(res["Z"], ref["Z"]) and np.array_equal(res["Y"], ref["Y"]), width


# 640 and 1280 products of 64^3 a launch (40 x 32, 64 x 40 tiles) are the last with
# widths 2 and 3; beyond, 4 up to 64 tiles a side and 5 above
@pytest.mark.parametrize("m,n", [(2560, 2048), (2624, 2048), (4096, 2560), (4096, 2624), (4160, 2560)])
def test_delivery_width_edges(m, n):
    p = wl.random_problem(m, n, 33, "f64", "general")
    res = pr.gpu_run(p)
    pr.assert_trajectory(p, res)
