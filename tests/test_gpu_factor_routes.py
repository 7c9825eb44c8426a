"""The factorisation's routes by size: one launch for one block per side, Grams
on 32 x 32, 64 x 64 and 128 x 128 tiles, one group of panels or several,
right-looking or left-looking. Factors against the oracle's explicit-inverse
route (1e-10, the agreement of the two fp64 routes on these bases), and a
batch large enough to take other routes than a single problem against the
single problem: the same sums in the same order, hence the same bits."""
import numpy as np
import pytest
import torch

import oracle
import parity as pr
from paper_2607_27042_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1, 64), (63, 64), (64, 65), (96, 1), (1024, 31), (1025, 33), (1152, 127), (1600, 66),
                                 (1024, 1088), (66, 1217)])
@pytest.mark.parametrize("reverse", [False, True])
def test_routes_match_oracle(m, n, reverse):
    p = wl.random_problem(m, n, 41, "f64", "general")
    X, A, B = p.widened()
    f = binding.Factors.from_bases(pr.to_dev(p.A), pr.to_dev(p.B), reverse=reverse)
    L, U, lamL, lamU = (t.cpu().numpy() for t in f.export())
    f.close()
    if reverse:
        A, B = np.ascontiguousarray(A[:, ::-1]), np.ascontiguousarray(B[::-1])
    Lo, lamLo, Uo, lamUo = oracle.factors(A, B)
    for got, ref in ((L, Lo), (U, Uo)):
        assert np.abs(got - ref).max() <= 1e-10 * max(1.0, np.abs(ref).max())
    np.testing.assert_allclose(lamL, lamLo, rtol=1e-10)
    np.testing.assert_allclose(lamU, lamUo, rtol=1e-10)


@pytest.mark.parametrize("m,n,count", [(512, 384, 18), (130, 70, 160), (64, 40, 300), (1152, 64, 2), (1650, 300, 3),
                                       (1650, 300, 4), (200, 2112, 5)])
def test_batch_routes_same_bits(m, n, count):
    g = torch.Generator(device="cuda").manual_seed(7)

    def basis(d):
        t = torch.randn(d, d, generator=g, device="cuda", dtype=torch.float64) / d ** 0.5
        t.diagonal().add_(2.0)
        return t
    As, Bs = [basis(m) for _ in range(count)], [basis(n) for _ in range(count)]
    fs = [binding.Factors(m, n) for _ in range(count)]
    binding.factor_batched(fs, As, Bs)
    one = binding.Factors(m, n)
    for p in (0, count // 2, count - 1):
        one.compute(As[p], Bs[p])
        for x, y in zip(one.export(), fs[p].export()):
            assert torch.equal(x, y), f"problem {p}"


# tiles of 64 x 64 and of 128 x 128 fill 256 compute units from 5/4 and from 0.85 per
# unit (one or two rounds) or two per unit on: Grams on 64 x 64 tiles, ragged and
# whole; on whole 128 x 128 tiles, one side or both, a round and more; beside a larger
# side
@pytest.mark.parametrize("m,n,count", [(512, 384, 6), (700, 321, 4), (130, 70, 60), (1024, 896, 4), (640, 512, 9),
                                       (768, 200, 26), (64, 1024, 16), (1024, 1100, 3), (1250, 896, 3)])
@pytest.mark.parametrize("kind", ["upper", "lower", "blocks"])
@pytest.mark.parametrize("dtype,reverse", [(torch.float32, False), (torch.float32, True), (torch.float64, True)])
def test_batch_gram_routes_same_bits(m, n, count, kind, dtype, reverse):
    """Bases with zero blocks, which the larger tiles skip, in both types and orders."""
    g = torch.Generator(device="cuda").manual_seed(m + n)

    def basis(d):
        t = torch.randn(d, d, generator=g, device="cuda", dtype=torch.float64) / d ** 0.5
        if kind == "blocks":
            at = torch.arange(d, device="cuda") // 100
            t *= at.unsqueeze(0) == at.unsqueeze(1)
        else:
            t = t.triu_() if kind == "upper" else t.tril_()
        t.diagonal().add_(2.0)
        return t.to(dtype)
    As, Bs = [basis(m) for _ in range(count)], [basis(n) for _ in range(count)]
    fs = [binding.Factors(m, n, reverse=reverse) for _ in range(count)]
    binding.factor_batched(fs, As, Bs)
    one = binding.Factors(m, n, reverse=reverse)
    for p in (0, count // 2, count - 1):
        one.compute(As[p], Bs[p])
        for x, y in zip(one.export(), fs[p].export()):
            assert torch.equal(x, y), f"problem {p}"


def test_small_side_beside_a_large_one():
    """Each side's Gram takes the route of its own size: the factors of a 200 side
    do not depend on the other side, but for the order of the panels' sums."""
    m, n = 200, 2944
    p, q = wl.random_problem(m, 64, 43, "f32", "general"), wl.random_problem(64, n, 44, "f32", "general")
    both = binding.Factors.from_bases(pr.to_dev(p.A), pr.to_dev(q.B)).export()
    left = binding.Factors.from_bases(pr.to_dev(p.A), pr.to_dev(p.B)).export()
    right = binding.Factors.from_bases(pr.to_dev(q.A), pr.to_dev(q.B)).export()
    for got, ref in ((both[0], left[0]), (both[1], right[1]), (both[2], left[2]), (both[3], right[3])):
        assert (got - ref).abs().max() <= 1e-12 * ref.abs().max()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("m,n,count", [(512, 384, 1), (512, 384, 6), (1024, 896, 4), (1152, 100, 1), (1152, 100, 2)])
def test_nonfinite_entry_beside_zero_blocks(value, m, n, count):
    """The larger Gram tiles skip products with a block of zeros; a NaN or an
    infinity in the other block still reaches its own column's pivot."""
    eye = [torch.eye(d, device="cuda", dtype=torch.float64) for d in (m, n)]
    fs = [binding.Factors(m, n) for _ in range(count)]
    As, Bs = [eye[0].clone() for _ in range(count)], [eye[1].clone() for _ in range(count)]
    As[-1][3, m - 2] = value
    if count == 1:
        fs[0].compute(As[0], Bs[0])
    else:
        binding.factor_batched(fs, As, Bs, check=False)
    with pytest.raises(binding.Gptq2dError) as e:
        binding.gptq2d_factor_check(fs[-1].handle)
    assert e.value.status == -2  # GPTQ2D_ERR_SINGULAR
    for f in fs[:-1]:
        binding.gptq2d_factor_check(f.handle)


@pytest.mark.parametrize("side", ["A", "B"])
@pytest.mark.parametrize("m,n", [(20, 64), (64, 96)])
def test_singular_side_is_reported(side, m, n):
    """Each side's error word is read, and cleared by the next factorisation."""
    A = torch.eye(m, device="cuda", dtype=torch.float64)
    B = torch.eye(n, device="cuda", dtype=torch.float64)
    bad = {"A": A.clone(), "B": B.clone()}
    bad[side][0, 0] = 0.0
    f = binding.Factors(m, n)
    f.compute(bad["A"], bad["B"])
    with pytest.raises(binding.Gptq2dError) as e:
        binding.gptq2d_factor_check(f.handle)
    assert e.value.status == -2  # GPTQ2D_ERR_SINGULAR
    f.compute(A, B)
    binding.gptq2d_factor_check(f.handle)
