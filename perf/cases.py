"""The work that users of this library have it do, as cases to be timed.

Every case goes through the public binding: a handle, its bases' factorisation
and the rounding sweep, on one device. A case is a dict of plain values:

  call     "step"     factorise the bases, then round X (one layer of a model)
           "round"    round a new X with factors that are already there
           "noalloc"  the same through the entry point that needs no workspace
           "factor"   factorise the bases and export the factors
           "batch"    `count` problems of one shape per call, factorised and
                      rounded in common launches (the small layers of a model)
  m, n     shape of X
  dtype    "f32" or "f64": X, the bases and Y (all arithmetic is fp64)
  reverse  round from the last row and column on
  basis    how A and B are drawn: "gram" and "scaled" and "heavy" and "spiked"
           are Cholesky factors of Grams of Gaussian, badly scaled Gaussian,
           heavy-tailed and spiked activations, "tri" a triangular matrix
           drawn directly, "dense" a general square matrix
"""
import math

import torch

from paper_2607_27042_amd import binding


def listed():
    def case(name, call, m, n, dtype, basis, reverse=False, count=1):
        return {"name": name, "call": call, "m": m, "n": n, "dtype": dtype, "basis": basis,
                "reverse": reverse, "count": count}

    return [
        # one tile: the smallest problem, all latency
        case("step 64x64 f64", "step", 64, 64, "f64", "gram"),
        # a serving loop that rounds small matrices with factors it keeps
        case("noalloc 200x120 f32", "noalloc", 200, 120, "f32", "gram"),
        # one small layer
        case("step 512x384 f32", "step", 512, 384, "f32", "scaled"),
        # a ragged shape, general bases, the other rounding order
        case("step 1000x700 f64 reverse", "step", 1000, 700, "f64", "dense", reverse=True),
        # factors made once and kept by the program, ragged sizes, general bases
        case("factor 3000x2000 f32", "factor", 3000, 2000, "f32", "dense"),
        # an attention projection of a language model
        case("step 4096x4096 f32", "step", 4096, 4096, "f32", "heavy"),
        # a further matrix of an MLP with factors that are already there
        case("round 4096x11008 f32", "round", 4096, 11008, "f32", "spiked"),
        # the largest square layer, in double precision throughout
        case("step 8192x8192 f64", "step", 8192, 8192, "f64", "tri"),
        # many one-tile problems per call
        case("batch 256 of 64x64 f64", "batch", 64, 64, "f64", "gram", count=256),
        # many small layers per call
        case("batch 64 of 512x384 f32", "batch", 512, 384, "f32", "scaled", count=64),
    ]


def _cost(call, m, n, count):
    c = 0.0
    if call != "factor":
        c += float(m) * n * (m + n)
    if call in ("step", "batch", "factor"):
        c += 1.7 * (float(m) ** 3 + float(n) ** 3)
    return c * count


def draw(rng):
    call = rng.choice(["step", "step", "round", "noalloc", "factor", "batch"])
    most = _cost("step", 8192, 8192, 1) * 0.9
    lo, hi = {"batch": (24, 1024), "noalloc": (24, 1300)}.get(call, (48, 11008))

    def size():
        d = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        # half of the sizes as layers have them (whole multiples of 64), half as they come
        return max(64, d // 64 * 64) if rng.random() < 0.5 else d

    while True:
        m, n = size(), size()
        count = int(round(math.exp(rng.uniform(math.log(4), math.log(256))))) if call == "batch" else 1
        if _cost(call, m, n, count) > most or count * m * n > 60_000_000:
            continue
        if call == "noalloc" and -(-m // 64) * -(-n // 64) * 64 * 64 * 32 > 60_000_000:
            continue
        if max(m, n) > 8192 and call != "round":
            continue
        break
    basis = rng.choice(["gram", "scaled", "heavy", "spiked", "tri", "dense"])
    return {"call": call, "m": m, "n": n, "dtype": rng.choice(["f32", "f32", "f64"]), "basis": basis,
            "reverse": rng.random() < 0.25, "count": count}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _basis(kind, d, g):
    """A basis of d columns, in 64 bits. Cholesky factors are upper triangular."""
    if kind == "dense":
        a = _randn(g, d, d) / math.sqrt(d)
        a.diagonal().add_(2.0)
        return a
    if kind == "tri":
        a = torch.triu(_randn(g, d, d), 1) / math.sqrt(d)
        a.diagonal().copy_(torch.exp(_uniform(g, math.log(0.5), math.log(2.0), d)))
        return a
    rows = max(256, 2 * d)
    if kind == "heavy":  # Student-t with four degrees of freedom
        chi = sum(_randn(g, rows, d).square_() for _ in range(4))
        w = _randn(g, rows, d).div_(chi.div_(4.0).sqrt_())
        del chi
    elif kind == "scaled":
        w = _randn(g, rows, d) * torch.exp(_uniform(g, math.log(0.1), math.log(10.0), d))
    elif kind == "spiked":
        v, _ = torch.linalg.qr(_randn(g, d, min(32, d)))
        w = _randn(g, rows, d) + math.sqrt(50.0) * (_randn(g, rows, v.shape[1]) @ v.T)
    else:
        w = _randn(g, rows, d)
    gram = (w.T @ w) / rows
    del w
    damp = gram.diagonal().mean() if kind in ("heavy", "spiked") else 1.0
    gram.diagonal().add_(0.01 * damp)
    return torch.linalg.cholesky(gram).T.contiguous()


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    m, n, dt = case["m"], case["n"], _dtype(case)
    X, A, B = [], [], []
    for _ in range(case["count"]):
        X.append((3.0 * _randn(g, m, n)).to(dt))
        A.append(_basis(case["basis"], m, g).to(dt))
        B.append(_basis(case["basis"], n, g).to(dt))
    return X, A, B


def prepare(case, seed):
    m, n, dt, count = case["m"], case["n"], _dtype(case), case["count"]
    X, A, B = _inputs(case, seed)
    f = [binding.Factors(m, n, reverse=case["reverse"]) for _ in range(count)]
    s = {"call": case["call"], "f": f, "X": X, "A": A, "B": B}
    if case["call"] == "factor":
        return s
    # outputs of a batch are stacked; each problem writes its own slice
    s["Z"] = torch.empty(count, m, n, dtype=torch.int32, device="cuda")
    s["Y"] = torch.empty(count, m, n, dtype=dt, device="cuda")
    s["obj"] = torch.empty(count, dtype=torch.float64, device="cuda")
    if case["call"] == "batch":
        handles, shapes = [x.handle for x in f], [(m, n)] * count
        s["fws"] = torch.empty(binding.gptq2d_factor_batched_workspace_size(count), dtype=torch.uint8, device="cuda")
        s["ws"] = torch.empty(binding.gptq2d_round_batched_workspace_size(handles), dtype=torch.uint8, device="cuda")
        s["factor"] = binding.gptq2d_factor_batched(handles, A, B, s["fws"], shapes=shapes, prepare=True)
        s["round"] = binding.gptq2d_round_batched(handles, X, list(s["Z"]), list(s["Y"]), s["obj"], s["ws"],
                                                  shapes=shapes, prepare=True)
        return s
    if case["call"] == "noalloc":
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    else:
        s["ws"] = f[0].workspace()
    if case["call"] in ("round", "noalloc"):
        f[0].compute(A[0], B[0])
        binding.gptq2d_factor_check(f[0].handle)
    return s


def run(s):
    f, call = s["f"][0], s["call"]
    if call == "factor":
        f.compute(s["A"][0], s["B"][0])
        return f.export()
    if call == "batch":
        s["factor"]()
        s["round"]()
    elif call == "noalloc":
        binding.gptq2d_round_noalloc(f.handle, s["X"][0], s["Z"][0], s["Y"][0], s["obj"], s["status"])
    else:
        if call == "step":
            f.compute(s["A"][0], s["B"][0])
        binding.gptq2d_round(f.handle, s["X"][0], s["Z"][0], s["Y"][0], s["obj"], s["ws"])
    return s["Z"], s["Y"], s["obj"]


def work(case):
    m, n, count = float(case["m"]), float(case["n"]), case["count"]
    es = 4 if case["dtype"] == "f32" else 8
    # the Gram of a triangular basis is a third of a general one's
    side = 5.0 / 3.0 if case["basis"] == "dense" else 1.0
    factor = {"bytes": es * (m * m + n * n), "flops": side * (m ** 3 + n ** 3)}
    sweep = {"bytes": m * n * (2 * es + 4), "flops": m * n * (m + n)}
    triangles = 8 * (m * m + n * n) / 2
    if case["call"] == "factor":
        return {"bytes": factor["bytes"] + 2 * triangles, "flops": factor["flops"]}
    if case["call"] in ("round", "noalloc"):
        return {"bytes": sweep["bytes"] + triangles, "flops": sweep["flops"]}
    return {k: count * (factor[k] + sweep[k]) for k in ("bytes", "flops")}


def tolerance(case):
    # All sums are 64-bit ones. Against exact() the factors were 2e-15 to 2.4e-13
    # off (largest entry 1.1e-11, for badly scaled bases), and Y in 64 bits
    # 2e-16 to 1e-14 (1.4e-13). In 32 bits an entry of Y whose 64-bit value
    # moved in its last places may round to the next float, which one entry in
    # 1e5 does at most. Z did not differ: only a value within about 1e-13 of a
    # half-integer could go either way.
    if case["call"] == "factor":
        return {"rel": 1e-12, "max": 5e-11, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 1e-9, "max": 3e-7, "differ": 1e-6}
    return {"rel": 5e-13, "max": 1e-11, "differ": 1e-6}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------

def _feedback(Q):
    """Unit-lower F and Lambda with Q^{-1} = F diag(Lambda) F^T."""
    # Q = R R^T with R upper, from the Cholesky factor of the index-reversed Q
    R = torch.linalg.cholesky(Q.flip(-2, -1)).flip(-2, -1)
    eye = torch.eye(Q.shape[-1], dtype=Q.dtype, device=Q.device).expand_as(Q)
    inv = torch.linalg.solve_triangular(R, eye, upper=True)
    diag = R.diagonal(dim1=-2, dim2=-1)
    return (inv * diag.unsqueeze(-1)).transpose(-2, -1), 1.0 / diag.square()


def _factors(A, B):
    L, lamL = _feedback(A.transpose(-2, -1).contiguous() @ A)
    F, lamU = _feedback(B @ B.transpose(-2, -1).contiguous())
    return L.contiguous(), F.transpose(-2, -1).contiguous(), lamL, lamU


def _sweep(X, L, U):
    """Entry (i, j) is rounded from Y = X + sum over earlier entries of
    L[i][i'] E[i'][j'] U[j'][j], one anti-diagonal at a time."""
    b, m, n = X.shape
    Ut = U.transpose(-2, -1).contiguous()  # row j holds U[:, j]
    Et = torch.zeros(b, n, m, dtype=X.dtype, device=X.device)
    C = torch.zeros_like(X)
    Y = torch.empty_like(X)
    xf, yf, cf, ef = X.view(b, -1), Y.view(b, -1), C.view(b, -1), Et.view(b, -1)
    for k in range(m + n - 1):
        i0, i1 = max(0, k - n + 1), min(m, k + 1)
        i = torch.arange(i0, i1, device=X.device)
        j0, j1 = k - (i1 - 1), k - i0 + 1
        # rows not yet rounded are zero in Et and C
        down = (L[:, i0:i1, :i1] * Et[:, j0:j1, :i1].flip(1)).sum(-1)
        right = (C[:, i0:i1, :j1] * Ut[:, j0:j1, :j1].flip(1)).sum(-1)
        at = i * n + (k - i)
        y = xf[:, at] + right + down
        e = torch.round(y) - y
        yf[:, at] = y
        cf[:, at] = down + e
        ef[:, (k - i) * m + i] = e
    return torch.round(Y), Y, Et.transpose(-2, -1)


def exact(case, seed):
    m, n, count = case["m"], case["n"], case["count"]
    if m * n * (m + n) * count > 1.5e11 or max(m, n) > 6000:
        return None  # minutes
    X, A, B = (torch.stack([t.double() for t in v]) for v in _inputs(case, seed))
    if case["reverse"]:  # the forward order on the index-reversed problem
        X, A, B = X.flip(-2, -1), A.flip(-1), B.flip(-2)
    L, U, lamL, lamU = _factors(A, B)
    if case["call"] == "factor":
        return L[0], U[0], lamL[0], lamU[0]
    Z, Y, E = _sweep(X.contiguous(), L, U)
    obj = (E.square() / (lamL.unsqueeze(-1) * lamU.unsqueeze(-2))).sum((-2, -1))
    if case["reverse"]:
        Z, Y = Z.flip(-2, -1), Y.flip(-2, -1)
    return Z.to(torch.int32), Y, obj
