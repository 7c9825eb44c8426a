"""bench.py's count of the Gram's products against the tiles that the library's
routes form, by size."""
import numpy as np
import pytest

import bench


def _upper(d):
    return np.triu(np.ones((d, d), dtype=np.float32))


@pytest.mark.parametrize("d,other,tiles", [(64, 64, 4), (64, 100, 3), (100, 64, 10), (512, 384, 136), (1000, 4096, 528),
                                           (1024, 700, 528)])
def test_small_sides_are_formed_densely(d, other, tiles):
    nk = -(-d // 64)
    for side in (0, 1):
        assert bench.gram_flop(_upper(d), side, False, other) == (tiles * 2.0 * 32 * 32 * 64 * nk,) * 2


@pytest.mark.parametrize("d,other", [(1024, 1100), (1025, 64), (1100, 1100), (1152, 64), (1217, 64)])
@pytest.mark.parametrize("reverse", [False, True])
def test_large_sides_on_their_envelope(d, other, reverse):
    """A triangular basis: the panel's 128-row block b reaches over 64-column
    blocks up to one end, so the product of blocks p >= q has the shorter one's."""
    nk = -(-d // 64)
    nb = -(-nk // 2)
    S = _upper(d).T if reverse else _upper(d)[:, ::-1].T
    length = [sum(bool(S[128 * b:128 * b + 128, 64 * k:64 * k + 64].any()) for k in range(nk)) for b in range(nb)]
    want = sum(min(length[p], length[q]) for p in range(nb) for q in range(p + 1)) * 2.0 * 128 * 128 * 64
    dense, env = bench.gram_flop(_upper(d), 0, reverse, other)
    assert dense == nb * (nb + 1) / 2 * nk * 2.0 * 128 * 128 * 64
    assert env == want and env < 0.55 * dense
