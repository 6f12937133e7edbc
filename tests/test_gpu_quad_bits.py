"""Quadratic objectives whose entries have one magnitude, counted bitwise: exact
against the oracle's evaluation of the same candidates."""
import numpy as np
import pytest

from oracle import gfors_oracle as O
from paper_2510_27117_amd import instances as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27117_amd import gfors
    return gfors


def _signed(n, degree, mag, seed, symmetric=True, diagonal=False, star=0):
    rng = np.random.default_rng(seed)
    k = max(1, int(n * degree / 2))
    i, j = rng.integers(0, n, k), rng.integers(0, n, k)
    if star:
        i, j = np.concatenate([i, np.zeros(star, int)]), np.concatenate([j, 1 + np.arange(star)])
    lo, hi = np.minimum(i, j), np.maximum(i, j)
    key = np.unique((lo * n + hi)[(lo == hi) if diagonal else (lo != hi)])
    i, j = key // n, key % n
    v = mag * rng.choice([-1, 1], key.size)
    P = I.max_cut_er(n, 0.0, seed)
    P.c = rng.integers(-9, 10, n).astype(P.c.dtype)
    if symmetric and not diagonal:
        i, j, v = np.concatenate([i, j]), np.concatenate([j, i]), np.concatenate([v, v])
    P.Q = I.csr_from_coo(n, n, i, j, v)
    return P


# 256 variables a tile, lists of 2,048 entries, counters flushed every 255 a lane, rows of 65,535 at most
CASES = {"tiny": dict(n=3, degree=2, mag=1), "255": dict(n=255, degree=12, mag=1), "256": dict(n=256, degree=30, mag=3),
         "257": dict(n=257, degree=60, mag=1), "upper": dict(n=1500, degree=8, mag=1000003, symmetric=False),
         "diagonal": dict(n=700, degree=900, mag=5, diagonal=True), "star": dict(n=61440, degree=1, mag=1, star=61430),
         "star_beyond": dict(n=70000, degree=1, mag=1, star=65600), "large": dict(n=20000, degree=10, mag=1)}


@pytest.mark.parametrize("K", [64, 192, 2048, 4096])
@pytest.mark.parametrize("name", list(CASES) + ["batch"])
def test_signed_entries_count_exactly(G, name, K):
    import torch
    if K > 2048 and CASES.get(name, {}).get("n", 0) > 5000:
        K = 128
    P = (I.concat_instances([_signed(600, 9, 2, 1), _signed(3, 2, 2, 2), _signed(301, 40, 2, 3)]) if name == "batch"
         else _signed(seed=7, **CASES[name]))
    g = G.Problem(P, G.default_params(K_max=K, autotune=0, power_iters=2))
    rng = np.random.default_rng(K)
    p = rng.choice(np.array([0.0, 0.3, 0.7, 1.0], dtype=np.float32), P.n)     # both kinds of fixed variables
    v, z = g.sample_eval(K, p_override=torch.from_numpy(p).cuda(), outputs=True)
    X = O.unpack_bits(g.candidates(), K).T.astype(np.int64)
    rows = np.repeat(np.arange(P.n), np.diff(P.Q.row_ptr))
    z = z.cpu().numpy()
    part = [(0, P.n)] if name != "batch" else [(0, 600), (600, 603), (603, 904)]
    for t, (a, b) in enumerate(part):
        e0, e1 = P.Q.row_ptr[a], P.Q.row_ptr[b]
        ref = P.c[a:b] @ X[a:b]
        for s in range(e0, e1, 20000):
            q = slice(s, min(s + 20000, e1))
            ref = ref + P.Q.val[q].astype(np.int64) @ (X[rows[q]] * X[P.Q.col[q]])
        assert np.array_equal(z[t], ref)
