"""Exact violation counts where most rows have one or two entries, among covering and
partitioning rows of any length: many tiles (256 threads each) and few (1,024), one to
64 candidate words, more rows per lane group than its counters hold at once."""
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


def _pairs(n, rows, others, seed):
    """`rows` rows of one or two entries with any coefficients, `others` of the lengths given."""
    rng = np.random.default_rng(seed)
    A, b, B, d = [], [], [], []
    for q in range(rows + len(others)):
        row = np.zeros(n, dtype=np.int64)
        if q < rows:
            row[rng.choice(n, size=1 + q % 2, replace=False)] = rng.integers(-3, 4, 1 + q % 2)
            if not row.any():
                row[0] = 1
            rhs = int(rng.integers(-3, 3))
        else:
            row[rng.choice(n, size=others[q - rows], replace=False)] = 1
            rhs = 1
        (A if q % 3 else B).append(row)
        (b if q % 3 else d).append(rhs)
    if not A:
        A, b = B, d
    return I.from_dense(rng.integers(-9, 10, n), A=np.array(A), b=np.array(b),
                        B=np.array(B) if B else None, d=np.array(d) if B else None)


def _check(G, P, parts, K, seed):
    import torch
    g = G.Problem(P, G.default_params(K_max=K, autotune=0, power_iters=2))
    rng = np.random.default_rng(seed)
    p = np.where(rng.random(P.n) < 0.7, rng.random(P.n), 0.0).astype(np.float32)
    p[rng.integers(0, P.n, 2)] = 1.0
    v, z = g.sample_eval(K, p_override=torch.from_numpy(p).cuda(), outputs=True)
    X = O.unpack_bits(g.candidates(), K)
    v, z, at = v.cpu().numpy(), z.cpu().numpy(), 0
    for t, part in enumerate(parts):
        vo, zo = O.evaluate(part, X[at:at + part.n] if X.shape[0] == P.n else X[:, at:at + part.n])
        assert np.array_equal(v[t], vo) and np.array_equal(z[t], zo), t
        at += part.n
    g.close()


@pytest.mark.parametrize("K", [64, 192, 1024, 4096])
@pytest.mark.parametrize("rows, others", [(3, []), (61, [1, 7, 8, 9, 16, 17]), (4500, [200, 63, 64])])
def test_few_tiles(G, rows, others, K):
    P = _pairs(260, rows, others, seed=rows)
    _check(G, P, [P], K, rows + K)


@pytest.mark.parametrize("K", [64, 320, 4096])
def test_many_tiles(G, K):
    """700 instances, a tile at least each; one with enough rows for its counters to be emptied under way."""
    base = [_pairs(40, 30, [8, 21], 1), _pairs(7, 5, [], 2), I.facility_location(3, 5, 3), _pairs(50, 1500, [9], 4)]
    parts = [base[t % 3] for t in range(699)] + [base[3]]
    _check(G, I.concat_instances(parts), parts, K, K)
