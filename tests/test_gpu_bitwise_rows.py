"""Bitwise row evaluation where a row is shared by several lane groups, and the
3D-assignment selection on tied, sparse and binary p: exact against the oracle."""
import numpy as np
import pytest

from oracle import assign3d_oracle as A3
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


def _rows_problem(lens, n, seed):
    """Covering, at-most-one and exactly-one rows (both signs) of the given lengths."""
    rng = np.random.default_rng(seed)
    A, b, B, d = [], [], [], []
    for q, ln in enumerate(lens):
        row = np.zeros(n, dtype=np.int64)
        row[rng.choice(n, size=ln, replace=False)] = 1
        kind = q % 4
        if kind == 0:
            A.append(row); b.append(1)
        elif kind == 1:
            A.append(-row); b.append(-1)
        elif kind == 2:
            B.append(row); d.append(1)
        else:
            B.append(-row); d.append(-1)
    c = rng.integers(-50, 50, size=n)
    return I.from_dense(c, A=np.array(A), b=np.array(b), B=np.array(B), d=np.array(d))


@pytest.mark.parametrize("K", [64, 192, 512, 1024, 4096])
@pytest.mark.parametrize("which", ["short", "long", "edges", "many"])
def test_shared_rows_count_exactly(G, which, K):
    n = 3000
    lens = {"short": [3, 7, 8, 9] * 6, "long": [2500, 1999, 3000, 1025] * 3,
            "edges": [63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513] * 2, "many": [40, 41, 47, 48] * 300}[which]
    P = _rows_problem(lens, n, seed=len(lens) + K)
    G_ = G.Problem(P, G.default_params(K_max=K, autotune=0, power_iters=2))
    rng = np.random.default_rng(K)
    # about one set variable per row, so that all three verdicts occur, and
    # deterministic variables of both kinds
    p = np.where(rng.random(n) < 0.5, 1.0 / np.mean(lens), 0.0).astype(np.float32)
    p[rng.integers(0, n, 2)] = 1.0
    import torch
    v, z = G_.sample_eval(K, p_override=torch.from_numpy(p).cuda(), outputs=True)
    X = O.unpack_bits(G_.candidates(), K)
    vo, zo = O.evaluate(P, X)
    assert np.array_equal(v.cpu().numpy()[0], vo)
    assert np.array_equal(z.cpu().numpy()[0], zo)


@pytest.mark.parametrize("n", [2, 21, 33])
@pytest.mark.parametrize("kind", ["equal", "binary", "few", "steps", "none"])
def test_selection_of_tied_entries(G, n, kind):
    import torch
    P = I.assignment_3d(n, seed=n)
    N, rng = n ** 3, np.random.default_rng(n)
    p = {"equal": np.full(N, 0.25), "binary": (rng.random(N) < 0.3).astype(float),
         "few": np.where(np.arange(N) % 997 == 5, rng.random(N), 0.0),
         "steps": rng.integers(0, 5, N) / 4.0, "none": np.zeros(N)}[kind].astype(np.float32)
    K, gamma, L = 128, 3, 4
    g = G.Problem(P, G.default_params(K_max=K, autotune=0, power_iters=2))
    g.sample_eval_assign3d(n, K, gamma, L, p_override=torch.from_numpy(p).cuda())
    X, _ = A3.assign3d_sample(p.astype(np.float64), P.c, n, K, gamma, L, seed=0, rnd=0)
    assert np.array_equal(g.candidates(), O.pack_bits(X))
