"""Sampler with up to 512 candidates (wavefronts share them and split the variables)
and just above: the oracle's bits and objectives, exactly."""
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


@pytest.mark.parametrize("cmax", [50, (1 << 21) - 1, 1 << 21, 1 << 40])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 448, 512, 576, 1024])
@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1025, 3001])
def test_sets_of_variables_match_oracle(G, n, K, cmax):
    import torch
    rng = np.random.default_rng(n + K)
    c = rng.integers(-cmax, cmax + 1, n)
    c[0] = cmax
    A = np.zeros((1, n), dtype=int)
    A[0, 0] = 1
    P = I.from_dense(c, A=A, b=np.array([0]))
    g = G.Problem(P, G.default_params(K_max=K, autotune=0, power_iters=2))
    p = rng.choice([0.0, 1.0, 0.5, 1e-7, 1.0 - 2.0 ** -24, 0.2], n).astype(np.float32)
    v, z = g.sample_eval(K, p_override=torch.from_numpy(p).cuda(), outputs=True)
    X = O.sample_bits(p.astype(np.float64), K, seed=0, rnd=0)
    assert np.array_equal(O.unpack_bits(g.candidates(), K), X)
    assert np.array_equal(z.cpu().numpy()[0], X.astype(np.int64) @ c.astype(np.int64))
