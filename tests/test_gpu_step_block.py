"""The one-launch step of dense int16 batches against the two products apart
(which a residual step keeps): the same sums in the same order, so every bit of
the state must agree."""
import numpy as np
import pytest

from paper_2510_27117_amd import instances as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27117_amd import gfors
    return gfors


# variables at the edges of 8-column loads and of 2,048-column tiles; rows at the
# edges of what a thread holds between the products (36) and of a group of four
@pytest.mark.parametrize("sizes", [[(2047, 35), (2048, 36), (2049, 37), (4096, 1)], [(16385, 40), (9, 3), (8191, 64)],
                                   [(40_001, 5), (1000, 29), (64, 4)]])
def test_joint_steps_equal_products_apart(G, sizes):
    P = I.concat_instances([I.knapsack_multi(n, m, seed=n + m) for n, m in sizes])
    a, b = (G.Problem(P, G.default_params(k_int=6, K_max=64, autotune=0)) for _ in range(2))
    rng = np.random.default_rng(3)
    x, xp, y = rng.random(P.n), rng.random(P.n), np.abs(rng.standard_normal(P.m1))
    for q in (a, b):
        q.set_launch_cfg(16, 4, 1, 1, 0, 0, 4, 5)
        q.set_state(x, xp, y, 0.02)
    for steps in (1, 2, 5):
        a.pdhg_steps(steps)
        for _ in range(steps):
            b.pdhg_steps(1, want_residuals=True)
        sa, sb = a.get_state(), b.get_state()
        for k in ("x", "x_prev", "y", "k"):
            assert np.array_equal(sa[k], sb[k]), (steps, k)
    for _ in range(3):
        a.run_rounds(1, 64)                       # replayed graph
        for _ in range(6):
            b.pdhg_steps(1, want_residuals=True)
        b.sample_eval(64)
        assert np.array_equal(a.get_state()["x"], b.get_state()["x"])
        assert np.array_equal(a.candidates(), b.candidates())
