"""Primal step with the duals staged in LDS, one to eight variables per thread and one
or several slices: the terms and their order are the plain kernel's, so are the bits."""
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


# variables per thread change at multiples of 262,144, slices at some 40,956 rows
@pytest.mark.parametrize("n,m,deg", [(1025, 7, 1), (262144, 40956, 2), (262145, 40957, 3), (524289, 81913, 4),
                                     (786433, 1003, 6), (1048577, 122870, 2), (1310721, 50001, 3), (1572865, 40000, 2),
                                     (1835009, 200003, 5), (2100001, 40961, 8)])
def test_staged_primal_equals_plain(G, n, m, deg):
    P = I.set_cover_columns(n, m, deg, seed=deg)
    g = G.Problem(P, G.default_params(k_int=20, K_max=64, autotune=0, power_iters=2))
    rng = np.random.default_rng(3)
    x, xp = rng.random(n).astype(np.float32), rng.random(n).astype(np.float32)
    y = rng.random(m).astype(np.float32)
    got = []
    for bits in (0, 4):
        g.set_launch_cfg(16, 1, 1, 1, 0, 0, 0, bits)
        g.set_state(x, xp, y, float(g.scales()["rho_min"][0]), k=3)
        g.pdhg_steps(2)
        got.append(g.get_state())
    assert np.array_equal(got[0]["x"], got[1]["x"]) and np.array_equal(got[0]["y"], got[1]["y"])
    g.close()
