"""Runs of steps with each instance in a workgroup's LDS against one launch per
step: the sums run over the same lanes in the same order, so every bit of the
state and of the residuals must agree."""
import numpy as np
import pytest

from paper_2510_27117_amd import instances as I
from tests._helpers import mixed_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27117_amd import gfors
    return gfors


def _no_q(P):
    P.Q = None
    return P


def _problems():
    tiny = I.from_dense([3], A=[[1]], b=[1])                                   # one variable, one row
    # dense rows: fewer variables than one load, ragged ends, one to four tiles, coefficients in
    # registers (few rows for the tiles) and in LDS
    dense = {"dense%d" % k: I.concat_instances([I.knapsack_multi(n, m, seed=n) for n, m in sizes]) for k, sizes in
             enumerate((((5, 3), (65, 1), (2047, 7)), ((2048, 9), (64, 16)), ((777, 17), (9, 2)), ((2049, 5), (4095, 13)),
                        ((8191, 8), (300, 1)), ((600, 61), (1000, 30)), ((6000, 10), (2047, 33))))}
    wide = I.concat_instances([I.knapsack_multi(n, m, seed=n, wmax=100_000) for n, m in ((64, 3), (257, 5))])
    sparse = I.concat_instances([I.set_cover_bernoulli(301, 97, 0.05, seed=3), _no_q(mixed_problem(150, seed=6)),
                                 I.facility_location(5, 19, seed=2), I.knapsack_multi(33, 2, seed=1)])
    return {"tiny": tiny, "cover": I.set_cover_bernoulli(1037, 301, 0.02, seed=1), **dense, "dense_int32": wide,
            "batch": sparse, "two_per_group": I.set_cover_columns(1500, 700, 4, seed=9),
            "long_rows": I.set_cover_bernoulli(900, 90, 0.15, seed=2),
            "unit_batch": I.concat_instances([I.set_cover_bernoulli(200, 100, 0.05, seed=s) for s in range(3)]),
            "equalities": _no_q(I.assignment_qap_like(9, seed=7))}


NAMES = ["tiny", "cover", "dense_int32", "batch", "two_per_group", "long_rows", "unit_batch", "equalities"]


@pytest.mark.parametrize("start", ["zero", "random"])
@pytest.mark.parametrize("name", NAMES + ["dense%d" % k for k in range(7)])
def test_resident_steps_equal_launch_per_step(G, name, start):
    P = _problems()[name]
    prm = G.default_params(k_int=7, K_max=64, autotune=0)
    a, b = G.Problem(P, prm), G.Problem(P, prm)
    base = a.launch_cfg()
    assert base["slices_dual"] == base["slices_primal"] == 1
    b.set_launch_cfg(**base)                                       # a launch per step from here on
    if start == "random":
        rng = np.random.default_rng(5)
        x, xp = rng.random(P.n), rng.random(P.n)
        y = rng.standard_normal(P.m1 + P.m2)
        y[: P.m1] = np.maximum(y[: P.m1], 0.0)
        for q in (a, b):
            q.set_state(x, xp, y, 0.05)
    for steps, res in ((1, False), (2, True), (7, False), (1, True)):
        for q in (a, b):
            q.pdhg_steps(steps, want_residuals=res)
        sa, sb = a.get_state(), b.get_state()
        for k in ("x", "x_prev", "y"):
            assert np.array_equal(sa[k], sb[k]), (name, steps, k)
        assert sa["k"] == sb["k"]
        if res:
            assert np.array_equal(a.residuals(), b.residuals())
    for q in (a, b):
        q.run_rounds(3, 64)
    assert np.array_equal(a.candidates(), b.candidates())
    assert np.array_equal(a.get_state()["x"], b.get_state()["x"])


@pytest.mark.parametrize("name", ["cover", "batch", "two_per_group"])
def test_resident_follows_tuned_lanes(G, name):
    """The tuned lanes per row / variable are those of the per-launch kernels too."""
    P = _problems()[name]
    a, b = G.Problem(P, G.default_params(k_int=20, K_max=64)), G.Problem(P, G.default_params(k_int=20, K_max=64))
    c = a.launch_cfg()
    b.set_launch_cfg(**c)
    for q in (a, b):
        q.pdhg_steps(41)
    for k in ("x", "x_prev", "y"):
        assert np.array_equal(a.get_state()[k], b.get_state()[k])
