"""Steps of the factorised reformulation with the narrow parts in one workgroup
each against the kernels that take any size (no LDS plan), within the bars of the
FP32 parity tests: 1e-5 after one or two steps from one state, 1e-4 free-running."""
import numpy as np
import pytest

from paper_2510_27117_amd import instances as I

from _helpers import rel_inf

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


def _problem(name):
    if name == "fl":          # signed-identity pivot block, no quadratic term
        return I.facility_location(7, 23, seed=5)
    if name == "one":         # a single pivot
        P = I.from_dense([4, -1, 3], A=[[1, 0, 1]], b=[1], B=[[1, 1, 1]], d=[1])
        P.meta["tu_pivots"] = np.array([1])
        return P
    kind, n = name.split("_")  # 2 n - 1 pivots: a thread each of 256, 512, 1024 or the general kernels
    P = I.assignment_qap_like(int(n), seed=3, q_per_var=6.0, tree="path" if kind == "path" else "random")
    return _no_q(P) if kind == "noq" else P


@pytest.mark.parametrize("steps, bar", [(1, 1e-5), (2, 1e-5), (41, 1e-4)])
@pytest.mark.parametrize("name", ["fl", "one", "path_9", "rand_17", "noq_20", "rand_128", "rand_129", "noq_256",
                                  "rand_257", "noq_512", "noq_513"])
def test_one_workgroup_against_general_kernels(G, name, steps, bar):
    P = _problem(name)
    T = G.TUReformulation(P, P.meta["tu_pivots"], factored=True)
    got = []
    for lds in (1, 0):
        prob = T.problem(G.default_params(k_int=20, K_max=64, power_iters=20, autotune=0, lu_lds=lds))
        if steps <= 2:      # from a state with every dual at work
            rng = np.random.default_rng(5)
            x, xp = rng.random(prob.n), rng.random(prob.n)
            prob.set_state(x, xp, np.abs(rng.standard_normal(prob.m1 + prob.m2)), float(prob.scales()["rho_min"][0]), k=3)
        prob.pdhg_steps(steps)
        got.append(prob.get_state())
        prob.close()
    for key in ("x", "y"):
        assert rel_inf(got[0][key], got[1][key]) <= bar, key
