"""Steps of the factorised reformulation: the one-workgroup kernels and the separate
ones add the same terms in the same order in FP64 and round once, so they agree in
every bit; and a row's update carries no FP32 accumulation."""
import numpy as np
import pytest

from paper_2510_27117_amd import instances as I
from tests.test_gpu_tu_steps import _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27117_amd import gfors
    return gfors


@pytest.mark.parametrize("name", ["fl", "one", "path_9", "rand_17", "noq_20", "rand_128", "rand_129", "noq_256",
                                  "rand_257", "noq_512"])
def test_one_workgroup_and_separate_kernels_agree_in_every_bit(G, name):
    P = _problem(name)
    T = G.TUReformulation(P, P.meta["tu_pivots"], factored=True)
    a, b = (T.problem(G.default_params(k_int=20, K_max=64, power_iters=20, autotune=0, lu_lds=lds)) for lds in (1, 0))
    rng = np.random.default_rng(5)
    x, xp = rng.random(a.n), rng.random(a.n)
    y, rho = np.abs(rng.standard_normal(a.m1 + a.m2)), float(a.scales()["rho_min"][0])
    for start in (True, False):
        for p in (a, b):
            if start:
                p.set_state(x, xp, y, rho, k=3)
            else:
                p.reset()
        for steps, res in ((1, False), (2, True), (41, False)):
            for p in (a, b):
                p.pdhg_steps(steps, want_residuals=res)
            sa, sb = a.get_state(), b.get_state()
            for key in ("x", "x_prev", "y"):
                assert np.array_equal(sa[key], sb[key]), (start, steps, key)
            if res:
                assert np.array_equal(a.residuals(), b.residuals())
    a.close()
    b.close()


@pytest.mark.parametrize("lds", [0, 1])
@pytest.mark.parametrize("n", [20, 40])
def test_row_updates_round_once(G, n, lds):
    """Rows of n^2 coefficients up to 10^6 (chunks of long rows) and of a few, x and the lift in
    multiples of 2^-10: every product and sum is exact in FP64, and the right-hand sides cancel all
    but about 1e-5 of the sum, of which an FP32 accumulation would keep two digits.  The update from
    the FP32 row data is then known to the rounding of y; one unit in the last place is allowed."""
    P = I.assignment_qap_like(n, seed=3, q_per_var=4.0, tree="random")
    rng = np.random.default_rng(n)
    rows = np.zeros((6, P.n), dtype=np.int64)
    rows[:4] = -rng.integers(1, 1_000_001, (4, P.n))
    for r in rows[4:]:
        r[rng.choice(P.n, 30, replace=False)] = -rng.integers(1, 1_000_001, 30)
    P.A, P.b = I.csr_from_dense(rows), np.zeros(6, dtype=np.int64)
    full = G.TUReformulation(P, P.meta["tu_pivots"])
    A1 = np.array(I.csr_to_dense(full.model.A))[:6].astype(np.float64)
    x, xp = (rng.integers(0, 1025, A1.shape[1]) / 1024.0 for _ in range(2))
    s = A1 @ (2 * x - xp)
    # b' = b - A s_0 for the fixed part s_0 of the lift: ask for b' a little above the sum
    b1 = np.rint(s + 1e-5 * np.abs(s))
    P.b = b1.astype(np.int64) - full.model.b[:6]
    T = G.TUReformulation(P, P.meta["tu_pivots"], factored=True)
    p = T.problem(G.default_params(k_int=20, K_max=64, power_iters=20, autotune=0, lu_lds=lds))
    sc = p.scales()
    sk, tau2 = float(sc["K_norm"][0]), np.float64(np.float32(sc["tau2"][0]))
    om = np.float64(np.float32(sc["row_scale"][:6] / sk))
    rt = np.float64(np.float32(b1 * sc["row_scale"][:6] / sk))
    p.set_state(x, xp, np.zeros(p.m1 + p.m2), float(sc["rho_min"][0]), k=3)
    p.pdhg_steps(1)
    want = np.maximum(tau2 * (rt - om * s), 0.0).astype(np.float32)
    got = p.get_state()["y"][:6]
    assert np.all(want > 0) and np.all(np.abs(rt - om * s) <= 1e-3 * np.abs(om * s))
    assert np.all(np.abs(got.astype(np.float64) - want) <= np.spacing(want)), (got, want)
    p.close()


@pytest.mark.parametrize("name", ["many_q", "many_rows"])
def test_one_workgroup_leaves_large_gradients_to_the_chip(G, name):
    """119 or 199 pivots with 200 to 400 entries each: the workgroup took 52 and 39 us a step where
    the separate kernels take 28.  Timed against them (without the LDS plan they are slower still)."""
    import torch
    if name == "many_q":
        P = I.assignment_qap_like(60, 3, q_per_var=400.0, tree="random")
    else:
        P = I.assignment_qap_like(100, 3, q_per_var=4.0, tree="random")
        P.A = I.csr_from_dense(-np.random.default_rng(0).integers(1, 9, (200, P.n)))
        P.b = np.full(200, -3 * P.n, dtype=np.int64)
    T = G.TUReformulation(P, P.meta["tu_pivots"], factored=True)
    best = []
    for lds in (1, 0):
        p = T.problem(G.default_params(k_int=200, K_max=64, power_iters=5, autotune=0, lu_lds=lds))
        p.run_rounds(2, 64)
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(p.stream)
            p.run_rounds(1, 64)
            b.record(p.stream)
            b.synchronize()
            t.append(a.elapsed_time(b))
        best.append(min(t))
        p.close()
    assert best[0] <= 1.1 * best[1], best
