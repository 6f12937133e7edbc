"""The form of the steps that a launch configuration stands for: runs of steps in
one launch (dual 6 / primal 8), steps over codes of x (primal 9), and the launches
whose sums both reproduce.  A configuration that was read keeps its form when it
is set, on the same problem or another one; the forms agree in every bit."""
import numpy as np
import pytest

from paper_2510_27117_amd import instances as I
from tests.test_gpu_q_codes import CASES, _box
from tests.test_gpu_resident import NAMES, _problems

pytestmark = pytest.mark.gpu

RUN, CODES = (6, 8), (0, 9)


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_27117_amd import gfors
    return gfors


def _form(p):
    c = p.launch_cfg()
    return c["bits_dual"], c["bits_primal"]


def _with(cfg, bits_dual, bits_primal, **more):
    return {**cfg, "bits_dual": bits_dual, "bits_primal": bits_primal, **more}


def _problem(kind):
    if kind == "run":
        return I.set_cover_bernoulli(200, 100, 0.05, seed=0), RUN
    return _box(140000, 8, 3, 3), CODES


@pytest.mark.parametrize("kind", ["run", "codes"])
@pytest.mark.parametrize("tuned", [0, 1])
def test_a_configuration_that_was_read_keeps_its_form(G, kind, tuned):
    P, form = _problem(kind)
    p = G.Problem(P, G.default_params(k_int=10, K_max=64, power_iters=20, autotune=tuned))
    cfg = p.launch_cfg()
    assert (cfg["bits_dual"], cfg["bits_primal"]) == form
    p.set_launch_cfg(**cfg)
    assert p.launch_cfg() == cfg
    other = G.Problem(P, G.default_params(k_int=10, K_max=64, power_iters=20, autotune=0))
    other.set_launch_cfg(**_with(cfg, 0, 0))             # launches, asked for by name
    assert other.launch_cfg() == _with(cfg, 0, 0)
    other.set_launch_cfg(**cfg)                          # a stored configuration brings its form along
    assert other.launch_cfg() == cfg
    other.set_launch_cfg(**_with(cfg, 0, 0))
    other.autotune()
    assert _form(other) == form
    p.close()
    other.close()


def test_forms_are_refused_where_they_do_not_apply(G):
    run, _ = _problem("run")
    codes, _ = _problem("codes")
    large = I.set_cover_columns(60_000, 6_000, 4, seed=1)
    prm = G.default_params(k_int=10, K_max=64, power_iters=20, autotune=0)
    for P, cfgs in ((run, [(4, 4, 1, 1, 0, 0, 6, 0), (4, 4, 1, 1, 0, 0, 0, 8), (3, 4, 1, 1, 0, 0, 6, 8),
                           (256, 4, 1, 1, 0, 0, 6, 8), (4, 4, 1, 1, 1, 0, 6, 8), (4, 4, 1, 1, 0, 0, 0, 9),
                           (4, 4, 1, 1, 0, 0, 7, 0), (4, 4, 1, 1, 0, 0, 0, 10)]),
                    (codes, [(1, 8, 1, 1, 0, 0, 0, 9), (1, 4, 1, 1, 0, 0, 6, 9), (1, 4, 1, 1, 0, 0, 6, 8)]),
                    (large, [(4, 4, 1, 1, 0, 0, 6, 8), (4, 4, 1, 1, 0, 0, 0, 9)])):
        p = G.Problem(P, prm)
        before = p.launch_cfg()
        for cfg in cfgs:
            with pytest.raises(G.GforsError):
                p.set_launch_cfg(*cfg)
            assert p.launch_cfg() == before
        p.close()


@pytest.mark.parametrize("name", NAMES + ["dense%d" % k for k in range(7)])
def test_run_of_steps_equals_its_launches(G, name):
    """Against the launches of the same lanes, from a state with every dual at work."""
    P = _problems()[name]
    prm = G.default_params(k_int=7, K_max=64, autotune=0)
    a, b = G.Problem(P, prm), G.Problem(P, prm)
    cfg = a.launch_cfg()
    a.set_launch_cfg(**_with(cfg, *RUN))
    # dense rows of 16-bit coefficients: the dense-block tiles, else lanes per row / variable
    b.set_launch_cfg(**_with(cfg, *((4, 5) if name.startswith("dense") and name != "dense_int32" else (0, 0))))
    assert _form(a) == RUN and _form(b) != RUN
    rng = np.random.default_rng(5)
    x, xp = rng.random(P.n), rng.random(P.n)
    y = rng.standard_normal(P.m1 + P.m2)
    y[: P.m1] = np.maximum(y[: P.m1], 0.0)
    for q in (a, b):
        q.set_state(x, xp, y, 0.05)
    for steps, res in ((1, False), (2, True), (7, False), (1, True), (40, False)):
        for q in (a, b):
            q.pdhg_steps(steps, want_residuals=res)
        sa, sb = a.get_state(), b.get_state()
        for k in ("x", "x_prev", "y"):
            assert np.array_equal(sa[k], sb[k]), (steps, k)
        assert sa["k"] == sb["k"]
        if res:
            assert np.array_equal(a.residuals(), b.residuals())
    a.close()
    b.close()


@pytest.mark.parametrize("name, lanes", [("columns", (1, 1)), ("columns", (4, 1)), ("columns", (4, 2)), ("columns", (16, 8)),
                                         ("batch", (1, 1)), ("batch", (4, 2)), ("batch", (64, 32)), ("cover", (2, 1))])
def test_run_of_steps_at_other_lanes(G, name, lanes):
    """Entries in registers (one or two rows / variables a group) and in LDS, by the lanes."""
    P = I.set_cover_columns(1500, 500, 3, seed=9) if name == "columns" else _problems()[name]
    prm = G.default_params(k_int=7, K_max=64, autotune=0)
    a, b = G.Problem(P, prm), G.Problem(P, prm)
    a.set_launch_cfg(*lanes, 1, 1, 0, 0, *RUN)
    b.set_launch_cfg(*lanes, 1, 1, 0, 0, 0, 0)
    for q in (a, b):
        q.pdhg_steps(33, want_residuals=True)
    for k in ("x", "x_prev", "y"):
        assert np.array_equal(a.get_state()[k], b.get_state()[k]), k
    assert np.array_equal(a.residuals(), b.residuals())
    a.close()
    b.close()


@pytest.mark.parametrize("name", ["largest", "least", "one_more", "ragged", "long", "empty_rows"])
@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_codes_equal_the_kernel_that_gathers(G, name, lanes):
    n, degree, vmax, star = CASES[name]
    P = _box(n, degree, vmax, 3, star)
    prm = G.default_params(k_int=7, K_max=64, autotune=0, power_iters=5)
    a, b = G.Problem(P, prm), G.Problem(P, prm)
    a.set_launch_cfg(1, lanes, 1, 1, 0, 0, *CODES)
    b.set_launch_cfg(1, lanes, 1, 1, 0, 0, 0, 0)
    assert _form(a) == CODES and _form(b) == (0, 0)
    rng = np.random.default_rng(7)
    x, xp = np.clip(rng.random(n) * 3 - 1, 0, 1).astype(np.float32), rng.random(n).astype(np.float32)
    for p in (a, b):
        p.set_state(x, xp, np.zeros(0), 0.01, k=3)
    for steps, res in ((1, False), (2, True), (67, False)):
        for p in (a, b):
            p.pdhg_steps(steps, want_residuals=res)
        for key in ("x", "x_prev"):
            assert np.array_equal(a.get_state()[key], b.get_state()[key]), (steps, key)
        if res:
            assert np.array_equal(a.residuals(), b.residuals())
    a.close()
    b.close()


def _hub(n, degree, star):
    """About `degree` entries a row and exactly `star` in row 0."""
    P = _box(n, degree, 3, 3)
    rng = np.random.default_rng(1)
    rows, col, val = np.repeat(np.arange(n), np.diff(P.Q.row_ptr)), np.asarray(P.Q.col), P.Q.values()
    keep = (rows != 0) & (col != 0)
    j = 1 + rng.permutation(n - 1)[:star]
    zero, one = np.zeros(star, int), np.ones(star, int)
    P.Q = I.csr_from_coo(n, n, np.concatenate([rows[keep], zero, j]), np.concatenate([col[keep], j, zero]),
                         np.concatenate([val[keep], one, one]))
    return P


@pytest.mark.parametrize("tuned", [0, 1])
@pytest.mark.parametrize("star, form", [(128, CODES), (129, (0, 0)), (60000, (0, 0))])
def test_long_rows_keep_the_kernel_with_more_lanes(G, star, form, tuned):
    """A row is walked by at most four lanes over codes: past 128 entries k_primal's lanes are ahead."""
    p = G.Problem(_hub(135000, 6, star), G.default_params(k_int=10, K_max=64, power_iters=5, autotune=tuned))
    assert _form(p) == form
    p.close()


@pytest.mark.parametrize("tuned", [0, 1])
@pytest.mark.parametrize("name, lanes", [("long_rows", (8, 1)), ("two_per_group", (1, 1)), ("cover", (2, 1)),
                                         ("batch", (8, 2)), ("tiny", (1, 1))])
def test_lanes_of_a_run_cover_an_instance_in_one_pass(G, name, lanes, tuned):
    """1,024 threads over the rows / variables of the largest instance: as many lanes as the mean
    row asks for, up to one pass.  Tuning looks at twice as many."""
    p = G.Problem(_problems()[name], G.default_params(k_int=7, K_max=64, autotune=tuned))
    c = p.launch_cfg()
    assert _form(p) == RUN
    for got, want in zip((c["lpr_dual"], c["lpr_primal"]), lanes):
        assert got == want if not tuned else got in (want, 2 * want)
    p.close()


@pytest.mark.parametrize("P, untuned, tuned", [
    (lambda: I.set_cover_columns(3000, 500, 4, 1), True, True),
    (lambda: I.set_cover_columns(4000, 700, 4, 1), False, False),
    (lambda: I.concat_instances([I.set_cover_columns(4000, 700, 4, s) for s in range(4)]), True, True),
    (lambda: I.knapsack_multi(500, 61, 1), False, False),
    (lambda: I.knapsack_multi(2000, 38, 1), True, False),
    (lambda: I.knapsack_multi(500, 24, 1), True, True),
    (lambda: I.knapsack_multi(6000, 9, 1), True, True),
    (lambda: I.knapsack_multi(500, 60, 1, wmax=100_000), True, True),
    (lambda: I.concat_instances([I.knapsack_multi(500, 61, s) for s in range(64)]), True, True)])
def test_runs_only_where_a_workgroup_is_ahead_of_the_chip(G, P, untuned, tuned):
    bip = P()
    for at, want in ((0, untuned), (1, tuned)):
        p = G.Problem(bip, G.default_params(k_int=7, K_max=64, power_iters=5, autotune=at))
        assert (_form(p) == RUN) == want, at
        cfg = p.launch_cfg()
        p.set_launch_cfg(min(cfg["lpr_dual"], 64), min(cfg["lpr_primal"], 64), 1, 1, 0, 0, *RUN)   # it fits all the same
        assert _form(p) == RUN
        p.autotune()
        assert (_form(p) == RUN) == tuned
        p.close()


@pytest.mark.parametrize("name", ["run", "whole_steps", "codes", "rows_apart", "many_tiles"])
def test_kernel_times_are_those_of_ordinary_calls(G, name):
    """Kinds that ran, with their launches; the steps advance as pdhg_steps does, bit for bit."""
    P, cfg, steps = {
        "run": (lambda: _problem("run")[0], None, {"primal": 9}),
        "whole_steps": (lambda: I.concat_instances([I.knapsack_multi(300, 7, seed=s) for s in range(3)]),
                        (16, 4, 1, 1, 0, 0, 4, 5), {"dual": 1, "primal": 9}),
        "codes": (lambda: _problem("codes")[0], None, {"primal": 9}),
        "rows_apart": (lambda: I.facility_location(7, 40, 2), (4, 4, 1, 1, 0, 0, 0, 0), {"dual": 9, "primal": 9}),
        "many_tiles": (lambda: I.set_cover_columns(90_000, 9_000, 4, 1), None, {"dual": 9, "primal": 9})}[name]
    P = P()
    a, b = (G.Problem(P, G.default_params(k_int=9, K_max=64, power_iters=5, autotune=0)) for _ in range(2))
    for p in (a, b):
        if cfg:
            p.set_launch_cfg(*cfg)
    kt = a.kernel_times(9, 64)
    b.pdhg_steps(9)
    b.sample_eval(64)
    want = {**steps, "sample": 1, "argmin_update": 1, "extract_best": 1}
    if P.Q is not None:
        want["eval_quad"] = 1
    got = {k: c for k, (ms, c) in kt.items() if c}
    for k in ("eval_cover", "eval_general", "reduce_cand"):    # by the rows' kinds and the tiles
        if k in got:
            want[k] = 1
    assert got == want
    assert all((ms > 0) == (c > 0) for ms, c in kt.values())
    assert ("eval_cover" in got or "eval_general" in got) == (P.m1 + P.m2 > 0)
    assert ("reduce_cand" in got) == (name in ("codes", "many_tiles"))
    assert not (name == "run" and "eval_general" in got) and not (name == "whole_steps" and "eval_cover" in got)
    sa, sb = a.get_state(), b.get_state()
    assert all(np.array_equal(sa[k], sb[k]) for k in ("x", "x_prev", "y")) and sa["k"] == sb["k"]
    a.close()
    b.close()


@pytest.mark.parametrize("sizes, launches", [([(2048, 24)], False), ([(2049, 3)], True), ([(600, 25)], True),
                                             ([(300, 5), (8000, 8)], True), ([(300, 5), (2000, 9)], False)])
def test_single_steps_of_wide_dense_rows_are_launches(G, sizes, launches):
    P = I.concat_instances([I.knapsack_multi(n, m, seed=n) for n, m in sizes])
    a, b = (G.Problem(P, G.default_params(k_int=9, K_max=64, power_iters=5, autotune=0)) for _ in range(2))
    assert _form(a) == RUN
    kt = {n: a.kernel_times(n, 64) for n in (1, 2)}
    assert kt[1]["dual"][1] == int(launches) and kt[1]["primal"][1] == 1
    assert kt[2]["dual"][1] == 0 and kt[2]["primal"][1] == 2
    a.reset()
    for n, res in ((1, False), (1, True), (4, False), (1, False), (2, True)):
        a.pdhg_steps(n, want_residuals=res)
    b.pdhg_steps(9, want_residuals=True)
    sa, sb = a.get_state(), b.get_state()
    assert all(np.array_equal(sa[k], sb[k]) for k in ("x", "x_prev", "y")) and sa["k"] == sb["k"]
    assert np.array_equal(a.residuals(), b.residuals())
    a.close()
    b.close()
