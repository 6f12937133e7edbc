"""Long runs of steps, which replay a captured graph once a problem has launched
64 steps one by one, against the same steps launched singly: the same kernels in
the same order, so every bit of the state, the counter and the residuals agrees."""
import ctypes
import threading
import time

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


def _pair(G, kind):
    """Two problems of one launch shape each, neither of whose steps run in one workgroup."""
    prm = G.default_params(k_int=10, K_max=64, power_iters=5, autotune=0)
    if kind == "factorised":
        P = I.assignment_qap_like(40, seed=3, q_per_var=6.0, tree="random")
        return [G.TUReformulation(P, P.meta["tu_pivots"], factored=True).problem(prm) for _ in range(2)]
    P, cfg = {"csr": lambda: (I.set_cover_columns(20011, 1999, 5, 1), (16, 4, 1, 1, 0, 0, 0, 0)),
              "bitmaps": lambda: (I.set_cover_columns(600_000, 60_000, 5, 1), (1, 1, 8, 1, 1, 1, 2, 2)),
              "sliced": lambda: (I.set_cover_columns(600_000, 60_000, 5, 1), (1, 4, 8, 1, 1, 0, 1, 1)),
              "whole_steps": lambda: (I.concat_instances([I.knapsack_multi(n, 9, seed=n) for n in (5000, 777, 2048)]),
                                      (16, 4, 1, 1, 0, 0, 4, 5)),
              "codes": lambda: (I.max_cut_er(140_000, 4.0, seed=1), None)}[kind]()
    out = [G.Problem(P, prm) for _ in range(2)]
    for p in out:
        if cfg:
            p.set_launch_cfg(*cfg)
    return out


@pytest.mark.parametrize("kind", ["csr", "bitmaps", "sliced", "whole_steps", "codes", "factorised"])
def test_replayed_runs_equal_single_steps(G, kind):
    a, b = _pair(G, kind)
    for p in (a, b):                        # past the steps that are launched first (in runs too short for a graph)
        for _ in range(2):
            p.pdhg_steps(63)
    for odd in (0, 1):                      # from both buffers
        for p in (a, b):
            p.pdhg_steps(odd)
        for steps, res in ((64, False), (65, True), (97, False), (100, True)):
            a.pdhg_steps(steps, want_residuals=res)
            for _ in range(steps - 1):
                b.pdhg_steps(1)
            b.pdhg_steps(1, want_residuals=res)
            sa, sb = a.get_state(), b.get_state()
            for key in ("x", "x_prev", "y"):
                assert np.array_equal(sa[key], sb[key]), (odd, steps, key)
            assert sa["k"] == sb["k"]
            if res:
                assert np.array_equal(a.residuals(), b.residuals())
    for p in (a, b):                        # a round from the state that a replay left
        p.run_rounds(1, 64)
    assert np.array_equal(a.candidates(), b.candidates())
    a.close()
    b.close()


def test_first_long_run_of_a_problem_costs_no_graph(G):
    """A problem's first 64 steps in one call against 32 and 32, which are launches on every host
    (replays are faster than launches where the host is slow, so they are no measure here); after
    60 steps in short calls, since a new stream's first launches cost more."""
    P = I.set_cover_columns(30_000, 3_000, 3, seed=0)
    first, halves = [], []
    for _ in range(8):
        p = G.Problem(P, G.default_params(k_int=10, K_max=64, power_iters=5))
        for _ in range(2):
            p.pdhg_steps(30)
            p.synchronize()
        for out, runs in ((first, (64,)), (halves, (32, 32)), (halves, (32, 32))):
            t = time.perf_counter()
            for steps in runs:
                p.pdhg_steps(steps)
            p.synchronize()
            out.append(time.perf_counter() - t)
        p.close()
    assert min(first) <= 1.25 * min(halves), (first, halves)


@pytest.mark.parametrize("what", ["rounds", "steps", "creation"])
def test_a_given_stream_is_never_captured(G, what):
    """Captures run on a stream of the library's own: what other threads enqueue meanwhile on the
    stream that a problem was given (a step of another problem there) must not end in its graph.
    Another thread asks all the while whether the given stream is being captured."""
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream()
    handle, status = ctypes.c_void_p(stream.cuda_stream), ctypes.c_int(0)
    asked, seen, stop = [0], [0], threading.Event()

    def watch():
        while not stop.is_set():
            assert hip.hipStreamIsCapturing(handle, ctypes.byref(status)) == 0
            asked[0] += 1
            seen[0] += status.value != 0

    prm = G.default_params(k_int=300, K_max=64, power_iters=5, autotune=0)
    if what == "creation":                  # a factorised problem times its launches as replayed graphs
        prm.autotune = 1
        P = I.assignment_qap_like(40, seed=3, q_per_var=6.0, tree="random")
        T = G.TUReformulation(P, P.meta["tu_pivots"], factored=True)
    else:
        p = G.Problem(I.set_cover_columns(20011, 1999, 5, 1), prm, stream=stream)
        for _ in range(2):
            p.pdhg_steps(63)
        p.synchronize()
    thread = threading.Thread(target=watch)
    thread.start()
    for odd in range(6):
        if what == "rounds":
            p.set_launch_cfg(**p.launch_cfg())      # drops the graphs: the next rounds capture again
            p.run_rounds(1, 64)
        elif what == "steps":
            p.set_launch_cfg(**p.launch_cfg())
            p.pdhg_steps(64 + odd % 2)
        else:
            T.problem(prm, stream=stream).close()
    stream.synchronize()
    stop.set()
    thread.join()
    assert asked[0] > 100 and seen[0] == 0, (asked, seen)
    if what != "creation":
        p.close()


def test_captures_on_several_threads_and_after_the_last_problem(G):
    """Capture streams are shared by problems and threads and given back with the last problem."""
    P = I.set_cover_columns(20011, 1999, 5, 1)
    prm = G.default_params(k_int=10, K_max=64, power_iters=5, autotune=0)
    for _ in range(2):
        probs, out = [G.Problem(P, prm) for _ in range(6)], [None] * 6

        def work(i):
            for odd in range(4):
                probs[i].pdhg_steps(64 + odd % 2)
                probs[i].run_rounds(1, 64)
            out[i] = probs[i].get_state()["x"]

        threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert all(o is not None and np.array_equal(o, out[0]) for o in out)
        for p in probs:
            p.close()
