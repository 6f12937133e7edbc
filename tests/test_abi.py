"""The C-ABI library loads and exports every entry point include/gfors.h declares
(no device work: this runs without a GPU)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "gfors.h")
LIB = os.path.join(ROOT, "paper_2510_27117_amd", "libgfors.so")


def declared_symbols():
    txt = open(HEADER).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(gfors_[a-z_0-9]+)\s*\(", txt)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2510_27117_amd import build
        build.build()
    return ctypes.CDLL(LIB)


def test_every_declared_symbol_is_exported(lib):
    syms = declared_symbols()
    assert len(syms) >= 15
    for s in syms:
        assert hasattr(lib, s), s


def test_binding_names_cover_header():
    from paper_2510_27117_amd import gfors
    assert sorted(gfors.EXPORTS) == declared_symbols()


def test_default_params_and_workspace_size(lib):
    from paper_2510_27117_amd import gfors
    p = gfors.default_params()
    assert p.sigma == 0.99 and p.K_max == 1024 and p.k_int == 100 and p.power_iters == 200
    L = gfors.load_library()
    nb = ctypes.c_size_t(0)
    assert L.gfors_workspace_bytes(2_000_000, 200_000, 0, 10_000_000, 0, 0, 1,
                                   ctypes.byref(p), ctypes.byref(nb)) == 0
    # candidates alone take n * K/64 * 8 bytes
    assert nb.value > 2_000_000 * 16 * 8
    # bad K_max is rejected with a message
    p.K_max = 100
    assert L.gfors_workspace_bytes(10, 1, 0, 1, 0, 0, 1, ctypes.byref(p), ctypes.byref(nb)) == -1
    assert b"K_max" in L.gfors_last_error()
    p.K_max = 1024
    assert L.gfors_workspace_bytes(0, 1, 0, 1, 0, 0, 1, ctypes.byref(p), ctypes.byref(nb)) == -1


def test_missing_library_fails_loudly(tmp_path):
    from paper_2510_27117_amd import gfors
    saved = gfors._lib
    gfors._lib = None
    try:
        with pytest.raises(RuntimeError):
            gfors.load_library(str(tmp_path / "nope.so"))
    finally:
        gfors._lib = saved


@pytest.mark.parametrize("n, m1, m2, nnzA, nnzB, nnzQ, T, K, most", [
    (200, 100, 0, 1000, 0, 0, 1, 256, 417288),
    (64, 8, 0, 64, 0, 64, 1, 64, 138248),
    (1024, 0, 0, 0, 0, 4096, 1, 64, 321544),
    (200000, 0, 0, 0, 0, 2000000, 1, 2048, 180002056),
    (3000, 300, 10, 30000, 100, 0, 3, 1024, 3208720),
    (40000, 20000, 0, 400000, 0, 0, 1024, 64, 70235140),
    (300000, 30000, 0, 3000000, 0, 0, 5000, 512, 517837604),
    (2000000, 200000, 0, 10000000, 0, 0, 1, 1024, 1345622280)])
def test_workspace_does_not_grow(n, m1, m2, nnzA, nnzB, nnzQ, T, K, most):
    """A problem that fits a workspace (the static one among them) keeps fitting."""
    from paper_2510_27117_amd import gfors
    prm, out = gfors.default_params(K_max=K), ctypes.c_size_t()
    assert gfors.load_library().gfors_workspace_bytes(n, m1, m2, nnzA, nnzB, nnzQ, T, ctypes.byref(prm), ctypes.byref(out)) == 0
    assert out.value <= most


def _factored(name):
    import numpy as np
    from paper_2510_27117_amd import gfors, instances as I
    if name == "long_rows":          # more chunks of long rows than pivots
        P = I.assignment_qap_like(20, seed=3, q_per_var=4.0, tree="random")
        P.A = I.csr_from_dense(-np.random.default_rng(0).integers(1, 9, (300, P.n)))
        P.b = np.full(300, -900, dtype=np.int64)
    else:
        P = I.assignment_qap_like(int(name), seed=3, q_per_var=6.0, tree="random")
    return gfors.TUReformulation(P, P.meta["tu_pivots"], factored=True)


@pytest.mark.parametrize("name, most", [("12", 389636), ("40", 1014532), ("long_rows", 3337392)])
def test_workspace_of_the_factorised_form_does_not_grow(name, most):
    from paper_2510_27117_amd import gfors
    T, prm, out = _factored(name), gfors.default_params(K_max=256), ctypes.c_size_t()
    assert gfors.load_library().gfors_workspace_bytes_tu(T.handle, ctypes.byref(prm), ctypes.byref(out)) == 0
    assert out.value <= most
