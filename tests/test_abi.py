"""The C-ABI library loads and exports every symbol include/hfmm.h declares;
host-only entry points behave as documented (no GPU needed)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "hfmm.h")
LIB = os.path.join(ROOT, "paper_1010_1482_amd", "libhfmm.so")


def declared_symbols():
    txt = open(HEADER).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(hfmm_[a-z_]+)\s*\(", txt)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        pytest.fail("libhfmm.so is not built (run __graft_entry__.build())")
    return C.CDLL(LIB)


def test_every_declared_symbol_is_exported(lib):
    syms = declared_symbols()
    assert len(syms) >= 15
    for s in syms:
        assert hasattr(lib, s), s


def test_binding_lists_every_symbol():
    from paper_1010_1482_amd import hfmm
    assert sorted(hfmm.SYMBOLS) == declared_symbols()


def test_host_only_entry_points(lib):
    from paper_1010_1482_amd import hfmm
    b = hfmm.arena_bytes(1 << 20, 0, 64, 10, hfmm.FMM, hfmm.FP32)
    assert b > (1 << 20) * 100
    assert hfmm.arena_bytes(1000, 0, 64, 4, hfmm.TREECODE, hfmm.FP64) > 0
    with pytest.raises(hfmm.HfmmError) as e:
        hfmm.arena_bytes(1000, 0, 64, 17, hfmm.FMM, hfmm.FP32)
    assert e.value.code == hfmm.E_UNSUPPORTED
    with pytest.raises(hfmm.HfmmError) as e:
        hfmm.arena_bytes(1000, 0, 0, 4, hfmm.FMM, hfmm.FP32)
    assert e.value.code == hfmm.E_INVAL
    lib.hfmm_strerror.restype = C.c_char_p
    assert lib.hfmm_strerror(-2) == b"arena too small"
    out = C.c_void_p()
    L = hfmm._lib()
    # null arena / negative sizes are rejected before any device work
    assert L.hfmm_build_tree(None, None, None, -1, 64, None, 0, None,
                             C.byref(out)) == hfmm.E_INVAL
    assert L.hfmm_build_tree(None, None, None, 10, 64, C.c_void_p(1), 1 << 20, None,
                             C.byref(out)) == hfmm.E_INVAL  # null coordinates
    assert L.hfmm_get_stats(None, None) == hfmm.E_INVAL
    # null tree handles
    assert L.hfmm_evaluate(None, None, None, None, 0, 4, 0.5, hfmm.FMM, hfmm.FP32, 0.0,
                           None, None, None, None, None) == hfmm.E_INVAL
    flags = C.c_uint32(7)
    assert L.hfmm_status(None, None, C.byref(flags)) == hfmm.E_INVAL and flags.value == 0
    assert L.hfmm_export_targets(None, None, None) == hfmm.E_INVAL
    assert L.hfmm_export_target_lists(None, 0, None, None, None) == hfmm.E_INVAL
    L.hfmm_strerror.restype = C.c_char_p
    assert b"overflow" in L.hfmm_strerror(hfmm.E_OVERFLOW)


def test_new_methods_and_time_loop_host_checks(lib):
    from paper_1010_1482_amd import hfmm
    assert hfmm.arena_bytes(1 << 20, 0, 64, 3, hfmm.TREECODE_FMMLIST, hfmm.FP32) > 0
    with pytest.raises(hfmm.HfmmError) as e:
        hfmm.arena_bytes(1000, 0, 64, 4, 7, hfmm.FP32)
    assert e.value.code == hfmm.E_UNSUPPORTED
    L = hfmm._lib()
    done = C.c_int(-1)
    arena = C.c_void_p(1)  # never dereferenced: every call below fails its checks
    # negative n, negative steps, NaN dt, null arena: rejected before device work
    for n, steps, dt, ar in ((-1, 1, 1e-3, arena), (10, -1, 1e-3, arena),
                             (10, 1, float("nan"), arena), (10, 1, 1e-3, None)):
        rc = L.hfmm_leapfrog(*([None] * 7), n, dt, steps, 64, 4, 0.5, hfmm.FMM, hfmm.FP32,
                             0.0, 0.0625, ar, 1 << 30, *([None] * 4), C.byref(done), None, None)
        assert rc == hfmm.E_INVAL and done.value == 0
    # n > 0 with null state pointers
    rc = L.hfmm_leapfrog(*([None] * 7), 10, 1e-3, 1, 64, 4, 0.5, hfmm.FMM, hfmm.FP32, 0.0,
                         -1.0, arena, 1 << 30, *([None] * 4), C.byref(done), None, None)
    assert rc == hfmm.E_INVAL
    # NaN slack
    rc = L.hfmm_leapfrog(*([None] * 7), 10, 1e-3, 1, 64, 4, 0.5, hfmm.FMM, hfmm.FP32, 0.0,
                         float("nan"), arena, 1 << 30, *([None] * 4), C.byref(done), None, None)
    assert rc == hfmm.E_INVAL
    # refit: null handle or output, negative or non-finite slack
    kept = C.c_int(7)
    assert L.hfmm_refit(None, None, None, None, 0.1, None, C.byref(kept)) == hfmm.E_INVAL
    assert kept.value == 0
    # n = 0: nothing to do, every step counted
    builds = C.c_int(-1)
    rc = L.hfmm_leapfrog(*([None] * 7), 0, 1e-3, 3, 64, 4, 0.5, hfmm.FMM, hfmm.FP32, 0.0,
                         0.0625, arena, 1 << 30, *([None] * 4), C.byref(done), C.byref(builds),
                         None)
    assert rc == hfmm.OK and done.value == 3 and builds.value == 0


def test_bench_refuses_more_than_one_gpu():
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "one GPU" in r.stderr


def test_treecode_arena_estimate(lib):
    from paper_1010_1482_amd import hfmm
    n = 1 << 22
    for leaf in (1, 2, 4, 8, 32):
        base = hfmm.arena_bytes(n, 0, leaf, 3, hfmm.TREECODE, hfmm.FP32)
        # some 250 bytes per particle and 750 per cell, a quarter more and 64 MB;
        # the lists, which depend on theta, are no part of it
        assert base < 1.25 * (300 * n + 800 * (4 * n / leaf + 4096)) + (64 << 20)
        est = [hfmm.arena_bytes(n, 0, leaf, 3, hfmm.TREECODE, hfmm.FP32, theta=t)
               for t in (0.0, 0.3, 0.5, 0.8, 1.0, 2.0, float("inf"))]
        assert est == sorted(est, reverse=True)
        assert est[-1] == base and est[0] <= base + 4 * 2 ** 31
    # bytes that whole calls on Plummer spheres took
    for lg, leaf, theta, need in ((22, 32, 0.5, 4769e6), (22, 32, 0.7, 2458e6),
                                  (22, 32, 1.0, 1398e6), (22, 8, 1.0, 3684e6),
                                  (20, 8, 0.5, 3670e6), (20, 32, 0.3, 3429e6),
                                  (20, 32, 0.5, 1122e6), (18, 8, 0.3, 2638e6),
                                  (16, 8, 0.3, 458e6), (14, 8, 0.3, 64e6)):
        est = hfmm.arena_bytes(1 << lg, 0, leaf, 3, "treecode", "fp32", theta=theta)
        assert need < est < 2.5 * need + (200 << 20), (lg, leaf, theta, est)
    # other methods know no theta
    assert hfmm.arena_bytes(n, theta=0.5) == hfmm.arena_bytes(n)


def test_fmm_arena_estimate_counts_whole_rows(lib):
    # multipoles, local expansions, P2L sums (FP64), an FP32 copy, the M2L
    # operand (p^2 floats and more) and twelve partial results per cell, in rows
    # of p^2 numbers padded to 16, a quarter more
    from paper_1010_1482_amd import hfmm
    n, leaf = 1 << 20, 64
    cells = 4 * n // leaf
    for prec in ("fp32", "fp64", "bf16x3", "fp16"):
        for p in range(6, 12):
            ldm = (p * p + 15) // 16 * 16
            rows = cells * (ldm * (3 * 8 + 4 + 12 * 4) + p * p * 4)
            # beyond the rows: 224 bytes and more per particle, 1300 per cell
            est = hfmm.arena_bytes(n, 0, leaf, p, "fmm", prec)
            assert est >= 1.25 * (rows + 224 * n + 1300 * cells), (prec, p)
    # an operator table of the same size does not hide it: orders 10 and 9 of
    # FP32 differ by the rows of 112 and 96 numbers at least
    d = (hfmm.arena_bytes(n, 0, leaf, 10, "fmm", "fp32") -
         hfmm.arena_bytes(n, 0, leaf, 9, "fmm", "fp32"))
    assert d >= 1.25 * cells * 16 * (3 * 8 + 4 + 12 * 4)
