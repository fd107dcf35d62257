"""The library's own choice of lanes per instance (lane schedule), read from the
built library on the CPU."""
import ctypes as C

import pytest

from paper_2602_19699_amd import cbic, inputs as I

PM, ARM, LQ = (I.SYS_POINT_MASS, 4, 2), (I.SYS_PLANAR3, 6, 3), (I.SYS_LQ, 6, 3)


def choice(system, B, ragged, **o):
    """(lanes per instance, trials per line-search round)"""
    lib = C.CDLL(cbic.LIB_PATH)
    find, default = lib._ZN4cbic13find_launcherEiiiii, lib._ZN4cbic13default_groupEPKNS_8LauncherEiPK15cbic_solve_optsbi
    find.restype = C.c_void_p
    opts = cbic.Options(**o)
    L = find(*system, opts.precision, 0)
    oc = opts.c()
    code = default(C.c_void_p(L), B, C.byref(oc), ragged, 0)
    return code & 0xFF, (code >> 8) or (code & 0xFF)


def rounds(B):
    t = 1
    while t < 16 and 2 * t * B <= 65536:
        t *= 2
    return t


@pytest.mark.parametrize("B", [1, 4096, 4097, 8192, 8193, 16384, 16385, 32768, 32769, 65536, 1 << 20, 2**31 - 1])
@pytest.mark.parametrize("form", [{}, dict(u_max=4.0), dict(regularization=1), dict(u_max=4.0, regularization=1)],
                         ids=["clip", "bound", "lm", "bound_lm"])
def test_choice_is_a_kernel_and_keeps_the_rounds(B, form):
    # the launcher has kernels of these (lanes, trials) pairs, see lane_launch.hpp
    kernels = {(g, g) for g in (1, 2, 4, 8, 16)} | {(8, 1), (8, 2), (8, 4), (16, 8)}
    for system in (PM, ARM, LQ):
        for prec in (0, 1):
            for ragged in (False, True):
                for stop, it in ((0, 6), (0, 20), (0, 50), (1, 20), (1, 50)):
                    lanes, trials = choice(system, B, ragged, precision=prec, stop_mode=stop, max_iter=it, **form)
                    assert trials == rounds(B)
                    assert (lanes, trials) in kernels | ({(16, 4)} if system is ARM and prec else set())
                    assert system is not LQ or lanes == trials


@pytest.mark.parametrize("system,prec,B", [(ARM, 1, 12000), (ARM, 1, 16384), (ARM, 1, 32768), (ARM, 1, 65536),
                                           (ARM, 0, 4097), (ARM, 0, 16384), (ARM, 0, 32768), (ARM, 0, 65536),
                                           (PM, 1, 8192), (PM, 1, 32768), (PM, 1, 65536), (PM, 0, 8192), (PM, 0, 65536)])
def test_even_batches_that_fill_the_chip_keep_narrow_groups(system, prec, B):
    # one horizon and a short fixed budget: groups wider than their rounds took
    # up to 1.5 times as long (with the arm's bound 2.1 times)
    forms = [{}, dict(u_max=4.0)] if system is ARM else [{}]
    for form in forms:
        assert choice(system, B, False, precision=prec, max_iter=6, **form) == (rounds(B), rounds(B)), form


@pytest.mark.parametrize("system,prec,B,lanes", [(ARM, 1, 8192, 16), (ARM, 1, 16384, 16), (ARM, 1, 65536, 8),
                                                 (ARM, 0, 8192, 16), (ARM, 0, 16384, 8), (PM, 1, 8192, 16),
                                                 (PM, 1, 32768, 8), (PM, 0, 16384, 8)])
def test_ragged_batches_take_wide_groups(system, prec, B, lanes):
    assert choice(system, B, True, precision=prec) == (lanes, rounds(B))


@pytest.mark.parametrize("prec,B", [(1, 16384), (1, 65536), (0, 16384), (0, 65536)])
def test_long_budgets_of_the_point_mass_take_wide_groups(prec, B):
    # converged instances freeze on the way: as with a tolerance stop
    for o in (dict(max_iter=50), dict(max_iter=8, stop_mode=1)):
        assert choice(PM, B, False, precision=prec, **o) == (8, rounds(B))


@pytest.mark.parametrize("B", [64, 5000, 8193, 16384, 40000])
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
def test_the_autotuner_times_the_own_choice(B, ragged, prec):
    # each width with as many trials as lanes, and what an untuned solve takes,
    # so that a tuned solve is no slower than an untuned one
    lib = C.CDLL(cbic.LIB_PATH)
    find, cands = lib._ZN4cbic13find_launcherEiiiii, lib._ZN4cbic15tune_candidatesEPKNS_8LauncherEiPK15cbic_solve_optsbiPi
    find.restype = C.c_void_p
    oc = cbic.Options(precision=prec).c()
    for system in (PM, ARM, LQ):
        out = (C.c_int * 8)()
        n = cands(C.c_void_p(find(*system, prec, 0)), B, C.byref(oc), ragged, 0, out)
        got = [(c & 0xFF, (c >> 8) or (c & 0xFF)) for c in out[:n]]
        assert got[:5] == [(g, g) for g in (1, 2, 4, 8, 16)] and len(set(got)) == n
        assert choice(system, B, ragged, precision=prec) in got
    n = cands(C.c_void_p(find(I.SYS_QUAD_SYNTH, 37, 12, prec, 0)), B, C.byref(oc), ragged, 0, out)
    assert list(out[:n]) == ([1, 2] if prec else [1])
