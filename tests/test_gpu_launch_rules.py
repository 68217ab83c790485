"""Launches whose size takes the library to another path than the small
geometries of the other tests: tiles ordered in several strips, workgroups
that fetch for a later tile, deep launches, three FP64 steps per launch.  Every path gives the bits of single steps.
"""
import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm(require_gpu):
    import torch
    torch.cuda.set_device(0)
    from paper_1701_00702_amd import lbm as mod
    return mod


def _cavity(nx, ny, qt):
    return dict(W.scaled_cavity(W.case_c2()[0], nx, ny), thermal_lattice=qt)


def _run(lbm, ps, prec, steps, spl=None):
    s = lbm.Solver(ps if len(ps) > 1 else ps[0], prec)
    if spl:
        lbm.lbm_set_launch(s.h, 512, 1, 1, 0, steps_per_launch=spl, tile_shape=0)
    for c, q in enumerate(ps):
        s.set_initial(c, *W.initial_temperatures(q, 30 + c, amplitude=1e-2))
    s.step(steps)
    out = [(s.state(c), s.diagnostics(c)) for c in range(len(ps))]
    s.close()
    return out


def _same(a, b):
    for (x, dx), (y, dy) in zip(a, b):
        assert np.array_equal(x, y)
        for k in ("flux_E", "flux_M", "E_int", "M_int", "liquid_fraction"):
            assert dx[k] == dy[k], k


@pytest.mark.parametrize("prec,qt", [("f32h64", 9), ("f32", 9), ("f32", 5), ("f32h64", 5), ("f16split", 9), ("f16", 9)])
@pytest.mark.parametrize("sizes", [[(1601, 1030)], [(1000, 700), (64, 64), (1700, 640)]], ids=["one", "batch"])
def test_many_rounds_of_tiles_are_bitwise_single_steps(lbm, prec, qt, sizes):
    # over three rounds of tiles (fetching ahead), 50 and 53 tile columns (two strips), ragged edges
    ps = [_cavity(nx, ny, qt) for nx, ny in sizes]
    _same(_run(lbm, ps, prec, 20, 1), _run(lbm, ps, prec, 20))


DEEP = {
    "smallest": lambda q: [_cavity(4, 4, q)],
    "thin": lambda q: [_cavity(5, 37, q)],
    "256 smallest tiles": lambda q: [_cavity(128, 128, q)],
    "one column more": lambda q: [_cavity(129, 128, q)],
    "151": lambda q: [_cavity(151, 151, q)],
    "193x191": lambda q: [_cavity(193, 191, q)],
    "256 largest tiles": lambda q: [_cavity(256, 256, q)],
    "not deep": lambda q: [_cavity(257, 256, q)],
    "corner walls": lambda q: [dict(W.case_corner(100)[0], thermal_lattice=q)],
    "bounce-back": lambda q: [dict(_cavity(41, 60, q), solid_treatment=1)],
    "batch": lambda q: [_cavity(33, 70, q), _cavity(64, 48, q), _cavity(16, 16, q)],
    "bands": lambda q: [dict(_cavity(70, 150, q), band_rows=34)],
}


@pytest.mark.parametrize("prec", ["f64", "f32", "f32h64"])
@pytest.mark.parametrize("qt", [9, 5])
@pytest.mark.parametrize("case", list(DEEP))
def test_small_handles_are_bitwise_single_steps(lbm, case, qt, prec):
    # handles of at most 256 small tiles run deep launches; every count of
    # steps up to a launch's most, a replayed graph and a remainder of one
    ps = DEEP[case](qt)
    chunks = [1, 2, 3, 4, 5, 6, 7, 197, 1]
    ref = _run(lbm, ps, prec, sum(chunks), 1)
    s = lbm.Solver(ps if len(ps) > 1 else ps[0], prec)
    for c, q in enumerate(ps):
        s.set_initial(c, *W.initial_temperatures(q, 30 + c, amplitude=1e-2))
    for n in chunks:
        s.step(n)
    got = [(s.state(c), s.diagnostics(c)) for c in range(len(ps))]
    s.close()
    _same(ref, got)


def test_autotune_keeps_or_leaves_the_deep_launches(lbm, tmp_path):
    # whichever it picks, the bits stay, and the cached choice is taken again
    p = _cavity(64, 64, 9)
    ref = _run(lbm, [p], "f32h64", 200, 1)
    path = str(tmp_path / "tune.txt")
    for _ in range(2):
        s = lbm.Solver(p, "f32h64")
        s.set_initial(0, *W.initial_temperatures(p, 30, amplitude=1e-2))
        s.step(7)
        lbm.lbm_autotune(s.h, 3, path)
        s.step(193)
        _same(ref, [(s.state(0), s.diagnostics(0))])
        s.close()
    assert len(open(path).read().splitlines()) == 1


FP64 = {
    "380 tiles, D2Q9 two steps": lambda q: [_cavity(300, 300, q)],
    "384 tiles": lambda q: [_cavity(384, 256, q)],
    "ragged": lambda q: [_cavity(701, 613, q)],
    "rounds of tiles": lambda q: [_cavity(1601, 1030, q)],
    "batch": lambda q: [_cavity(333, 270, q), _cavity(64, 48, q), _cavity(5, 400, q)],
    "bands": lambda q: [dict(_cavity(370, 350, q), band_rows=34)],
    "periodic": lambda q: [W.make_params(nx=6, ny=17, bc_x=1, gravity_axis=0, porosity=0.9, Ra=100.0, Pr=5.0,
                                         Da=0.05, Ste=1.0, k_ratio=1.0, cap_ratio=1.0, Nu_i=0.0, k_f=0.02,
                                         T_hot=1.0, T_cold=0.0, T_init=1.0, T_solidus=-2.0, T_liquidus=-1.0,
                                         thermal_lattice=q)],
}


@pytest.mark.parametrize("qt", [9, 5])
@pytest.mark.parametrize("case", list(FP64))
def test_own_fp64_launches_are_bitwise_single_steps(lbm, case, qt):
    # beyond the deep sizes: every remainder of three steps, a replayed graph
    ps = FP64[case](qt)
    chunks = [1, 3, 4, 5, 100, 1]
    ref = _run(lbm, ps, "f64", sum(chunks), 1)
    s = lbm.Solver(ps if len(ps) > 1 else ps[0], "f64")
    assert lbm.lbm_get_launch(s.h)["steps_per_launch"] == 2
    for c, q in enumerate(ps):
        s.set_initial(c, *W.initial_temperatures(q, 30 + c, amplitude=1e-2))
    for n in chunks:
        s.step(n)
    got = [(s.state(c), s.diagnostics(c)) for c in range(len(ps))]
    with pytest.raises(lbm.LbmError):
        lbm.lbm_set_launch(s.h, 512, 1, 1, 0, steps_per_launch=3, tile_shape=0)
    s.close()
    _same(ref, got)


def test_autotune_of_an_fp64_handle_keeps_the_bits(lbm, tmp_path):
    p = _cavity(400, 333, 5)
    ref = _run(lbm, [p], "f64", 120, 1)
    path = str(tmp_path / "tune.txt")
    for _ in range(2):
        s = lbm.Solver(p, "f64")
        s.set_initial(0, *W.initial_temperatures(p, 30, amplitude=1e-2))
        s.step(8)
        assert lbm.lbm_autotune(s.h, 3, path)["steps_per_launch"] in (1, 2)
        s.step(112)
        _same(ref, [(s.state(0), s.diagnostics(0))])
        s.close()
    assert len(open(path).read().splitlines()) == 1
