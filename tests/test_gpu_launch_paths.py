"""Which launches a handle runs: lbm_launch_steps at both sides of each size where
the library changes to launches of its own, after a shape is set and after the
autotuner; and three FP64 steps per launch of a periodic problem.  (That every
path gives the bits of single steps is tested beside this.)
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


def _cavity(nx, ny, qt=9):
    return dict(W.scaled_cavity(W.case_c2()[0], nx, ny), thermal_lattice=qt)


def _channel(nx, ny, qt=9):
    return W.make_params(nx=nx, ny=ny, bc_x=1, gravity_axis=0, porosity=0.9, Ra=100.0, Pr=5.0, Da=0.05, Ste=1.0,
                         k_ratio=1.0, cap_ratio=1.0, Nu_i=0.0, k_f=0.02, T_hot=1.0, T_cold=0.0, T_init=1.0,
                         T_solidus=-2.0, T_liquidus=-1.0, thermal_lattice=qt)


# storage, cavities, steps per launch and, for launches a caller can't ask for, the tile
RULES = [
    ("f32h64", [_cavity(64, 64)], (6, 8, 8)),
    ("f32h64", [_cavity(128, 128)], (6, 8, 8)),            # 256 tiles
    ("f32h64", [_cavity(129, 128)], (6, 12, 12)),
    ("f32h64", [_cavity(200, 200)], (6, 16, 12)),
    ("f32h64", [_cavity(256, 256)], (5, 16, 16)),
    ("f32h64", [_cavity(257, 256)], (3, 32, 10)),
    ("f32", [_cavity(256, 256, 5)], (5, 16, 16)),
    ("f64", [_cavity(64, 64)], (5, 8, 8)),
    ("f64", [_cavity(151, 151)], (4, 16, 8)),
    ("f64", [_cavity(256, 256, 5)], (4, 16, 16)),
    ("f64", [_cavity(257, 256)], (2,)),             # 288 three-step tiles
    ("f64", [_cavity(300, 300)], (2,)),             # 380
    ("f64", [_cavity(384, 256)], (3, 32, 8)),              # 384
    ("f64", [_cavity(257, 256, 5)], (3, 32, 10)),
    ("f64", [_cavity(128, 64), _cavity(128, 64)], (5, 8, 8)),
    ("f64", [_cavity(384, 200), _cavity(384, 56)], (3, 32, 8)),
    ("f64", [_cavity(65, 65)] * 30, (2,)),                 # 810, all at walls, 4 on the fullest CU against 5
    ("f64", [_cavity(20000, 4)], (2,)),
    ("f64", [_cavity(500, 300)], (3, 32, 8)),              # 608, a sixth at walls
    ("f64", [_cavity(64, 64)] * 64, (3, 32, 8)),           # 1024, all at walls, 4 against 7
    ("f64", [_channel(280, 685)], (3, 32, 8)),             # walls at the bottom and the top only
    ("f64", [_cavity(65, 65, 5)] * 30, (3, 32, 10)),
    ("f64", [_channel(64, 64)], (2,)),              # periodic: not deep
    ("f32h64", [_channel(64, 64)], (3, 32, 10)),
    ("f64", [_channel(320, 330)], (3, 32, 8)),
    ("f16split", [_cavity(64, 64)], (3,)),          # no deep form
]


@pytest.mark.parametrize("i", range(len(RULES)))
def test_launches_by_size(lbm, i):
    prec, ps, want = RULES[i]
    s = lbm.Solver(ps if len(ps) > 1 else ps[0], prec)
    got, lc = lbm.lbm_launch_steps(s.h), lbm.lbm_get_launch(s.h)
    if len(want) == 1:     # the shape a caller may set, with its tile
        assert got == (*want, lc["tile_w"], lc["tile_h"]) and want[0] == lc["steps_per_launch"]
    else:
        assert got == want
    # a shape that is set is the shape that runs
    for spl in (1, 2):
        lbm.lbm_set_launch(s.h, 512, 1, 1, 0, steps_per_launch=spl, tile_shape=0)
        lc = lbm.lbm_get_launch(s.h)
        assert lbm.lbm_launch_steps(s.h) == (spl, lc["tile_w"], lc["tile_h"])
    # and the way back, bit for bit like a handle that never left
    assert lbm.lbm_reset_launch(s.h) == got[0] and lbm.lbm_launch_steps(s.h) == got
    t = lbm.Solver(ps if len(ps) > 1 else ps[0], prec)
    assert lbm.lbm_get_launch(s.h) == lbm.lbm_get_launch(t.h)
    s.step(23), t.step(23)
    assert np.array_equal(s.state(), t.state())
    s.close()
    t.close()


def test_autotuned_launches_are_reported(lbm, tmp_path):
    # whichever is chosen, a second handle that reads the choice runs the same
    path, seen = str(tmp_path / "tune.txt"), []
    for _ in range(2):
        s = lbm.Solver(_cavity(64, 64), "f64")
        s.step(7)
        lc = lbm.lbm_autotune(s.h, 20, path)
        seen.append(lbm.lbm_launch_steps(s.h))
        assert seen[-1][0] > 3 or seen[-1] == (lc["steps_per_launch"], lc["tile_w"], lc["tile_h"])
        s.close()
    assert seen[0] == seen[1]


@pytest.mark.parametrize("qt", [9, 5])
def test_three_fp64_steps_of_a_periodic_problem_are_single_steps(lbm, qt):
    p, out = _channel(320, 330, qt), []
    for spl in (1, None):
        s = lbm.Solver(p, "f64")
        if spl:
            lbm.lbm_set_launch(s.h, 512, 1, 1, 0, steps_per_launch=spl, tile_shape=0)
        else:
            assert lbm.lbm_launch_steps(s.h)[0] == 3
        s.set_initial(0, *W.initial_temperatures(p, 30, amplitude=1e-2))
        for n in (1, 3, 4, 5, 100, 1):
            s.step(n)
        out.append((s.state(), s.diagnostics()))
        s.close()
    assert np.array_equal(out[0][0], out[1][0])
    for k in ("flux_E", "flux_M", "E_int", "M_int", "liquid_fraction"):
        assert out[0][1][k] == out[1][1][k], k
