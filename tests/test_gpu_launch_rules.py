"""Launches whose size takes the library to another path than the small
geometries of the other tests: tiles ordered in several strips, workgroups
that fetch for a later tile.  Every path gives the bits of single steps.
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
