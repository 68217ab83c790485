"""Field planes through pinned slots and several threads equal the planes
copied one at a time, which go the other way: pieces that fill no slot, one, all
of them and several rounds, ragged last pieces, the longest rows, batches.
"""
import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu
NAMES = ("ux", "uy", "T_pcm", "T_mf", "f_l", "rho")


@pytest.fixture(scope="module")
def lbm(require_gpu):
    import torch
    torch.cuda.set_device(0)
    from paper_1701_00702_amd import lbm as mod
    return mod


def _planes(lbm, s, c, y0, rows):
    nx = s.shape(c)[1]
    out = {}
    for i, k in enumerate(NAMES):
        out[k] = np.full((rows, nx), -7.0)
        lbm._check(lbm._lib.lbm_fields_rows(s.h, c, y0, rows, *[lbm._dptr(out[k]) if j == i else None for j in range(6)]))
    return out


@pytest.mark.parametrize("prec", ["f64", "f32h64", "f16split"])
@pytest.mark.parametrize("sizes", [[(4, 4)], [(256, 512)], [(257, 1030)], [(1000, 1701)], [(131072, 5)], [(131073, 5)],
                                   [(40, 30), (1025, 600), (4, 9)]])
def test_planes_through_slots_are_the_planes(lbm, sizes, prec):
    ps = [W.scaled_cavity(W.case_c2()[0], nx, ny) for nx, ny in sizes]
    s = lbm.Solver(ps if len(ps) > 1 else ps[0], prec)
    for c, q in enumerate(ps):
        s.set_initial(c, *W.initial_temperatures(q, 30 + c, amplitude=1e-2))
    for n in (0, 3):
        s.step(n)
        for c, (nx, ny) in enumerate(sizes):
            whole, part = s.fields(c), s.fields_rows(ny // 3, ny - 1 - ny // 3, c)
            for k, v in _planes(lbm, s, c, 0, ny).items():
                assert np.array_equal(whole[k], v), k
                assert np.array_equal(part[k], v[ny // 3:ny - 1]), k
    s.close()
