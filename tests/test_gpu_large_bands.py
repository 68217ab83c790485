"""GPU checks of bands of more than a gigabyte, across whose boundary a tile
reaches further than 2^31 bytes from its first block: FP64 rows of 200 000
nodes against the oracle, and a large band_rows against the automatic bands, bit
for bit, with one, two and three steps per launch and with the library's own
launches.
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


def _run(lbm, p, prec, T, steps, spl):
    s = lbm.Solver(p, prec)
    if spl:
        lbm.lbm_set_launch(s.h, 512, 1, 1, 0, steps_per_launch=spl, tile_shape=0)
    s.set_initial(0, *T)
    s.step(steps)
    out = s.state(), s.fields(), s.diagnostics()
    s.close()
    return out


def test_long_fp64_rows_match_the_oracle(lbm):
    import oracle
    from test_gpu_parity import field_errors
    p = dict(W.scaled_cavity(W.case_c1()[0], 200000, 70), L_char=127.0)
    T = W.initial_temperatures(p, 4)
    o = oracle.Oracle(p)
    o.set_initial(*T)
    o.step(9)
    r = o.fields()
    first = None
    for spl in (1, 2, None):
        print(f"200000x70 FP64, steps per launch: {spl or 'own'}", flush=True)
        state, f, _ = _run(lbm, p, "f64", T, 9, spl)
        e = field_errors(f, r, p)
        assert max(e.values()) < 1e-10, (spl, e)
        assert first is None or np.array_equal(first, state), spl
        first = state
    del o


# one band of band_rows rows (above 2^30 bytes) and a short one
@pytest.mark.parametrize("prec,qt,ny,rows", [("f64", 9, 740, 700), ("f64", 5, 950, 900), ("f32", 9, 1300, 1250),
                                             ("f32h64", 9, 1300, 1250), ("f16split", 9, 1900, 1850)])
def test_large_bands_give_the_bits_of_automatic_bands(lbm, prec, qt, ny, rows):
    p = dict(W.scaled_cavity(W.case_c2()[0], 8192, ny), thermal_lattice=qt)
    T = W.initial_temperatures(p, 30, amplitude=1e-2)
    ref, _, d = _run(lbm, p, prec, T, 13, 1)
    assert d["nonfinite"] == 0
    for spl in (1, 2, None) if prec == "f64" else (1, 2, 3, None):
        print(f"8192x{ny} {prec} D2Q{qt}, bands of {rows} rows, steps per launch: {spl or 'own'}", flush=True)
        state, _, e = _run(lbm, dict(p, band_rows=rows), prec, T, 13, spl)
        assert np.array_equal(ref, state), spl
        for k in ("flux_E", "flux_M", "E_int", "M_int", "liquid_fraction"):
            assert d[k] == e[k], (spl, k)
