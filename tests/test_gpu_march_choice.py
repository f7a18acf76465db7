"""Which levels march: levels beyond the boxes do only where that is predicted to pay.

A level of more than 64 planes or 2^20 cells is smoothed by blocks that march in z or by half-sweep
launches, whichever is predicted to take less time (FERROX_TB=1: the march wherever it can run,
0: no blocks).  The three give the same bits, also where marching and launched levels follow each
other; a stack with a semiconductor half is launched on levels whose march took longer.
"""
import numpy as np
import pytest

from paper_2210_15668_amd import workloads as W

pytestmark = pytest.mark.gpu

B, L = 1, 0                                        # LEVEL_BLOCKED, LEVEL_LAUNCHES
# lateral x, y, planes of ferroelectric, dielectric, semiconductor; the two finest levels' modes
CASES = [(80, 80, 76, 4, 70, (L, L)), (96, 96, 196, 4, 0, (B, B)), (64, 64, 146, 4, 150, (B, L))]


@pytest.mark.parametrize("prec", [W.PREC_FP64, W.PREC_MIXED])
@pytest.mark.parametrize("case", CASES)
def test_levels_march_where_it_pays(monkeypatch, case, prec):
    from paper_2210_15668_amd import ferrox as fx
    assert (fx.LEVEL_BLOCKED, fx.LEVEL_LAUNCHES) == (B, L)
    nx, ny, fe, de, sc, want = case
    layers = [(W.FE, fe, W.EPS_FE, 0.0), (W.DE, de, W.EPS_SIO2, 0.0)] + ([(W.SC, sc, W.EPS_SI, 1e24)] if sc else [])
    spec = W.layered(nx, ny, fe + de + sc + 2, layers, v_top=0.8, tol_rel=1e-12, prec=prec, max_cycles=400)
    P0 = W.random_P(spec, 73, amp=0.05)
    out, modes = {}, {}
    for tb in (None, "1", "0"):
        monkeypatch.delenv("FERROX_TB", raising=False)
        if tb:
            monkeypatch.setenv("FERROX_TB", tb)
        s = fx.Stack(spec, P0)
        modes[tb] = s.level_modes()
        info = s.run_steps(3, W.DT)
        out[tb] = (s.get(fx.FIELD_P), s.get(fx.FIELD_PHI), info.total_cycles)
        s.close()
    assert tuple(modes[None][:2]) == want
    assert tuple(modes["1"][:2]) == (B, B) and tuple(modes["0"][:2]) == (L, L)
    for tb in ("1", "0"):
        assert out[tb][2] == out[None][2]
        assert np.array_equal(out[tb][0], out[None][0]) and np.array_equal(out[tb][1], out[None][1])
