"""Blocked smoothing on the finest level and on extents that the tiles do not divide.

The finest level of a small stack runs its sweeps, transfers and Newton update in two launches
over 8 x 8 column tiles.  The expressions are those of the half-sweep launches (FERROX_TB=0), so
the fields must agree bit for bit: on the smallest extents a box fits (16), on tiles cut off in
x and y (the next level may then be odd and plainly stored), on every number of planes per
thread up to the most a box holds (64), with semiconductor planes and light cycles.
"""
import numpy as np
import pytest

from paper_2210_15668_amd import workloads as W

pytestmark = pytest.mark.gpu

# lateral x, y, planes of ferroelectric, dielectric, semiconductor (no level with x and y both
# odd: there the periodic corner cells share a colour, and two runs differ in the last bits)
SHAPES = [(16, 16, 4, 3, 0), (18, 24, 10, 4, 0), (20, 48, 16, 4, 3), (16, 50, 20, 5, 9), (36, 16, 30, 7, 10),
          (34, 20, 32, 8, 24)]


@pytest.mark.parametrize("prec", [W.PREC_FP64, W.PREC_MIXED])
@pytest.mark.parametrize("shape", SHAPES)
def test_blocked_finest_level_equals_launches(monkeypatch, shape, prec):
    from paper_2210_15668_amd import ferrox as fx
    nx, ny, fe, de, sc = shape
    layers = [(W.FE, fe, W.EPS_FE, 0.0), (W.DE, de, W.EPS_SIO2, 0.0)] + ([(W.SC, sc, W.EPS_SI, 1e24)] if sc else [])
    # 64 KB of level data keep small FP32 stacks wholly inside the coarse kernel: those have
    # no launches on the finest level to compare
    spec = W.layered(nx, ny, fe + de + sc + 3, layers, v_top=0.8, tol_rel=1e-12, prec=prec, max_cycles=400)
    P0 = W.random_P(spec, 71, amp=0.05)
    out, modes = {}, {}
    for tb in ("1", "0"):
        monkeypatch.setenv("FERROX_TB", tb)
        s = fx.Stack(spec, P0)
        modes[tb] = s.level_modes()
        info = s.run_steps(6, W.DT)
        out[tb] = (s.get(fx.FIELD_P), s.get(fx.FIELD_PHI), info.total_cycles)
        s.close()
    in_coarse = modes["0"][0] == fx.LEVEL_COARSE
    assert modes["1"][0] == (fx.LEVEL_COARSE if in_coarse else fx.LEVEL_BLOCKED)
    assert fx.LEVEL_BLOCKED not in modes["0"]
    assert out["1"][2] == out["0"][2]
    assert np.array_equal(out["1"][0], out["0"][0]) and np.array_equal(out["1"][1], out["0"][1])
