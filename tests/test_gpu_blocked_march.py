"""Blocked smoothing that marches in z: levels of more than 64 planes or 2^20 cells.

A level too large for boxes of whole columns is smoothed in 32 x 32 tiles of chunks of planes, with
all half-sweeps of a launch in flight over the planes.  The expressions are those of the half-sweep
launches (FERROX_TB=0), so the fields must agree bit for bit: on extents smaller than a box (a
cell then lies in it several times), on tiles cut off in x and y, on one chunk and on several
with a last one cut off, with semiconductor planes that start and end on even and odd planes.
"""
import numpy as np
import pytest

from paper_2210_15668_amd import workloads as W

pytestmark = pytest.mark.gpu

# lateral x, y, planes of ferroelectric, dielectric, semiconductor (no level with x and y both
# odd: there the periodic corner cells share a colour, and two runs differ in the last bits)
SHAPES = [(16, 16, 60, 6, 0), (18, 24, 50, 4, 9), (36, 50, 41, 7, 20), (72, 48, 130, 8, 3), (96, 160, 40, 9, 28)]


@pytest.mark.parametrize("prec", [W.PREC_FP64, W.PREC_MIXED])
@pytest.mark.parametrize("shape", SHAPES)
def test_marching_levels_equal_launches(monkeypatch, shape, prec):
    from paper_2210_15668_amd import ferrox as fx
    nx, ny, fe, de, sc = shape
    layers = [(W.FE, fe, W.EPS_FE, 0.0), (W.DE, de, W.EPS_SIO2, 0.0)] + ([(W.SC, sc, W.EPS_SI, 1e24)] if sc else [])
    spec = W.layered(nx, ny, fe + de + sc + 3, layers, v_top=0.8, tol_rel=1e-12, prec=prec, max_cycles=400)
    P0 = W.random_P(spec, 72, amp=0.05)
    out, modes = {}, {}
    for tb in ("1", "0"):
        monkeypatch.setenv("FERROX_TB", tb)
        s = fx.Stack(spec, P0)
        modes[tb] = s.level_modes()
        info = s.run_steps(3, W.DT)
        out[tb] = (s.get(fx.FIELD_P), s.get(fx.FIELD_PHI), info.total_cycles)
        s.close()
    assert modes["1"][0] == fx.LEVEL_BLOCKED
    assert fx.LEVEL_BLOCKED not in modes["0"]
    assert out["1"][2] == out["0"][2]
    assert np.array_equal(out["1"][0], out["0"][0]) and np.array_equal(out["1"][1], out["0"][1])
