"""The coarse kernel's levels at every number of cells per thread, and the boxes of 25 to 32 planes.

The coarse kernel keeps one, two or four red/black pairs of a level, or one, two or four cells of a
plainly stored one, in a thread's registers; plainly stored levels may take up to 152 KB of LDS, and
levels that fit one wave run without workgroup barriers.  The stacks take each of these, at level
sizes on either side of the limits; the trajectory must meet the oracle's to the 1e-10 of
tests/test_gpu_parity.py.
"""
import numpy as np
import pytest

from paper_2210_15668_amd import workloads as W

pytestmark = pytest.mark.gpu

FP64, MIXED = W.PREC_FP64, W.PREC_MIXED
# precision, lateral x, y, planes of ferroelectric, dielectric, semiconductor: the coarse levels
CASES = [(FP64, 16, 8, 11, 5, 0),       # red/black 16x8x16: 1024 pairs, one a thread
         (FP64, 16, 16, 8, 5, 0),       # 16x16x13: 1664 pairs, two a thread
         (MIXED, 16, 16, 9, 7, 0),      # 16x16x16: 2048 pairs, two a thread
         (MIXED, 16, 16, 16, 8, 0),     # 16x16x24: 3072 pairs, four a thread
         (FP64, 27, 21, 6, 5, 0),       # plain 27x21x6: 3402 cells, four a thread, and two on 27x21x3
         (FP64, 27, 19, 5, 3, 4),       # plain 27x19x6 and below with a semiconductor
         (MIXED, 45, 45, 5, 3, 0),      # plain 45x45x2: 4050 cells in 64 KB
         (MIXED, 43, 43, 6, 3, 6),      # plain 43x43x2: 3698 cells with a semiconductor, above 64 KB
         (FP64, 7, 9, 11, 5, 6),        # bottom 7x9x1: one wave, conjugate gradients
         (MIXED, 12, 20, 20, 6, 10),    # odd levels 3x5 under red/black ones
         (FP64, 66, 1, 20, 5, 10)]      # a single row, halved in x alone


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def stack(prec, nx, ny, fe, de, sc, **kw):
    layers = [(W.FE, fe, W.EPS_FE, 0.0), (W.DE, de, W.EPS_SIO2, 0.0)] + ([(W.SC, sc, W.EPS_SI, 1e24)] if sc else [])
    kw = {"v_top": -0.6, "tol_rel": 1e-13, "max_cycles": 400, **kw}
    return W.layered(nx, ny, fe + de + sc + 2, layers, prec=prec, **kw)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%dx%dx%d" % ("fp64" if c[0] == FP64 else "mixed", c[1], c[2],
                                                                     sum(c[3:])))
def test_coarse_levels_meet_the_oracle(orc, case):
    from paper_2210_15668_amd import ferrox as fx
    spec = stack(*case)
    P0 = W.random_P(spec, 84, amp=0.05)
    s = fx.Stack(spec, P0)
    info = s.run_steps(4, W.DT)
    P, phi = s.get(fx.FIELD_P), s.get(fx.FIELD_PHI)
    s.close()
    P_o, phi_o, _ = orc.run(spec, P0, 4, W.DT, tol=1e-13)
    print(f"  {case}: {info.total_cycles} cycles, P {rel(P, P_o):.1e} phi {rel(phi, phi_o):.1e}", flush=True)
    assert rel(P, P_o) <= 1e-10 and rel(phi, phi_o) <= 1e-10


@pytest.mark.parametrize("prec", [FP64, MIXED])
@pytest.mark.parametrize("shape", [(24, 18, 15, 4, 7), (40, 36, 20, 4, 8)])     # 26 and 32 planes
def test_boxes_of_four_cells_a_thread_equal_launches(monkeypatch, shape, prec):
    from paper_2210_15668_amd import ferrox as fx
    spec = stack(prec, *shape, tol_rel=1e-12)
    P0 = W.random_P(spec, 85, amp=0.05)
    out = {}
    for tb in ("1", "0"):
        monkeypatch.setenv("FERROX_TB", tb)
        s = fx.Stack(spec, P0)
        assert s.level_modes()[0] == (fx.LEVEL_BLOCKED if tb == "1" else fx.LEVEL_LAUNCHES)
        cycles = s.run_steps(4, W.DT).total_cycles
        out[tb] = (cycles, s.get(fx.FIELD_P), s.get(fx.FIELD_PHI))
        s.close()
    assert out["1"][0] == out["0"][0]
    assert np.array_equal(out["1"][1], out["0"][1]) and np.array_equal(out["1"][2], out["0"][2])
