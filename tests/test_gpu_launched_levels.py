"""The launches of levels that are not smoothed in blocks.

Most levels run in blocks, so the launches they replace are compared here with FERROX_TB=0, which
every case asserts to have left no blocked level: the prolongation by coarse columns against the
one by fine cells, and tuned launch shapes against the default ones, bit for bit on a stack and
in a batch.
"""
import numpy as np
import pytest

from paper_2210_15668_amd import workloads as W

pytestmark = pytest.mark.gpu

PRECS = [W.PREC_FP64, W.PREC_MIXED]


def stacks(prec):
    """A stack with two levels above 2^18 cells, and a batch with odd plane counts and both time orders."""
    large = W.shrink_lateral(W.mfism_large(prec), 160, 160).copy(tol_rel=1e-12)
    batch = [W.layered(96, 64, 48, [(W.FE, 30, W.EPS_FE, 0.0), (W.DE, 4, W.EPS_SIO2, 0.0)], v_top=0.5,
                       tol_rel=1e-12, prec=prec),
             W.layered(48, 32, 47, [(W.FE, 24, W.EPS_FE, 0.0), (W.DE, 4, W.EPS_SIO2, 0.0),
                                    (W.SC, 11, W.EPS_SI, 1e24)], v_top=-0.8, tol_rel=1e-12, time_order=2, prec=prec)]
    return large, batch


def run(fx, prec, tune=None):
    large, specs = stacks(prec)
    s = fx.Stack(large, W.random_P(large, 94, amp=0.05))
    b = fx.Batch(specs, [W.random_P(sp, 95 + q, amp=0.05) for q, sp in enumerate(specs)])
    levels = s.level_modes()
    assert levels[0] == levels[1] == fx.LEVEL_LAUNCHES and fx.LEVEL_BLOCKED not in levels
    modes = b.level_modes(2)
    assert modes[0] == fx.LEVEL_LAUNCHES and fx.LEVEL_BLOCKED not in modes
    if tune:
        for x in (s, b):
            info = x.autotune(tune)
            assert info.configs_timed >= info.levels >= 1
    cycles = s.run_steps(4, W.DT).total_cycles
    assert all(i.status == fx.FX_OK for i in b.run(4, W.DT))
    out = [s.get(fx.FIELD_P), s.get(fx.FIELD_PHI)]
    for q in range(len(specs)):
        out += [b.get(q, fx.FIELD_P), b.get(q, fx.FIELD_PHI)]
    s.close()
    b.close()
    return cycles, out


def same(a, b):
    assert a[0] == b[0]
    for q, (x, y) in enumerate(zip(a[1], b[1])):
        assert np.array_equal(x, y), q


@pytest.mark.parametrize("prec", PRECS)
def test_prolongation_by_coarse_columns_equals_by_fine_cells(monkeypatch, prec):
    from paper_2210_15668_amd import ferrox as fx
    monkeypatch.setenv("FERROX_TB", "0")
    monkeypatch.setenv("FERROX_PROLONG_CC", "1")
    a = run(fx, prec)
    monkeypatch.setenv("FERROX_PROLONG_CC", "0")
    same(a, run(fx, prec))


@pytest.mark.parametrize("prec", PRECS)
def test_tuned_launches_equal_default_ones(monkeypatch, tmp_path, prec):
    from paper_2210_15668_amd import ferrox as fx
    monkeypatch.setenv("FERROX_TB", "0")
    same(run(fx, prec), run(fx, prec, tune=str(tmp_path / "tune.txt")))
