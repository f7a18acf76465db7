"""Bottom solves of more than one cell per thread of the coarse kernel.

Odd lateral factors end the x-y coarsening early, so the coarsest level can hold up to 64 KB of
vectors: 2048 cells in FP64, 4096 in FP32 (mixed precision).  The conjugate gradients there keep
one, two or four cells in a thread's registers.  These stacks take a bottom just above 1024 cells, the
largest ones of FP64, one just above 2048 and the largest ones of FP32, with and without a semiconductor,
plainly stored and (2 x 1100) in red/black order, and as a single row.  The trajectory must
meet the oracle's to the 1e-10 of tests/test_gpu_parity.py.
"""
import numpy as np
import pytest

from paper_2210_15668_amd import workloads as W

pytestmark = pytest.mark.gpu

FP64, MIXED = W.PREC_FP64, W.PREC_MIXED
# precision, lateral x, y, planes of ferroelectric, dielectric, semiconductor, bottom cells
CASES = [(FP64, 33, 32, 6, 3, 0, 1056), (FP64, 39, 39, 6, 3, 6, 1521), (FP64, 45, 45, 5, 3, 0, 2025),
         (MIXED, 43, 47, 6, 3, 5, 2021), (MIXED, 51, 41, 6, 3, 5, 2091), (MIXED, 98, 98, 10, 4, 12, 2401),
         (MIXED, 64, 45, 8, 4, 9, 2880), (MIXED, 126, 126, 9, 4, 0, 3969), (MIXED, 2, 1100, 6, 3, 4, 2200),
         (MIXED, 3001, 1, 8, 4, 7, 3001)]


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def stack(prec, nx, ny, fe, de, sc, v=0.7):
    layers = [(W.FE, fe, W.EPS_FE, 0.0), (W.DE, de, W.EPS_SIO2, 0.0)] + ([(W.SC, sc, W.EPS_SI, 1e24)] if sc else [])
    return W.layered(nx, ny, fe + de + sc + 2, layers, v_top=v, tol_rel=1e-13, prec=prec, max_cycles=400)


def bottom_cells(fx, s):
    import ctypes as C
    n = [C.c_int() for _ in range(3)]
    assert fx.lib().stack_level_shape(s._h, fx.lib().stack_num_levels(s._h) - 1, *map(C.byref, n)) == 0
    return n[0].value * n[1].value * n[2].value


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%dx%d" % ("fp64" if c[0] == FP64 else "mixed", c[1], c[2]))
def test_large_bottom_meets_the_oracle(orc, case):
    from paper_2210_15668_amd import ferrox as fx
    spec = stack(*case[:6])
    P0 = W.random_P(spec, 81, amp=0.05)
    s = fx.Stack(spec, P0)
    assert bottom_cells(fx, s) == case[6]
    info = s.run_steps(3, W.DT)
    P, phi = s.get(fx.FIELD_P), s.get(fx.FIELD_PHI)
    s.close()
    P_o, phi_o, _ = orc.run(spec, P0, 3, W.DT, tol=1e-13)
    print(f"  {case}: {info.total_cycles} cycles, P {rel(P, P_o):.1e} phi {rel(phi, phi_o):.1e}", flush=True)
    assert rel(P, P_o) <= 1e-10 and rel(phi, phi_o) <= 1e-10


def test_large_bottom_in_a_batch_and_without_a_handle(orc):
    import torch
    from paper_2210_15668_amd import ferrox as fx
    specs = [stack(MIXED, 24, 20, 8, 4, 6), stack(MIXED, 98, 94, 7, 3, 6, v=-0.5), stack(MIXED, 54, 43, 6, 4, 0)]
    P0 = [W.random_P(sp, 82 + q, amp=0.05) for q, sp in enumerate(specs)]
    b = fx.Batch(specs, P0)
    b.run(3, W.DT)
    for q, sp in enumerate(specs):
        P_o, phi_o, _ = orc.run(sp, P0[q], 3, W.DT, tol=1e-13)
        assert rel(b.get(q, fx.FIELD_P), P_o) <= 1e-10 and rel(b.get(q, fx.FIELD_PHI), phi_o) <= 1e-10, q
    b.close()
    for q in (1, 2):
        phi = torch.zeros(P0[q].shape, dtype=torch.float64, device="cuda:0")
        fx.poisson_solve_static(specs[q], torch.from_numpy(P0[q]).cuda(), phi)
        phi_o, _ = orc.solve(specs[q], P0[q], tol=1e-13)
        assert rel(phi.cpu().numpy(), phi_o) <= 1e-10, q
