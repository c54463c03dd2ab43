"""The register budget that the library takes once there are more cells than
resident waves, against an explicit one: the same bits, counters included."""
import numpy as np
import pytest

from paper_2405_01713_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,R,thermal,opts", [
    (9, 30, True, dict()), (9, 30, True, dict(lu_precision=32, scheduler=1)),
    (21, 84, True, dict(lu_precision=32)), (21, 84, False, dict(scheduler=1)),
    (30, 120, False, dict()), (21, 84, False, dict(gmres_maxl=5, scheduler=1)),
    (21, 84, False, dict(jacobian=1)), (9, 30, False, dict(checkpoint_every=16, record_steps=512))])
@pytest.mark.parametrize("cells_per_simd", [2, 3, 4, 9])
def test_budget_by_cell_count(S, R, thermal, opts, cells_per_simd):
    """3 cells past 2, 3, 4 and 9 a SIMD: each side of the rule's steps (cells
    beside the waves two, three, four and five a SIMD hold)."""
    import torch
    from paper_2405_01713_amd import bdfx
    m = W.synthetic_mechanism(S, R, 1)
    n = 4 * cells_per_simd * torch.cuda.get_device_properties(0).multi_processor_count + 3
    c = W.cell_states(m, n, seed=5)
    y0, T, atol = c["y0"], c["T"], 1e-10
    if thermal:
        m, y0, T = W.thermal_mechanism(m), np.c_[y0[:, :S], T], None
        atol = np.array([1e-10] * S + [1e-6])
    out = []
    for wps in (0, 3):
        integ = bdfx.Integrator([m], y0, 1e-6, atol, T=T, waves_per_simd=wps, **opts)
        integ.integrate(0.0, 1e-8)
        torch.cuda.synchronize()
        out.append((integ.state(), integ.cell_stats()))
        integ.close()
    # (-10: a cell of more steps than its record holds)
    assert np.all(np.isin(out[0][1]["status"], (0, -10) if "record_steps" in opts else (0,)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("S,R,thermal,opts", [
    (9, 30, True, dict()), (16, 64, True, dict(lu_precision=32)), (20, 80, True, dict()),
    (21, 84, True, dict(lu_precision=32)), (30, 120, True, dict()), (9, 30, False, dict(jacobian=1)),
    (18, 60, False, dict(jacobian=1)), (21, 84, False, dict(jacobian=1, lu_precision=32)),
    (30, 120, False, dict(jacobian=1)), (30, 120, False, dict(gmres_maxl=5)), (30, 120, False, dict())])
def test_few_cells_kernel_against_the_budgets(S, R, thermal, opts):
    """Fewer cells than waves: the kernel with the compiler's registers (and, with
    the temperature, difference quotients or GMRES, its own lane addresses)
    against those of the three budgets."""
    import torch
    from paper_2405_01713_amd import bdfx
    m = W.synthetic_mechanism(S, R, 1)
    c = W.cell_states(m, 130, seed=6)
    y0, T, atol = c["y0"], c["T"], 1e-10
    y0[7, 0] = np.nan  # a failing cell among the others
    if thermal:
        m, y0, T = W.thermal_mechanism(m), np.c_[y0[:, :S], T], None
        atol = np.array([1e-10] * S + [1e-6])
    out = []
    for wps in (0, 3, 4, 5):
        integ = bdfx.Integrator([m], y0, 1e-6, atol, T=T, waves_per_simd=wps, **opts)
        integ.integrate(0.0, 1e-8)
        torch.cuda.synchronize()
        out.append((integ.state(), integ.cell_stats()))
        integ.close()
    assert np.sum(out[0][1]["status"] != 0) == 1
    for y, st in out[1:]:
        assert np.array_equal(out[0][0], y, equal_nan=True) and np.array_equal(out[0][1], st)
