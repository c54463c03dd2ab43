"""The autotuner's choice of kernel: by the cells of the bin, not of the sample,
and each kernel once."""
import json

import numpy as np
import pytest

from paper_2405_01713_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _integ(S, R, n, **opts):
    from paper_2405_01713_amd import bdfx
    m = W.synthetic_mechanism(S, R, 1)
    c = W.cell_states(m, n, seed=2)
    return bdfx.Integrator([m], c["y0"], 1e-6, 1e-10, T=c["T"], scheduler=1, **opts), c["y0"]


@pytest.mark.parametrize("S,R,per_cu", [(9, 30, 64), (16, 100, 128), (21, 84, 96)])
def test_small_sample_keeps_the_library_s_kernel(S, R, per_cu):
    """A sample of 4 cells a CU cannot tell whether several cells per wave, or
    more waves, are faster for the bin: the library's own kernel stays (its
    budget is 0), and the states and results are untouched."""
    import torch
    lu = 32 if S > 16 else 64
    integ, y0 = _integ(S, R, per_cu * _cu() + 1, lu_precision=lu)
    res = integ.autotune(0.0, 1e-8, sample_cells=4 * _cu())
    assert res[0]["waves_per_simd"] == 0 and res[0]["cells_per_wave"] == 1
    assert res[0]["waves_per_block"] in (1, 2, 4) and res[0]["ms"] > 0
    assert np.array_equal(integ.state(), y0)
    integ.integrate(0.0, 1e-8)
    torch.cuda.synchronize()
    y, st = integ.state(), integ.cell_stats()
    integ.close()
    ref, _ = _integ(S, R, per_cu * _cu() + 1, lu_precision=lu, waves_per_simd=3)
    ref.integrate(0.0, 1e-8)
    torch.cuda.synchronize()
    assert np.array_equal(ref.state(), y) and np.array_equal(ref.cell_stats(), st)
    ref.close()


@pytest.mark.parametrize("lu", [64, 32])
def test_one_kernel_above_32_species_is_one_budget(lu):
    """Above 32 species all budgets are one kernel: the pick is never left to
    the noise between equals (and the one-launch pair, which has no code for
    budget 5, stays available)."""
    for S, R in ((33, 100), (53, 325), (64, 130)):
        integ, _ = _integ(S, R, 512, lu_precision=lu)
        res = integ.autotune(0.0, 1e-8)
        integ.close()
        assert res[0]["waves_per_simd"] == 0


def test_cached_shape_of_a_small_batch_is_not_a_large_one_s(tmp_path):
    cache = str(tmp_path / "t.json")
    for k, n in enumerate((64, 6 * _cu(), 16 * _cu(), 64 * _cu(), 200 * _cu())):
        integ, _ = _integ(9, 30, n)
        integ.autotune(0.0, 1e-8, sample_cells=256, cache=cache)
        integ.close()
        with open(cache) as fh:
            assert len(json.load(fh)) == max(k, 1)  # (the first two are of one size)
