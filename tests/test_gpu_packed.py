"""Several cells per wave (the library's own launch shape for many cells of a
small mechanism) against one cell per wave: the same bits, counters included."""
import numpy as np
import pytest

from paper_2405_01713_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(w, y0, **opts):
    import torch
    from paper_2405_01713_amd import bdfx
    integ = bdfx.Integrator(w["mechs"], y0, 1e-6, 1e-10, T=w.get("T"), kscale=w.get("kscale"),
                            forcing=w.get("F"), **opts)
    integ.integrate(0.0, w["t_out"])
    torch.cuda.synchronize()
    y, st = integ.state(), integ.cell_stats()
    rec = integ.step_record([0, 1, 5]) if opts.get("record_steps") else None
    integ.close()
    return y, st, rec


def _cells(S, extra):
    """Cells that the library packs (40 a CU up to 4 species, 32 up to 16, 64
    above), and ``extra`` more so that the last wave is partly filled."""
    import torch
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    return (40 if S <= 4 else 32 if S <= 16 else 64) * cu + extra


@pytest.mark.parametrize("S,R,lu,sched", [(2, 3, 64, 1), (9, 30, 64, 0), (9, 30, 32, 1),
                                          (12, 70, 64, 1), (16, 64, 64, 1), (16, 65, 32, 1),
                                          (17, 30, 64, 1), (21, 84, 64, 0), (21, 130, 32, 1)])
def test_packed_matches_one_cell_per_wave(oracle, parity, S, R, lu, sched):
    m = W.synthetic_mechanism(S, R, 1)
    n = _cells(S, 3)
    c = W.cell_states(m, n, seed=11)
    y0 = c["y0"]
    y0[7, 0] = np.nan  # a failing cell among the others
    w = dict(mechs=[m], T=c["T"], t_out=1e-8, y0=y0, rtol=1e-6, atol=1e-10)
    y, st, _ = _run(w, y0, lu_precision=lu, scheduler=sched)
    y1, st1, _ = _run(w, y0, lu_precision=lu, scheduler=sched, waves_per_simd=3)
    assert st["status"][7] == -9 and np.all(np.delete(st["status"], 7) == 0)
    assert np.array_equal(st, st1) and np.array_equal(y, y1, equal_nan=True)
    k = np.r_[0:6, n - 30:n]
    yo, _ = oracle.integrate([m], y0[k], 0.0, 1e-8, 1e-6, 1e-10, T=c["T"][k])
    # (one whole cell of 36 may follow another valid step sequence, see conftest)
    parity(y[k], yo, dict(w, y0=y0[k], T=c["T"][k]), f"S={S}", min_frac=0.95)


def test_packed_generic_slots_forcing_scale_and_records(oracle):
    """Robertson cells (empty and repeated slots) with rate scales and a forcing,
    few allowed steps, and recorded steps."""
    n = _cells(3, 1)
    c = W.robertson_cells(n)
    F = np.zeros((n, 3))
    F[::3, 0] = 1e-3
    w = dict(mechs=[W.robertson_mechanism()], kscale=c["kscale"], F=F, t_out=40.0)
    for opts in (dict(), dict(max_steps=60), dict(record_steps=400)):
        y, st, rec = _run(w, c["y0"], **opts)
        y1, st1, rec1 = _run(w, c["y0"], waves_per_simd=3, **opts)
        assert np.array_equal(st, st1) and np.array_equal(y, y1)
        # 60 steps are too few for every cell, 400 recorded ones for some
        assert set(np.unique(st["status"])) <= ({-1} if "max_steps" in opts else
                                                {0, -10} if "record_steps" in opts else {0})
        for a, b in zip(rec or [], rec1 or []):
            assert all(np.array_equal(a[key], b[key]) for key in a)


@pytest.mark.parametrize("chunk", [64, 2 ** 31 - 1])
def test_static_packed_launch_ignores_the_chunk(chunk):
    """queue_chunk is the work-queue schedulers' option: a packed launch of the
    static one, which takes its cells from the counter too, pops single cells."""
    n = _cells(3, 1)
    c = W.robertson_cells(n)
    w = dict(mechs=[W.robertson_mechanism()], kscale=c["kscale"], t_out=1.0)
    y, st, _ = _run(w, c["y0"])
    y1, st1, _ = _run(w, c["y0"], queue_chunk=chunk)
    assert np.all(st["status"] == 0)
    assert np.array_equal(st, st1) and np.array_equal(y, y1)


def test_largest_chunk_hands_out_every_cell_once():
    """A chunk for which the 32-bit counter would wrap (64 waves that each pop
    2^31 - 1 cells) is bounded by the library."""
    c = W.robertson_cells(64)
    w = dict(mechs=[W.robertson_mechanism()], kscale=c["kscale"], t_out=1.0)
    y, st, _ = _run(w, c["y0"], scheduler=1)
    y1, st1, _ = _run(w, c["y0"], scheduler=1, queue_chunk=2 ** 31 - 1)
    assert np.array_equal(st, st1) and np.array_equal(y, y1)


def test_static_packed_launch_ignores_blocks_per_cu():
    """blocks_per_cu is the persistent schedulers' option; under the static one
    the cells keep all of the GPU (one block a CU would hold a tenth of them:
    several times the time)."""
    import time

    import torch
    from paper_2405_01713_amd import bdfx
    n = _cells(3, 1)
    c = W.robertson_cells(n)
    best = []
    for opts in (dict(), dict(blocks_per_cu=1)):
        integ = bdfx.Integrator([W.robertson_mechanism()], c["y0"], 1e-6, 1e-10, kscale=c["kscale"], **opts)
        ms = []
        for _ in range(4):
            integ.set_state(c["y0"])
            torch.cuda.synchronize()
            t = time.perf_counter()
            integ.integrate(0.0, 40.0)
            torch.cuda.synchronize()
            ms.append(time.perf_counter() - t)
        best.append(min(ms))
        integ.close()
    assert best[1] < 2.0 * best[0], best


@pytest.mark.parametrize("S,R,lu,sched,per_cu", [(9, 64, 64, 1, 48), (12, 70, 64, 1, 128), (14, 48, 32, 0, 32),
                                                 (16, 64, 64, 1, 48), (16, 65, 32, 1, 48),
                                                 (17, 30, 32, 1, 96), (21, 84, 32, 0, 96),
                                                 (21, 110, 32, 1, 96)])
def test_packed_from_the_cells_that_the_reactions_ask_for(S, R, lu, sched, per_cu):
    """As above at the counts from which mechanisms of more reactions are packed."""
    import torch
    m = W.synthetic_mechanism(S, R, 1)
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + 3
    c = W.cell_states(m, n, seed=11)
    y0 = c["y0"]
    y0[7, 0] = np.nan  # a failing cell among the others
    w = dict(mechs=[m], T=c["T"], t_out=1e-8)
    y, st, _ = _run(w, y0, lu_precision=lu, scheduler=sched)
    y1, st1, _ = _run(w, y0, lu_precision=lu, scheduler=sched, waves_per_simd=3)
    assert st["status"][7] == -9 and np.all(np.delete(st["status"], 7) == 0)
    assert np.array_equal(st, st1) and np.array_equal(y, y1, equal_nan=True)
