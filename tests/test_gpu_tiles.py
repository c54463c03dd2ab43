"""The matrix-core elimination above 16 species, at the edges of its tiles and
blocks (padded rows and columns, a last block of one to four columns)."""
import numpy as np
import pytest

from paper_2405_01713_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lu", [64, 32])
@pytest.mark.parametrize("S", [17, 19, 20, 31, 32, 33, 47, 49, 52, 54, 64])
def test_tile_edges(oracle, parity, S, lu):
    import torch
    from paper_2405_01713_amd import bdfx
    m = W.synthetic_mechanism(S, 4 * S, S)
    c = W.cell_states(m, 48, seed=S + 5)
    w = dict(mechs=[m], y0=c["y0"], T=c["T"], rtol=1e-6, atol=1e-10, t_out=1e-7)
    integ = bdfx.Integrator([m], c["y0"], 1e-6, 1e-10, T=c["T"], lu_precision=lu)
    integ.integrate(0.0, 1e-7)
    torch.cuda.synchronize()
    y, st = integ.state(), integ.cell_stats()
    integ.close()
    assert np.all(st["status"] == 0)
    yo, _ = oracle.integrate([m], c["y0"], 0.0, 1e-7, 1e-6, 1e-10, T=c["T"])
    # adaptive control may put a cell onto another valid step sequence (see
    # conftest; it then has to match the tight reference): two whole cells of 48
    parity(y, yo, w, f"S={S} LU{lu}", min_frac=0.95)
