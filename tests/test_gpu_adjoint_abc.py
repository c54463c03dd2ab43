"""The adjoint sweep's A + B <=> C kernels against the general ones: the same
bits.  A mechanism of such reactions with one A <=> C reaction added, whose rate
(exp(-700) times a mass fraction) is below the last bit of every sum it enters,
runs the general kernels and has the same solution and gradient."""
import numpy as np
import pytest

from paper_2405_01713_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,R,every", [(9, 63, 0), (21, 84, 0), (21, 127, 16), (30, 40, 0), (53, 128, 0)])
def test_abc_sweep_matches_the_general_one(S, R, every):
    import torch
    from paper_2405_01713_amd import bdfx
    m = W.synthetic_mechanism(S, R, 3)
    g = dict(m, n_reactions=R + 1)
    for k in ("reac", "prod"):
        g[k] = np.concatenate([m[k], np.full_like(m[k][:1], -1)])
        g[k][R, 0] = m[k][0, 0]
    for k in ("lnA", "EaR", "lnK"):
        g[k] = np.concatenate([m[k], [0.0]])
    g["lnA"][R] = -700.0
    c = W.cell_states(m, 37, seed=2)
    ybar = np.random.default_rng(4).standard_normal(c["y0"].shape)
    out = []
    for mech in (m, g):
        integ = bdfx.Integrator([mech], c["y0"], 1e-6, 1e-10, T=c["T"], record_steps=2048,
                                checkpoint_every=every)
        integ.integrate(0.0, 1e-7)
        y0_bar, lnA_bar = integ.adjoint(ybar)
        torch.cuda.synchronize()
        assert np.all(integ.cell_stats()["status"] == 0)
        out.append((integ.state(), y0_bar.cpu().numpy(), lnA_bar.cpu().numpy()[0, :R]))
        integ.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
