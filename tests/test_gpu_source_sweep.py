"""GPU parity of the residual + restriction kernel of levels >= 128^3 and of
the sweep that forms a coarse level's FAS source (FP64, levels >= 128^3 below
the finest), against the FP64 oracle.

256^3 has one such coarse level (128^3: one x tile, z-chunks of 4 planes).  In
F and W cycles the level is visited twice and the second visit reads the
stored source; nu_pre = 0 keeps the source in a launch of its own; nu_pre = 2
follows it with an ordinary sweep.  Iterates agree to 1e-11 relative, as in the
other fixed-cycle tests (the two sides evaluate the same FP64 expressions in
different algebraic forms).
"""
import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2110_00566_amd as mg

pytestmark = pytest.mark.gpu
OM = 0.3089


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("name,nu1,nu2,cycle", [("dgp", 1, 1, mg.CYCLE_W), ("dgp", 0, 1, mg.CYCLE_V),
                                                ("dgp", 2, 1, mg.CYCLE_V),
                                                ("poisson", 1, 0, mg.CYCLE_F),
                                                ("kmo2", 1, 1, mg.CYCLE_F)])
def test_source_with_sweep(name, nu1, nu2, cycle):
    n = 256
    delta = inputs.lognormal_delta(n, 3)
    phi0 = 3.0 * inputs.gaussian_field(n, 8, lambda k: k ** -3.0)
    if name == "dgp":
        om, solve, kw = oracle.dgp_model(1.0, OM, 1.0), mg.solve_dgp, dict(a=1.0, h0rc=1.0)
    elif name == "poisson":
        om, solve, kw = oracle.linear_model(0.7), mg.solve_poisson, dict(s=0.7)
    else:
        om = oracle.kmo_model(n, 0.05 * n, 2, 5.0, 0.2)
        solve, kw = mg.solve_kmouflage, dict(box_mpch=0.05 * n, n_k=2, k0=5.0, beta=0.2)
    r = oracle.solve(om, delta, phi0=phi0, tol=0.0, max_cycles=2, nu1=nu1, nu2=nu2, cycle=cycle)
    phi, st = solve(g(delta), phi0=g(phi0), tol=0.0, max_cycles=2, nu_pre=nu1, nu_post=nu2,
                    cycle=cycle, **kw)
    assert np.isfinite(r.phi).all()
    assert np.abs(phi.cpu().numpy() - r.phi).max() <= 1e-11 * np.abs(r.phi).max()
    np.testing.assert_allclose(st["eps_hist"], r.hist[:2], rtol=1e-8)
