"""GPU parity of the fused kernels of the levels below 128^3 (sweep + residual +
restriction, prolongation + sweep) and of the single-workgroup tail.

Fixed-cycle solves against the FP64 oracle from a non-zero field.  8^3 is one
block, whose halo wraps onto itself, over a tail of 4^3 alone; 16^3 adds the
8^3 tail level; 32^3 and 64^3 have one and two fused levels over the whole
tail, and the first reduction pending in the tail or in a coarse source.
Sweep counts 0, 2 and 3 mix the fused and the separate kernels.  Both sides
evaluate the same FP64 expressions in different algebraic forms: iterates
agree to 1e-11 relative, as in the other fixed-cycle tests.
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


@pytest.mark.parametrize("n", [8, 16, 32, 64])
@pytest.mark.parametrize("nu1,nu2,cycle", [(1, 1, mg.CYCLE_V), (2, 3, mg.CYCLE_V),
                                           (0, 1, mg.CYCLE_W), (3, 0, mg.CYCLE_V),
                                           (1, 2, mg.CYCLE_F)])
@pytest.mark.parametrize("name", ["dgp", "kmo2", "newton"])
def test_fixed_cycles_from_a_field(n, nu1, nu2, cycle, name):
    delta = inputs.lognormal_delta(n, 4)
    if name == "newton":
        delta *= 0.02
    phi0 = (0.05 if name == "newton" else 2.0) * inputs.gaussian_field(n, 9, lambda k: k ** -3.0)
    if name == "dgp":
        om, solve, kw = oracle.dgp_model(0.8, OM, 2.0), mg.solve_dgp, dict(a=0.8, h0rc=2.0)
    elif name == "newton":
        om, solve, kw = oracle.dgp_newton_model(0.8, OM, 1.0), mg.solve_dgp_newton, dict(a=0.8)
    else:
        om = oracle.kmo_model(n, 0.05 * n, 2, 5.0, 0.2)
        solve, kw = mg.solve_kmouflage, dict(box_mpch=0.05 * n, n_k=2, k0=5.0, beta=0.2)
    r = oracle.solve(om, delta, phi0=phi0, tol=0.0, max_cycles=2, nu1=nu1, nu2=nu2, cycle=cycle)
    phi, st = solve(g(delta), phi0=g(phi0), tol=0.0, max_cycles=2, nu_pre=nu1, nu_post=nu2,
                    cycle=cycle, **kw)
    assert np.isfinite(r.phi).all()
    assert np.abs(phi.cpu().numpy() - r.phi).max() <= 1e-11 * np.abs(r.phi).max()
    assert np.allclose(st["eps_hist"], r.hist[:2], rtol=1e-8)
