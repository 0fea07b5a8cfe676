"""GPU parity of the Newton-Gauss-Seidel comparator on coarse levels >= 128^3.

At 256^3 the level of 128^3 runs the sweep that forms the level's FAS source,
the ordinary sweep, the sweep with the prolongation and the residual with a
right-hand side.  The Newton source differs from the closed-form one: it takes
the centre value and the face sums of the field before the sweep.  Cycles
of type F and W read a source again; nu_pre = 2 follows the source sweep with
an ordinary one, nu_pre = 0 keeps the source in a launch of its own.  Iterates
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


@pytest.mark.parametrize("nu1,nu2,cycle", [(1, 1, mg.CYCLE_F), (2, 2, mg.CYCLE_V),
                                           (1, 1, mg.CYCLE_W), (0, 1, mg.CYCLE_V)])
def test_newton_fixed_cycles_256(nu1, nu2, cycle):
    n = 256
    delta = 0.02 * inputs.lognormal_delta(n, 4)
    phi0 = 0.05 * inputs.gaussian_field(n, 9, lambda k: k ** -3.0)
    r = oracle.solve(oracle.dgp_newton_model(0.8, OM, 1.0), delta, phi0=phi0, tol=0.0,
                     max_cycles=2, nu1=nu1, nu2=nu2, cycle=cycle)
    phi, st = mg.solve_dgp_newton(g(delta), phi0=g(phi0), a=0.8, tol=0.0, max_cycles=2,
                                  nu_pre=nu1, nu_post=nu2, cycle=cycle)
    assert np.isfinite(r.phi).all()
    assert np.abs(phi.cpu().numpy() - r.phi).max() <= 1e-11 * np.abs(r.phi).max()
    np.testing.assert_allclose(st["eps_hist"], r.hist[:2], rtol=1e-8)
