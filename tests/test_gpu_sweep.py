"""GPU parity of the red-black sweep kernel (both colours in one launch, with
and without the prolongation), on levels >= 128^3.

Fixed-cycle solves against the FP64 oracle.  128^3 has one 64-column tile in
x (both halo columns wrap onto the tile itself) and z-chunks of 4 planes, so
every step of a march is a guarded one; 256^3 has two x tiles and chunks of
32 planes.  Sweep counts of 2 and 3 chain sweeps without a residual between;
a non-zero start gives the cross terms a field to act on.  As in the other
fixed-cycle tests the two sides evaluate the same FP64 expressions in
different algebraic forms: iterates agree to 1e-11 relative.
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


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.mark.parametrize("name,n,nu1,nu2,cycle", [("dgp", 128, 3, 2, mg.CYCLE_V),
                                                  ("dgp", 256, 2, 1, mg.CYCLE_F),
                                                  ("kmo2", 128, 2, 3, mg.CYCLE_W),
                                                  ("kmo3", 256, 1, 2, mg.CYCLE_V),
                                                  ("poisson", 128, 0, 1, mg.CYCLE_V)])
def test_sweeps_from_a_field(name, n, nu1, nu2, cycle):
    delta = inputs.lognormal_delta(n, 4)
    phi0 = 5.0 * inputs.gaussian_field(n, 9, lambda k: k ** -3.0)
    if name == "dgp":
        om = oracle.dgp_model(0.8, OM, 2.0)
        solve, kw = mg.solve_dgp, dict(a=0.8, h0rc=2.0)
    elif name == "poisson":
        om = oracle.linear_model(0.7)
        solve, kw = mg.solve_poisson, dict(s=0.7)
    else:
        k = 2 if name == "kmo2" else 3
        om = oracle.kmo_model(n, 0.05 * n, k, 5.0, 0.2)
        solve, kw = mg.solve_kmouflage, dict(box_mpch=0.05 * n, n_k=k, k0=5.0, beta=0.2)
    r = oracle.solve(om, delta, phi0=phi0, tol=0.0, max_cycles=1, nu1=nu1, nu2=nu2, cycle=cycle)
    phi, st = solve(g(delta), phi0=g(phi0), tol=0.0, max_cycles=1, nu_pre=nu1, nu_post=nu2,
                    cycle=cycle, **kw)
    assert np.isfinite(r.phi).all()
    assert rel(phi.cpu().numpy(), r.phi) <= 1e-11
    assert st["eps_hist"][0] == pytest.approx(r.hist[0], rel=1e-8)


@pytest.mark.parametrize("n", [128, 256])
def test_profile_counts_two_passes_per_sweep(n):
    d = g(inputs.lognormal_delta(n, 1))
    _, st = mg.solve_dgp(d, tol=0.0, max_cycles=2, nu_pre=2, nu_post=2, profile=True)
    # two pre-sweeps and the second post-sweep of each cycle are timed (the
    # first post-sweep includes the prolongation)
    assert st["pass_count"] == 2 * 2 * 3
    assert st["pass_ms_avg"] > 0.0
