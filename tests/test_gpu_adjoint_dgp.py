"""GPU parity of the nDGP adjoint kernels of levels >= 128^3, which rebuild
the Jacobian coefficients from dK/dSigma and phi in every colour pass, residual
and coarse source.

Fixed cycles against the FP64 oracle adjoint.  At 128^3 both halo columns of a
tile wrap onto the tile itself and a z-chunk has 4 planes (every step of a
march is a guarded one); 256^3 has two x tiles and chunks of 32 planes.  Sweep
counts of 0, 2 and 3 chain passes without a residual between; phi is any field
(the adjoint is linear in mu for each) and mu0 a non-zero start.  Tolerance:
that of the other adjoint parity tests, 1e-10 relative.
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


@pytest.mark.parametrize("n,nu1,nu2", [(128, 1, 1), (128, 3, 2), (128, 0, 1), (256, 2, 0)])
def test_dgp_adjoint_from_a_field(n, nu1, nu2):
    delta = inputs.lognormal_delta(n, 2)
    phi = 2.0 * inputs.gaussian_field(n, 3, lambda k: k ** -3.0)
    w, mu0 = inputs.gaussian_weights(n, 5), 0.1 * inputs.gaussian_weights(n, 6)
    r = oracle.adjoint(oracle.dgp_model(0.8, OM, 2.0), delta, phi, w, mu0=mu0, tol=0.0,
                       max_cycles=1, nu1=nu1, nu2=nu2)
    grad, mu, st = mg.solve_adjoint(0, mg.dgp_params(0.8, OM, 2.0), g(delta), g(phi), g(w),
                                    mu0=g(mu0), tol=0.0, max_cycles=1, nu_pre=nu1, nu_post=nu2)
    assert np.isfinite(r.mu).all()
    for a, b in ((mu, r.mu), (grad, r.grad)):
        assert np.abs(a.cpu().numpy() - b).max() <= 1e-10 * np.abs(b).max()
    np.testing.assert_allclose(st["eps_hist"], r.hist[:1], rtol=1e-9)
