"""Model terms outside the range in which the kernels shorten the square root
and the division.

nDGP with a large crossover scale: alpha falls as 1 / h0rc, and alpha^2 leaves
that range at 1e15 (FP32) and 1e116 (FP64).  There beta_DGP is proportional to
h0rc, so that h0rc phi solves the same equation for every h0rc: the reference
is the FP64 field at h0rc = 1e9 (relative error of the proportionality 1e-9).
FP32 solves reach 1e-6 of their field on these meshes.
Meshes: 32^3 (kernels of the small levels), 128^3 (tiled kernels).
"""
import pytest
import torch

import inputs
import paper_2110_00566_amd as mg

pytestmark = pytest.mark.gpu


def delta_of(n):
    return torch.from_numpy(inputs.lognormal_delta(n, 11)).to("cuda")


@pytest.mark.parametrize("n", [32, 128])
@pytest.mark.parametrize("h0rc,precision,tol", [(1e13, mg.MG_FP32, 1e-5), (1e15, mg.MG_FP32, 1e-5),
                                                (1e19, mg.MG_FP32, 1e-5), (1e17, mg.MG_FP64, 1e-8),
                                                (1e130, mg.MG_FP64, 1e-8),
                                                (1e145, mg.MG_FP64, 1e-8)])
def test_dgp_with_a_large_crossover_scale(n, h0rc, precision, tol):
    d = delta_of(n)
    ref = mg.solve_dgp(d, h0rc=1e9, tol=0.0, max_cycles=16)[0] * 1e9
    phi, st = mg.solve_dgp(d, h0rc=h0rc, tol=0.0, max_cycles=16, precision=precision)
    assert st["status"] == mg.MG_NOT_CONVERGED and st["n_clamped"] == 0   # tol = 0
    assert float((phi * h0rc - ref).abs().max()) <= tol * float(ref.abs().max())
