"""Model terms outside the range in which the kernels shorten the square root
and the division.

nDGP with a large crossover scale: alpha falls as 1 / h0rc, and alpha^2 leaves
that range at 1e15 (FP32) and 1e116 (FP64).  There beta_DGP is proportional to
h0rc, so that h0rc phi solves the same equation for every h0rc: the reference
is the FP64 field at h0rc = 1e9 (relative error of the proportionality 1e-9).
FP32 solves reach 1e-6 of their field on these meshes.
Meshes: 32^3 (kernels of the small levels), 128^3 (tiled kernels).

Kmouflage with a divisor that overflows where the field is steepest: one period
of a sine of gradient 4 with n_k = 8, whose divisor reaches 6e38 (above the
largest FP32 number) or 6e308 (above the largest FP64 number), with delta = 0.
The reference is the FP64 oracle's field after the same cycle, at 6e300 for
6e308: the term no longer depends on k0 there (the oracle's fields at 6e60, 6e300
and 6e305 agree to 4e-13; with more periods per box they do not, as coarse levels
then hold nothing but rounding errors).  A perturbation of the start by 1e-15
moves the oracle's field by up to 6e-12: FP64 1e-10.  FP32 second differences of a
field of 80 are good to 1.5e-5, the term to 4e-5, and the inverse Laplacian of
128 cells multiplies that by 415 against a field of 0.45: 5%.
"""
import math

import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2110_00566_amd as mg

pytestmark = pytest.mark.gpu


def test_fp32_kmouflage_with_a_small_density():
    # delta = 1e-30: the term is linear there, and every factor of the FP32 sums
    # stays a normal number; reference: the FP64 field
    d = delta_of(32) * 1e-30
    kw = dict(box_mpch=32.0, n_k=3, beta=0.2, tol=0.0, max_cycles=12)
    ref, _ = mg.solve_kmouflage(d, **kw)
    phi, _ = mg.solve_kmouflage(d, precision=mg.MG_FP32, **kw)
    assert float((phi - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


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


@pytest.mark.parametrize("n", [32, 128])
@pytest.mark.parametrize("ten,ten_ref,precision,tol", [(38, 38, mg.MG_FP32, 5e-2),
                                                       (38, 38, mg.MG_FP64, 1e-10),
                                                       (308, 300, mg.MG_FP64, 1e-10)])
def test_kmouflage_with_an_overflowing_divisor(n, ten, ten_ref, precision, tol):
    x = (np.arange(n) + 0.5) * (2.0 * math.pi / n)
    phi0 = np.broadcast_to(4.0 / math.sin(2.0 * math.pi / n) * np.sin(x), (n, n, n)).copy()

    def k0(e):   # c~ a1 g^7 = 6 10^e at g = 16, with c~ = 2997.92458, a1 = 17/3 8 k0
        return 6.0 * 10.0 ** (e - 20) / (2997.92458 * 16.0 ** 7) * 3.0 / 17.0 / 8.0 * 1e20

    lam = math.sqrt(0.5)
    ref = oracle.solve(oracle.kmo_model(n, float(n), 8, k0(ten_ref), 0.1, lam), np.zeros_like(phi0),
                       phi0=phi0, tol=0.0, max_cycles=1).phi
    p = torch.from_numpy(phi0).cuda()
    phi, st = mg.solve_kmouflage(torch.zeros_like(p), phi0=p, box_mpch=float(n), n_k=8, k0=k0(ten),
                                 beta=0.1, lam=lam, tol=0.0, max_cycles=1, precision=precision)
    assert st["status"] == mg.MG_NOT_CONVERGED   # tol = 0
    assert all(math.isfinite(e) for e in st["eps_hist"])
    assert np.abs(phi.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
