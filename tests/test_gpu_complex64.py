"""GPU parity of the complex64 COCG path in whole energies and gradients: forced at every frequency
on grids that would take the real-form FP64 solves (mixed_min_omega = 0), and by default on planes
that these have no shape for.  More than one refinement per system shows that complex64 ran: the
real form counts one residual check per system."""
import numpy as np
import pytest
import torch

from oracle import energy as oenergy
from oracle import gradient as ograd
from paper_2504_01816_amd import api
from paper_2504_01816_amd import lib as L
from tests.test_gpu_real_form import make, rel

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OM, W = np.array([2.0, 0.3]), np.array([0.6, 0.9])
# at every frequency by request, or because the plane has no real-form shape
CASES = [((12, 13, 14), "periodic", 0.0), ((13, 12, 15), "dirichlet", 0.0), ((50, 48, 12), "periodic", 0.2)]


@pytest.fixture(scope="module", params=CASES, ids=lambda p: "%dx%dx%d-%s-%g" % (p[0] + p[1:]))
def case(request):
    shape, bc, min_omega = request.param
    print("complex64", shape, bc, min_omega, flush=True)
    c = make(shape, 3, 31, bc)
    V0 = np.random.default_rng(32).standard_normal((4, c.nd))
    return c, V0, dict(cocg_tol=1e-11, subspace_iters=2, ec_tol=0.0, precision=L.RPA_MIXED,
                       mixed_min_omega=min_omega)


@pytest.mark.parametrize("mode", [L.RPA_WARM, L.RPA_INDEPENDENT])
def test_complex64_energy_matches_oracle(case, mode):
    c, V0, opts = case
    r = api.rpa_energy(api.device_cell(c, DEV), 4, OM, W, [torch.tensor(V0, device=DEV)],
                       dict(opts, freq_mode=mode), save=True)
    st = r["stats"]
    assert r["status"] == 0 and st["refinements"] > 2 * st["cocg_systems"]
    ref = oenergy.rpa_energy(c.vloc, c.psi.T, c.eps, c.shape, c.h, V0.T, OM, W, 1e-11, 5000, 2,
                             mode="warm" if mode == L.RPA_WARM else "independent", bc=c.bc)
    for C, Cref in zip(r["Csave"][0].cpu().numpy(), ref["C_saved"]):
        # solutions that meet 1e-11 differ by cond(A) 1e-11, about 1e-9 here, and the second step's
        # block by that times the condition of R^T R, below 100 for four vectors
        assert rel(C, Cref) < 1e-7


def test_complex64_gradient_matches_oracle(case):
    c, V0, opts = case
    V = np.ascontiguousarray([np.linalg.qr(V0.T)[0].T] * 2)
    Q = np.linalg.qr(np.random.default_rng(33).standard_normal((4, 4)))[0]
    C = (Q * -np.linspace(0.05, 0.4, 4)) @ Q.T
    C = np.stack([0.5 * (C + C.T)] * 2)
    g, rc, st = api.rpa_energy_backward(api.device_cell(c, DEV), OM, W, torch.tensor(V, device=DEV),
                                        torch.tensor(C, device=DEV), 1.0, opts)
    assert rc == 0 and st["refinements"] > 2 * st["cocg_systems"]
    ref = ograd.energy_backward(c.vloc, c.psi.T, c.eps, c.shape, c.h, OM, W, [v.T for v in V], list(C),
                                1e-11, 5000, bc=c.bc)
    # solutions that meet 1e-11 differ by cond(A) 1e-11, about 1e-9 here
    assert rel(g.cpu().numpy(), ref) < 1e-8
