"""GPU checks of the small dense kernels at the edges of their panels and memory classes: Ritz
values (tridiagonal form and bisection, in LDS up to 120 columns, a launch per column beyond), the
log-det energy and the Cholesky orthonormalisation (panels of 16, LDS up to 120), the Jacobi
vectors of the backward (LDS up to 88), and the parity-split bases of an isolated box (axes up to
175 points in LDS)."""
import numpy as np
import pytest
import torch

from oracle import coulomb as ocoul
from oracle import gradient as ograd
from paper_2504_01816_amd import api, synth
from paper_2504_01816_amd import lib as L
from tests.test_gpu_real_form import make

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nr", [1, 2, 15, 16, 17, 63, 64, 65, 119, 120, 121, 150])
def test_subspace_algebra(nr):
    # C is the kernels' own; its eigenvalues, energy and the new block are recomputed on the host
    c = make((10, 9, 12), 2, 11)
    V = np.linalg.qr(np.random.default_rng(nr).standard_normal((c.nd, nr)))[0].T.copy()
    Vt = torch.tensor(V, device=DEV)
    r = api.rpa_subspace_iter(api.device_cell(c, DEV), 0.8, 1.3, Vt,
                              dict(cocg_tol=1e-12, subspace_iters=1, ec_tol=0.0))
    C = r["C"].cpu().numpy()
    mu = np.linalg.eigvalsh(0.5 * (C + C.T))
    # bisection and the tridiagonal form are backward stable: a few m eps of the norm
    assert np.abs(r["ritz"] - mu).max() <= 8 * nr * 2.3e-16 * np.abs(mu).max()
    # the factor of I - C (entries of order one) is backward stable: ln det moves by at most a few
    # eps per column, whatever the size of the eigenvalues
    L = np.linalg.cholesky(np.eye(nr) - 0.5 * (C + C.T))
    E = 1.3 / (2 * np.pi) * (2 * np.log(np.diag(L)).sum() + np.trace(C))
    assert abs(r["E"] - E) <= 1.3 / (2 * np.pi) * 16 * nr * 2.3e-16
    Vn = Vt.cpu().numpy()
    assert np.abs(Vn @ Vn.T - np.eye(nr)).max() < 1e-10


@pytest.mark.parametrize("nr", [3, 88, 89])
def test_backward_with_jacobi_vectors(nr):
    c = make((8, 7, 12), 2, 12)
    rng = np.random.default_rng(nr)
    V = np.linalg.qr(rng.standard_normal((c.nd, nr)))[0].T.copy()
    Q = np.linalg.qr(rng.standard_normal((nr, nr)))[0]
    C = (Q * -rng.uniform(0.01, 0.4, nr)) @ Q.T
    C = 0.5 * (C + C.T)
    g, rc, _ = api.rpa_energy_backward(api.device_cell(c, DEV), [0.9], [1.1],
                                       torch.tensor(V[None], device=DEV),
                                       torch.tensor(C[None], device=DEV), 1.0,
                                       dict(cocg_tol=1e-12))
    ref = ograd.energy_backward(c.vloc, c.psi.T, c.eps, c.shape, c.h, [0.9], [1.1], [V.T], [C],
                                1e-12, 5000)
    assert rc == 0
    assert np.abs(g.cpu().numpy() - ref).max() < 1e-8 * np.abs(ref).max()


@pytest.mark.parametrize("shape", [(7, 8, 12), (11, 20, 33), (7, 9, 175), (7, 8, 177)])
def test_box_bases(shape):
    c = synth.uniform_cell(shape, 0.45)
    c.bc = "dirichlet"
    X = np.random.default_rng(1).standard_normal((2, c.nd))
    for power in (1, 2):
        out = api.rpa_apply_coulomb(api.device_cell(c, DEV), torch.tensor(X, device=DEV), power)
        ref = ocoul.nu_apply(X.T, shape, 0.45, power, bc="dirichlet").T
        assert np.abs(out.cpu().numpy() - ref).max() < 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nfreq,nr", [(1, 5), (32, 5), (33, 5), (3, 121)])
def test_batched_frequencies_share_the_dense_launches(nfreq, nr):
    # every frequency's energy as in a run of its own: lists of 32 matrices, and beyond 120 columns
    # one work matrix for all
    c = make((8, 7, 12), 2, 17)
    V0 = np.random.default_rng(18).standard_normal((nr, c.nd))
    om, wt = np.linspace(0.5, 6.0, nfreq), np.linspace(1.0, 2.0, nfreq)
    opts = dict(cocg_tol=1e-12, subspace_iters=2, ec_tol=0.0, freq_mode=L.RPA_INDEPENDENT)
    dc, V = api.device_cell(c, DEV), torch.tensor(V0, device=DEV)
    E = api.rpa_energy(dc, nr, om, wt, [V], opts)["E_freq"][0].tolist()
    for f in {0, nfreq // 2, nfreq - 1}:
        one = api.rpa_energy(dc, nr, om[f:f + 1], wt[f:f + 1], [V], opts)["E_freq"][0].tolist()
        # the solves meet 1e-12; the energy moves by cond(A) times that at most
        assert abs(E[f] - one[0]) <= 1e-9 * abs(one[0]), (f, E[f], one[0])
