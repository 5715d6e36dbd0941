"""Workspaces smaller than the size query's answer: the least state of a call (r, p, p', x of every
system and the call's own blocks, as the library asked for it before it kept longer rings of basis
vectors for small launches) is accepted, and a call in it gives the same results to rounding."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import fd
from oracle.chi0 import build_rhs
from paper_2504_01816_amd import api
from paper_2504_01816_amd import lib as L
from tests.test_gpu_real_form import make, rel

# (operation, grid, N_s, vectors, options) -> bytes of the least state
LEAST = [
    (L.RPA_OP_CHI0, (27, 27, 25), 2, 2, dict(cocg_tol=1e-11), 4086032),
    (L.RPA_OP_CHI0, (27, 27, 25), 2, 2, dict(cocg_tol=1e-11, precision=1), 4742928),
    (L.RPA_OP_CHI0, (24, 24, 24), 2, 3, dict(cocg_tol=1e-11), 4647704),
    (L.RPA_OP_CHI0, (24, 24, 24), 2, 3, dict(cocg_tol=1e-11, precision=1), 5366808),
    (L.RPA_OP_CHI0, (12, 13, 14), 3, 4, dict(cocg_tol=1e-11), 1470256),
    (L.RPA_OP_CHI0, (12, 13, 14), 3, 4, dict(cocg_tol=1e-11, precision=1), 1689136),
    (L.RPA_OP_CHI0, (13, 11, 13), 1, 1, dict(cocg_tol=1e-11), 106756),
    (L.RPA_OP_CHI0, (13, 11, 13), 1, 1, dict(cocg_tol=1e-11, precision=1), 130052),
    (L.RPA_OP_CHI0, (35, 37, 13), 1, 1, dict(cocg_tol=1e-11), 945412),
    (L.RPA_OP_CHI0, (35, 37, 13), 1, 1, dict(cocg_tol=1e-11, precision=1), 1148420),
    (L.RPA_OP_CHI0, (46, 47, 12), 2, 1, dict(cocg_tol=1e-11), 2908424),
    (L.RPA_OP_CHI0, (46, 47, 12), 2, 1, dict(cocg_tol=1e-11, precision=1), 3428104),
    (L.RPA_OP_CHI0, (20, 25, 32), 2, 2, dict(cocg_tol=1e-11), 3586576),
    (L.RPA_OP_CHI0, (20, 25, 32), 2, 2, dict(cocg_tol=1e-11, precision=1), 4162832),
    (L.RPA_OP_CHI0, (24, 23, 25), 3, 2, dict(cocg_tol=1e-11, precision=1, cocg_max_iter=57), 5358872),
    (L.RPA_OP_CHI0, (13, 11, 13), 2, 64, dict(cocg_tol=1e-11, max_systems=6), 627224),
    (L.RPA_OP_CHI0, (24, 24, 24), 2, 3, dict(cocg_tol=1e-11, precision=1, mixed_min_omega=0.0), 5366808),
    (L.RPA_OP_CHI0, (52, 50, 12), 2, 2, dict(cocg_tol=1e-11, precision=1), 8115984),
    (L.RPA_OP_CHI0, (24, 24, 24), 2, 3, dict(cocg_tol=1e-11, flags=1), 11962632),
    (L.RPA_OP_BACKWARD, (12, 13, 14), 2, 3, dict(cocg_tol=1e-11), 1004568),
    (L.RPA_OP_BACKWARD, (12, 13, 14), 2, 3, dict(cocg_tol=1e-11, precision=1), 1014296),
    (L.RPA_OP_BACKWARD, (20, 20, 21), 2, 3, dict(cocg_tol=1e-11), 3845400),
    (L.RPA_OP_BACKWARD, (20, 20, 21), 2, 3, dict(cocg_tol=1e-11, precision=1), 3879448),
    (L.RPA_OP_BACKWARD, (27, 27, 25), 2, 3, dict(cocg_tol=1e-11), 8333848),
    (L.RPA_OP_BACKWARD, (27, 27, 25), 2, 3, dict(cocg_tol=1e-11, precision=1), 8407576),
    (L.RPA_OP_SUBSPACE, (24, 24, 24), 2, 8, dict(cocg_tol=1e-11, subspace_iters=2, ec_tol=0.0), 15963424),
    (L.RPA_OP_SUBSPACE, (11, 13, 12), 2, 130, dict(cocg_tol=1e-11, subspace_iters=1, ec_tol=0.0), 33634592),
    (L.RPA_OP_ENERGY, (24, 24, 24), 2, 4, dict(cocg_tol=1e-11, subspace_iters=2, ec_tol=0.0), 8871424),
    (L.RPA_OP_ENERGY, (20, 20, 21), 2, 4, dict(cocg_tol=1e-11, subspace_iters=2, ec_tol=0.0, freq_mode=1), 11039488),
]


def call(so, op, cell, ns, nv, opts, ptr, ws, ws_bytes, out):
    """The C entry point of the operation; ptr(k, count) is a device address for argument k."""
    o, nd = L.default_options(**opts), int(np.prod(cell.n))
    one = (ctypes.c_double * 2)(1.0, 0.5)
    c = ctypes.byref(cell)
    if op == L.RPA_OP_CHI0:
        return so.rpa_apply_chi0(c, 0.5, nv, ptr(0, nv * nd), ptr(1, nv * nd), ctypes.byref(o), out, ws,
                                 ws_bytes, None)
    if op == L.RPA_OP_SUBSPACE:
        E = ctypes.c_double()
        return so.rpa_subspace_iter(c, 0.5, 1.0, nv, ptr(0, nv * nd), None, ptr(1, nv * nv), None,
                                    ctypes.byref(E), None, ctypes.byref(o), out, ws, ws_bytes, None)
    if op == L.RPA_OP_ENERGY:
        v0 = (ctypes.c_void_p * 1)(ptr(0, nv * nd))
        cs = (ctypes.c_void_p * 1)(ptr(1, 2 * nv * nv))
        ec = (ctypes.c_double * 1)()
        return so.rpa_energy(1, c, (ctypes.c_int32 * 1)(nv), 2, one, one, v0, None, cs, ctypes.byref(o),
                             ec, None, None, out, ws, ws_bytes, None)
    return so.rpa_energy_backward(c, 2, one, one, nv, ptr(0, 2 * nv * nd), ptr(2, 2 * nv * nv), 1.0,
                                  ptr(1, nd), ctypes.byref(o), out, ws, ws_bytes, None)


@pytest.mark.parametrize("op,n,ns,nv,opts,least", LEAST)
def test_least_state_is_accepted(op, n, ns, nv, opts, least):
    # host only: without a device an accepted call goes on to the first HIP call and fails there
    if torch.cuda.is_available():
        pytest.skip("made-up addresses: for hosts without a GPU")
    so = L.load()
    c = L.RpaCell()
    c.n[0], c.n[1], c.n[2] = n
    c.n_occ, c.h, c.v_loc, c.psi = ns, 0.45, 0x1000, 0x2000
    eps = np.arange(ns, dtype=np.float64)
    c.eps = eps.ctypes.data_as(ctypes.POINTER(ctypes.c_double))

    def ptr(k, count):
        return 0x100000 * (k + 1)

    assert call(so, op, c, ns, nv, opts, ptr, 0x10000000, least, None) == L.RPA_EHIP
    assert call(so, op, c, ns, nv, opts, ptr, 0x10000000, int(0.8 * least), None) == L.RPA_EWORKSPACE


@pytest.mark.parametrize("n,ns,nr,ncell,gib", [(48, 64, 256, 64, 204.44), (32, 28, 112, 200, 159.08),
                                               (40, 36, 36, 128, 137.02)])
def test_cells_that_share_the_budget_keep_to_it(n, ns, nr, ncell, gib):
    # many concurrent cells, each with few systems in flight: the longer rings are not added to the
    # 128 GiB of state that they share (gib: the whole workspace without them)
    cells = (L.RpaCell * ncell)()
    for c in cells:
        c.n[0] = c.n[1] = c.n[2] = n
        c.n_occ, c.h = ns, 0.4
    out = ctypes.c_size_t(0)
    assert L.load().rpa_workspace_size(L.RPA_OP_ENERGY, ncell, cells, (ctypes.c_int32 * ncell)(*[nr] * ncell),
                                       8, None, ctypes.byref(out)) == 0
    assert out.value <= 1.03 * gib * 2 ** 30, out.value / 2 ** 30


@pytest.mark.gpu
@pytest.mark.parametrize("op,n,ns,nv,opts,least", LEAST)
def test_least_state_gives_the_same_results(op, n, ns, nv, opts, least):
    print("least workspace", op, n, ns, nv, opts, flush=True)
    so, dev = L.load(), "cuda:0"
    dc = api.device_cell(make(n, ns, 21), dev)
    c = dc.c_struct()
    rng = np.random.default_rng(22)
    nd = dc.nd
    blocks = np.ascontiguousarray([np.linalg.qr(rng.standard_normal((nd, nv)))[0].T for _ in range(2)])
    Q = np.linalg.qr(rng.standard_normal((nv, nv)))[0]
    Cm = (Q * -np.linspace(0.1, 0.4, nv)) @ Q.T
    full = api.workspace_size(op, dc, nv, 2, L.default_options(**opts))
    outs = []
    for ws_bytes in (full, min(full, least)):
        args = [torch.tensor(blocks, device=dev),
                torch.full((max(nv * nd, 2 * nv * nv),), float("nan"), dtype=torch.float64, device=dev),
                torch.tensor(np.stack([0.5 * (Cm + Cm.T)] * 2), device=dev)]
        # the workspace holds not-a-numbers and 64 KiB behind it that have to stay
        buf = torch.full((ws_bytes // 8 + 8192 + 64,), float("nan"), dtype=torch.float64, device=dev)
        off = (-buf.data_ptr()) % 256 // 8
        end = off + (ws_bytes + 7) // 8
        buf[end:] = 7.0
        st = L.RpaStats()
        torch.cuda.synchronize()
        rc = call(so, op, c, ns, nv, opts, lambda k, m: args[k].data_ptr(), buf.data_ptr() + 8 * off,
                  ws_bytes, ctypes.byref(st))
        torch.cuda.synchronize()
        assert rc == 0, L.last_error()
        assert bool((buf[end:] == 7.0).all())
        out = args[1][:{L.RPA_OP_CHI0: nv * nd, L.RPA_OP_SUBSPACE: nv * nv,
                        L.RPA_OP_ENERGY: 2 * nv * nv, L.RPA_OP_BACKWARD: nd}[op]].cpu().numpy()
        outs.append((out, st.as_dict()))
    (a, sa), (b, sb) = outs
    # both meet a residual of 1e-11: cond(A) times that, and the second subspace step's inverse of
    # the spread of the Ritz values
    assert np.isfinite(a).all() and rel(b, a) < 1e-8
    assert abs(sa["cocg_iters_total"] - sb["cocg_iters_total"]) <= sa["cocg_systems"]
    assert sa["n_unconverged"] == sb["n_unconverged"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("share", [1.0, 0.5])
def test_breakdowns_in_the_least_state(share, monkeypatch):
    # complex64 solves that break down at the first step (solved afresh in real form, whose pool
    # reaches into the residuals), all of them or the half whose |b^T A b| / (|b| |A b|) is below
    # the threshold; what remains breaks down later, if at all, and is continued from its residual
    print("least workspace, breakdowns", share, flush=True)
    so, dev = L.load(), "cuda:0"
    n, ns, nv, least = (12, 13, 14), 3, 4, 1689136
    cell = make(n, ns, 23)
    dc = api.device_cell(cell, dev)
    U = np.random.default_rng(24).standard_normal((nv, dc.nd))
    b = build_rhs(U.T, cell.psi.T, cell.h ** 3)[0]
    Ab = fd.hamiltonian_apply(b, cell.vloc, n, cell.h) - (np.tile(cell.eps, nv) + 0.5j) * b
    ratio = np.abs((b * Ab).sum(0)) / np.linalg.norm(b, axis=0) / np.linalg.norm(Ab, axis=0)
    monkeypatch.setenv("RPA_MIXED_BD_TOL", repr(float(np.quantile(ratio, 0.5)) if share < 1 else 1e300))
    X = torch.tensor(U, device=dev)
    ref, _, _ = api.rpa_apply_chi0(dc, 0.5, X, dict(cocg_tol=1e-11))
    out, st = torch.empty_like(X), L.RpaStats()
    buf = torch.empty(least + 256, dtype=torch.uint8, device=dev)
    o = dict(cocg_tol=1e-11, precision=L.RPA_MIXED, mixed_min_omega=0.0)
    rc = call(so, L.RPA_OP_CHI0, dc.c_struct(), ns, nv, o, lambda k, m: (X, out)[k].data_ptr(),
              buf.data_ptr() + (-buf.data_ptr()) % 256, least, ctypes.byref(st))
    torch.cuda.synchronize()
    assert rc == 0 and st.fp64_fallbacks >= share * ns * nv and st.n_breakdown == 0
    assert rel(out.cpu().numpy(), ref.cpu().numpy()) < 1e-8
