"""GPU parity of the real-form COCG kernel (real Lanczos basis, one sweep per iteration) against
the oracle's complex COCG, at the edges of its launch shapes: the smallest grid, one, two and
three rows per thread with and without a ragged last row group, odd and even n2, the classes of
the register-resident kernel by column height and plane, an isolated box, iteration caps around the ring of basis vectors, and launches of few and of many systems."""
import numpy as np
import pytest
import torch

from oracle import chi0 as ochi0
from paper_2504_01816_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    print(*a, flush=True)


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def make(shape, ns, seed, bc="periodic", h=0.45):
    """A cell with random orthonormal orbitals and eigenvalues below the spectrum of H, which is
    all that the solver sees of a ground state."""
    rng = np.random.default_rng(seed)
    nd = int(np.prod(shape))
    q = np.linalg.qr(rng.standard_normal((nd, ns)))[0].T
    vloc = rng.uniform(-1.0, 0.5, nd)
    eps = np.sort(rng.uniform(-2.0, -1.2, ns))
    return synth.Cell(shape, h, vloc, np.ascontiguousarray(q / np.sqrt(h ** 3)), eps, 0.0, 0.0,
                      seed, bc=bc)


def chi0(c, X, omega, tol, **opts):
    out, rc, st = api.rpa_apply_chi0(api.device_cell(c, DEV), omega, torch.tensor(X, device=DEV),
                                     dict(cocg_tol=tol, **opts))
    return out.cpu().numpy(), rc, st


# two FP64 solvers that meet a residual of 1e-12 differ by cond(A) 1e-12 <= 1e-9 here
@pytest.mark.parametrize("shape,bc", [
    ((7, 7, 12), "periodic"), ((7, 8, 13), "dirichlet"),
    ((16, 16, 16), "periodic"), ((18, 17, 15), "dirichlet"), ((24, 23, 14), "periodic"),
    ((32, 32, 12), "periodic"), ((33, 32, 12), "periodic"), ((35, 37, 13), "periodic"),
    ((35, 37, 12), "dirichlet"), ((48, 45, 12), "periodic"), ((47, 46, 13), "periodic"),
    ((46, 47, 12), "dirichlet"), ((52, 50, 12), "periodic")])
def test_real_form_matches_oracle(shape, bc, capfd, monkeypatch):
    say("real form", shape, bc)
    monkeypatch.setenv("RPA_COCG_VERBOSE", "1")
    c = make(shape, 2, 3, bc)
    X = np.random.default_rng(4).standard_normal((2, c.nd))
    for omega in (0.1, 2.0):
        out, rc, st = chi0(c, X, omega, 1e-12)
        ref, iters, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, omega, shape, c.h, 1e-12,
                                         5000, bc=bc)
        assert rc == 0 and rel(out.T, ref) < 1e-9, (omega, rel(out.T, ref))
        assert abs(st["cocg_iters_total"] - int(iters.sum())) <= iters.size
    # planes over 48 x 48 points stay on the complex kernel
    assert ("rcocg shape" in capfd.readouterr().err) == (shape[0] * shape[1] <= 48 * 48)


@pytest.mark.parametrize("cap", [1, 2, 3, 7, 8, 9, 16, 17])
def test_real_form_iteration_caps(cap):
    # the partial solution after `cap` steps, with a ring that is part full, full and just reused;
    # rounding alone separates the two after this few steps
    say("real form cap", cap)
    c = make((12, 13, 14), 3, 5)
    X = np.random.default_rng(6).standard_normal((2, c.nd))
    out, rc, st = chi0(c, X, 0.5, 1e-14, cocg_max_iter=cap)
    ref, _, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, 0.5, c.shape, c.h, 1e-14, cap)
    assert rc == 1 and st["cocg_iters_max"] == cap and st["n_unconverged"] == 6
    assert rel(out.T, ref) < 1e-11


def test_real_form_bits_do_not_depend_on_the_launch():
    # few systems keep a short ring, many a long one, and slots serve one system after another:
    # a column's bits are the same in every launch, and a zero column gives exactly zero
    say("real form, launch independence")
    c = make((14, 12, 13), 4, 7)
    X = np.random.default_rng(8).standard_normal((600, c.nd))
    X[5] = 0.0
    many, rc, st = chi0(c, X, 0.3, 1e-10)
    assert rc == 0 and st["cocg_systems"] == 2400 and np.all(many[5] == 0.0)
    few, _, _ = chi0(c, X[3:7], 0.3, 1e-10)
    assert np.array_equal(few, many[3:7])
    mixed, _, _ = chi0(c, X[3:7], 0.1, 1e-10, precision=1)
    fp64, _, _ = chi0(c, X[3:7], 0.1, 1e-10)
    assert np.array_equal(mixed, fp64)


def test_real_form_eigenvector_right_hand_sides():
    # plane waves on a constant potential: every right-hand side is an eigenvector of A, so the
    # first step converges and the sum of squares that gives beta cancels; a small second wave
    # then needs exactly one more step
    say("real form, eigenvectors")
    shape = (12, 14, 16)
    c = synth.uniform_cell(shape, 0.5, 0.3)
    z, y, x = np.meshgrid(*(np.arange(n) for n in shape[::-1]), indexing="ij")
    w1 = np.cos(2 * np.pi * x / 12).reshape(-1)
    w2 = np.sin(2 * np.pi * (y / 14 + 2 * z / 16)).reshape(-1)
    X = np.stack([w1, w2, w1 + 1e-5 * w2])
    out, rc, st = chi0(c, X, 0.7, 1e-10)
    ref, iters, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, 0.7, shape, 0.5, 1e-10, 5000)
    assert rc == 0 and st["cocg_iters_total"] == int(iters.sum())
    assert rel(out.T, ref) < 1e-12


@pytest.mark.parametrize("shape,bc", [((12, 13, 14), "periodic"), ((12, 13, 14), "dirichlet"),
                                      ((35, 37, 12), "dirichlet"), ((35, 37, 13), "periodic"),
                                      ((48, 45, 12), "periodic")])
def test_mixed_real_form_is_checked_and_continued(shape, bc):
    # the mixed path at omega >= mixed_min_omega: one exact residual per system; with a cap below
    # what the solves need, every system goes on in FP64 from x and that residual
    say("mixed, real form with the exact residual", shape, bc)
    c = make(shape, 2, 9, bc)
    X = np.random.default_rng(10).standard_normal((2, c.nd))
    ref, iters, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, 0.5, shape, c.h, 1e-10, 5000,
                                     bc=bc)
    out, rc, st = chi0(c, X, 0.5, 1e-10, precision=1)
    assert rc == 0 and st["refinements"] == 4 and st["n_unconverged"] == 0
    # the residual is met by both, so they differ by at most 2 cond(A) 1e-10
    assert rel(out.T, ref) < 1e-8
    cap = int(0.7 * iters.min())
    out, rc, st = chi0(c, X, 0.5, 1e-10, precision=1, cocg_max_iter=cap)
    assert rc == 0 and st["fp64_fallbacks"] == 4 and st["n_unconverged"] == 0
    assert rel(out.T, ref) < 1e-8


@pytest.mark.parametrize("shape,kind", [
    ((12, 12, 12), "resident"), ((7, 9, 12), "resident"), ((20, 25, 13), "resident"),
    ((21, 24, 15), "resident"), ((16, 32, 20), "resident"), ((52, 8, 12), "resident"),
    ((20, 20, 21), "resident-ring"), ((28, 18, 22), "resident-ring"),
    ((29, 22, 14), "resident-ring"), ((24, 24, 24), "resident-ring"),
    ((11, 10, 26), "resident-ring"), ((7, 8, 23), "resident-ring"), ((26, 27, 12), "resident-ring"),
    ((16, 15, 27), "resident-ring"), ((20, 22, 32), "resident-ring"),
    ((27, 27, 25), "streaming"), ((20, 25, 32), "streaming"), ((12, 12, 33), "streaming")])
def test_resident_classes(shape, kind, capfd, monkeypatch):
    # every class edge, periodic and isolated, real solutions and (mixed) complex ones
    say("resident classes", shape, kind)
    monkeypatch.setenv("RPA_COCG_VERBOSE", "1")
    X = np.random.default_rng(12).standard_normal((2, int(np.prod(shape))))
    for bc in ("periodic", "dirichlet"):
        c = make(shape, 2, 13, bc)
        ref, iters, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, 0.4, shape, c.h, 1e-12,
                                         5000, bc=bc)
        out, rc, st = chi0(c, X, 0.4, 1e-12)
        err = capfd.readouterr().err
        assert "shape %s " % kind in err, err
        assert rc == 0 and rel(out.T, ref) < 1e-9, rel(out.T, ref)
        assert abs(st["cocg_iters_total"] - int(iters.sum())) <= iters.size
        out, rc, st = chi0(c, X, 0.4, 1e-12, precision=1)
        assert rc == 0 and rel(out.T, ref) < 1e-9 and st["refinements"] == 4


@pytest.mark.parametrize("shape", [(16, 18, 17), (23, 24, 19), (30, 30, 30)])
def test_step_caps_of_every_kernel(shape):
    # partial solutions after few steps, FP64: resident, resident with a ring, streaming
    say("caps", shape)
    c = make(shape, 2, 14)
    X = np.random.default_rng(15).standard_normal((1, c.nd))
    for cap in (1, 2, 8, 9):
        out, rc, st = chi0(c, X, 0.5, 1e-14, cocg_max_iter=cap)
        ref, _, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, 0.5, shape, c.h, 1e-14, cap)
        assert rc == 1 and st["cocg_iters_max"] == cap and rel(out.T, ref) < 1e-11


@pytest.mark.parametrize("shape", [(12, 12, 33), (35, 37, 12), (46, 47, 12)])
@pytest.mark.parametrize("cap", [1, 8, 9, 15, 16, 17, 33])
def test_streaming_iteration_caps(shape, cap):
    # the partial solution after `cap` steps of the streaming kernel with one, two and three rows per
    # thread, in launches that keep a ring of 16 vectors (five vectors per system, 256 workgroups)
    # and in ones that keep 8: part full, full and just reused; the solves give the same bits
    say("streaming cap", shape, cap)
    c = make(shape, 2, 15)
    X = np.random.default_rng(16).standard_normal((2, c.nd))
    many, rc, st = chi0(c, np.concatenate([X] * 244), 0.5, 1e-14, cocg_max_iter=cap)
    ref, _, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, 0.5, c.shape, c.h, 1e-14, cap)
    few, _, _ = chi0(c, X, 0.5, 1e-14, cocg_max_iter=cap)
    assert rc == 1 and st["cocg_iters_max"] == cap
    assert rel(many[-2:].T, ref) < 1e-11 and rel(few.T, ref) < 1e-11
    # the projections of both launches are summed in as many parts (128 points each, at most 2048
    # over the tiles of 64 systems), so the right-hand sides are the same bits too
    if c.nd // 128 <= 2048 // 16:
        assert np.array_equal(many[:2], few) and np.array_equal(many[-2:], few)


@pytest.mark.parametrize("shape", [(35, 37, 12), (47, 46, 12), (41, 25, 12)])
def test_ragged_periodic_grids_of_the_smallest_height(shape):
    # rows that do not divide by the rows per thread, n2 = 12: the last plane that a sweep reads past
    # the periodic top is stored after the first of its two barriers
    say("ragged, n2 = 12", shape)
    c = make(shape, 2, 17)
    X = np.random.default_rng(18).standard_normal((2, c.nd))
    for omega in (0.1, 2.0):
        ref, iters, _ = ochi0.chi0_apply(X.T, c.vloc, c.psi.T, c.eps, omega, shape, c.h, 1e-12, 5000)
        for precision in (0, 1):
            out, rc, st = chi0(c, X, omega, 1e-12, precision=precision)
            # two FP64 solvers that meet a residual of 1e-12 differ by cond(A) 1e-12 <= 1e-9 here
            assert rc == 0 and rel(out.T, ref) < 1e-9, (omega, precision, rel(out.T, ref))


@pytest.mark.parametrize("shape", [(12, 13, 14), (20, 20, 21), (12, 12, 33), (35, 37, 12)])
def test_tiny_right_hand_sides_are_solved_or_reported(shape):
    # scaled by 1e-100 the solves are those of the unscaled block; by 1e-160 the squares of the
    # residuals are no normal numbers: a breakdown, or zero where complex64 stands for the block
    say("tiny right-hand sides", shape)
    c = make(shape, 2, 19)
    X = np.random.default_rng(20).standard_normal((2, c.nd))
    ref, rc, st = chi0(c, X, 0.5, 1e-10)
    out, rc2, st2 = chi0(c, X * 1e-100, 0.5, 1e-10)
    assert rc == 0 and rc2 == 0 and abs(st2["cocg_iters_total"] - st["cocg_iters_total"]) <= 4
    assert rel(out * 1e100, ref) < 1e-8              # both meet 1e-10, cond(A) times that
    for omega, precision in ((0.5, 0), (0.1, 1)):
        with pytest.raises(RuntimeError, match="breakdown"):
            chi0(c, X * 1e-160, omega, 1e-10, precision=precision)
    out, rc, st = chi0(c, X * 1e-160, 0.5, 1e-10, precision=1)
    assert rc == 0 and np.all(out == 0.0) and st["fp64_fallbacks"] == 0
