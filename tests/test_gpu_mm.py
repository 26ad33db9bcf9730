"""The GPU Maffettone-Minale integrator (sclbm_mm_integrate) against the FP64
reference of oracle/mm.py on OU-driven trajectories (same RK4 scheme, the GPU
contracts multiply-adds: agreement to 1e-10)."""
import numpy as np
import pytest

from oracle import mm
from paper_2112_09972_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_mm_gpu_matches_reference():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_09972_amd as sc
    ntraj, nrows, R = 6, 801, 10.0
    tau_d = wl.eta_s() * R / wl.SIGMA
    A = np.stack([wl.ou_gradient_table(500 + t, 64, nrows, mach=0.05 + 0.03 * t) for t in range(ntraj)])
    Mg = sc.mm_integrate(A, tau_d, 1.0, substeps=2, record_every=50).cpu().numpy()
    assert Mg.shape == (ntraj, 17, 3, 3)
    for t in range(ntraj):
        Mo = mm.integrate(A[t].reshape(nrows, 3, 3), tau_d, 1.0, substeps=2, record_every=50)
        assert np.abs(Mg[t] - Mo).max() <= 1e-10
    # deformations span a useful range
    Ds = [mm.deformation(M) for M in Mg[:, -1]]
    assert max(Ds) > 0.01


@pytest.mark.parametrize("ntraj,nrows,substeps,every,start", [
    (1, 1, 1, 1, "I"), (1, 2, 1, 1, "I"), (16, 9, 1, 3, "I"), (17, 10, 3, 1, "I"), (33, 8, 2, 7, "I"),
    (8193, 6, 1, 2, "I"), (1, 1, 2, 1, "M0"), (1, 2, 1, 1, "M0"), (64, 4, 2, 1, "M0"), (65, 7, 3, 2, "M0")])
def test_mm_chunks_and_starts(ntraj, nrows, substeps, every, start):
    """Both kernels (start from I, any start) at the edges of their trajectory
    groups (16 and 64) and substep chunks (8 and 2), an asymmetric start included,
    against the FP64 reference.  Up to 27 RK4 steps of about 100 roundings of
    1.1e-16 each on entries of order one: 3e-13 if they all added up."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_09972_amd as sc
    rng = np.random.default_rng(ntraj * 100 + nrows)
    A = 0.02 * rng.standard_normal((ntraj, nrows, 9))
    M0 = None if start == "I" else np.eye(3).reshape(9) + 0.1 * rng.standard_normal((ntraj, 9))
    got = sc.mm_integrate(A, 19.0, 1.3, substeps=substeps, record_every=every, M0=M0).cpu().numpy()
    assert got.shape == (ntraj, 1 + (nrows - 1) // every, 3, 3)
    for t in sorted({0, 15 % ntraj, 16 % ntraj, ntraj // 2, ntraj - 1}):
        ref = mm.integrate(A[t].reshape(nrows, 3, 3), 19.0, 1.3, substeps=substeps, record_every=every,
                           M0=None if M0 is None else M0[t].reshape(3, 3))
        assert np.abs(got[t] - ref).max() <= 3e-13, (t, np.abs(got[t] - ref).max())


@pytest.mark.parametrize("fill", [np.nan, np.inf])
@pytest.mark.parametrize("ntraj,nrows,valid,substeps,start", [
    (3, 12, 2, 1, "I"), (17, 40, 9, 1, "I"), (17, 40, 8, 2, "I"), (5, 30, 23, 3, "I"), (4, 12, 1, 1, "I"),
    (8193, 7, 4, 1, "I"), (70, 12, 5, 2, "M0")])
def test_mm_records_do_not_depend_on_later_rows(ntraj, nrows, valid, substeps, start, fill):
    """Tables padded past their `valid` rows (with NaN or infinity): every record up
    to row valid - 1 holds the same bytes as with a table of `valid` rows, at and
    off the edges of the eight-substep chunks; the records after it are not finite."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_09972_amd as sc
    rng = np.random.default_rng(ntraj + valid)
    A = 0.02 * rng.standard_normal((ntraj, nrows, 9))
    A[:, valid:] = fill
    M0 = None if start == "I" else np.eye(3).reshape(9) + 0.1 * rng.standard_normal((ntraj, 9))
    got = sc.mm_integrate(A, 19.0, 1.3, substeps=substeps, M0=M0).cpu().numpy()
    want = sc.mm_integrate(A[:, :valid], 19.0, 1.3, substeps=substeps, M0=M0).cpu().numpy()
    assert np.isfinite(want).all()
    assert np.array_equal(got[:, :valid], want)
    assert not np.isfinite(got[:, valid:]).any()
