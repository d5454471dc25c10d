"""The panel kernels of the thin QR (lrp_tsqr below the solves that keep the column kernels): widths
at and around the 16-column panels and the 64-row waves, ragged last blocks, rank caps that stack
whole and broken tiles, zero columns and rows, and columns of extreme magnitude.

Tolerances: a Householder QR of m rows is columnwise backward stable, |A_c - (QR)_c| <= k p eps
|A_c| per level with a modest k; 20 per level here, and the same for Q^T Q - I."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0**-52


def _tree_r(A, r_max):
    """R by LAPACK through the same tree: the signs of a Householder QR's rows depend on it."""
    p, rows, step, levels = A.shape[1], A, 256, 0
    while True:
        Rs = []
        for b in range(0, rows.shape[0], step):
            R = np.linalg.qr(np.vstack([rows[b:b + step], np.zeros((max(0, p - step), p))]), mode="r")
            Rs.append(np.vstack([R, np.zeros((r_max - R.shape[0], p))]))
        levels += 1
        if len(Rs) == 1:
            return Rs[0][:p], levels
        rows, step = np.vstack(Rs), 256 // r_max * r_max


CASES = [(n, p, rm) for n, p, rm in [
    (2, 1, 1), (64, 64, 64), (255, 16, 16), (256, 17, 64), (257, 15, 64), (300, 64, 64), (513, 1, 64),
    (1000, 33, 45), (1000, 31, 32), (1025, 49, 64), (1300, 63, 63), (2000, 47, 48), (4095, 20, 20),
    (5000, 5, 7), (16385, 64, 64), (16385, 32, 64), (70000, 17, 24)]]


@pytest.mark.parametrize("kind", ["rand", "scaled", "zeros"])
@pytest.mark.parametrize("n,p,r_max", CASES)
def test_panel_qr(n, p, r_max, kind):
    import torch

    from paper_2607_06021_amd import Solver, fortran

    print(f"panel qr n={n} p={p} r_max={r_max} {kind}", flush=True)
    rng = np.random.default_rng(1000 * p + n)
    A = rng.standard_normal((n, p))
    if kind == "scaled":  # squares outside the range of the reciprocal square root's Newton steps
        A *= 10.0 ** rng.choice([-150.0, 0.0, 150.0], p)
    if kind == "zeros":
        A[:, rng.random(p) < 0.3] = 0.0
        A[n // 3: n // 2] = 0.0
    with Solver(n, r_max, 1e-10) as s:
        Qd, Rd = s.tsqr(fortran(torch.from_numpy(A).cuda()))
        Q, R = Qd.cpu().numpy(), Rd.cpu().numpy()
    Rt, levels = _tree_r(A, r_max)
    tol = 20.0 * levels * p * EPS
    norms = np.sqrt(np.sum((A / np.maximum(np.abs(A).max(0), 1e-300)) ** 2, 0)) * np.abs(A).max(0)
    assert np.array_equal(np.tril(R, -1), np.zeros((p, p)))
    assert np.linalg.norm(Q.T @ Q - np.eye(p)) <= tol
    scale = np.where(norms > 0.0, norms, 1.0)
    assert np.linalg.norm(Q @ (R / scale) - A / scale, axis=0).max() <= tol
    if kind != "zeros" and n > 2 * p:  # well-conditioned: R is determined, row signs included
        assert np.abs((R - Rt) / scale).max() <= 1e3 * tol
