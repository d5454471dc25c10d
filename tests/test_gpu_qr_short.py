"""The panel QR where a level is one short block: Q's formation then covers 64, 128 or 256 rows. Matrices
of one block with rows at and around 64 and 128, and trees whose root has so few rows, through both entry
points (a context's r_max stacks r_max rows per block, the allocation-free one p). Tolerances as in
test_gpu_panel_qr.py: 20 p eps per level, columnwise."""
import numpy as np
import pytest

from test_gpu_panel_qr import EPS, _tree_r

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p", [(1, 1), (17, 17), (20, 17), (33, 32), (63, 33), (64, 1), (64, 64), (65, 17), (65, 64),
                                 (127, 49), (128, 48), (129, 33), (192, 64), (257, 17), (300, 40), (513, 32), (520, 33)])
def test_short_levels(n, p):
    import torch

    from paper_2607_06021_amd import Solver, fortran, lrp

    print(f"short qr n={n} p={p}", flush=True)
    A = np.random.default_rng(100 * n + p).standard_normal((n, p)) * 10.0 ** np.linspace(0, -6, p)
    Ad = fortran(torch.from_numpy(A).cuda())
    out = []
    if n > 2:
        with Solver(n, p, 1e-10) as s:
            out.append(s.tsqr(Ad))
    Q, R = torch.full_like(Ad, float("nan")), torch.full((p, p), float("nan"), dtype=torch.float64, device="cuda").t()
    st = torch.cuda.current_stream().cuda_stream
    assert lrp.lib().lrp_tsqr_noalloc(n, p, Ad.data_ptr(), n, Q.data_ptr(), n, R.data_ptr(), p, st) == 0
    torch.cuda.synchronize()
    out.append((Q, R))
    Rt, levels = _tree_r(A, p)
    tol = 20.0 * levels * p * EPS
    norms = np.linalg.norm(A, axis=0)
    for Qd, Rd in out:
        Qh, Rh = Qd.cpu().numpy(), Rd.cpu().numpy()
        assert np.array_equal(np.tril(Rh, -1), np.zeros((p, p)))
        assert np.linalg.norm(Qh.T @ Qh - np.eye(p)) <= tol
        assert np.linalg.norm(Qh @ (Rh / norms) - A / norms, axis=0).max() <= tol
        if n > 2 * p:  # well-conditioned: R is determined, row signs included
            assert np.abs((Rh - Rt) / norms).max() <= 1e3 * tol
