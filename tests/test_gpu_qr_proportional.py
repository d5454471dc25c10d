"""Exactly proportional columns that are one large entry and noise at its rounding level, as the fibers of
a sine mode are: after the first column the QR has nothing left to factor. Through both entry points and
with the column kernels of the FP64 solves.

Bound: of column c = a_c column 0 the first reflector leaves, per level of the tree, the rounding of its
own formation and update: the reciprocals and roots (1 eps each, 3), the products and sums (half an eps
each, 8): 7 eps of the large entry, 8 with the noise rows."""
import numpy as np
import pytest

from test_gpu_panel_qr import EPS, _tree_r
from test_gpu_solve_kernels import SolveKernels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", [0, 0.3, 1])
@pytest.mark.parametrize("n,p", [(64, 17), (256, 33), (1000, 20), (5000, 64)])
def test_proportional_columns(n, p, where):
    import torch

    from paper_2607_06021_amd import Solver, fortran, lrp

    print(f"proportional qr n={n} p={p} at {where}", flush=True)
    rng = np.random.default_rng(n + p)
    base = 1e-17 * rng.standard_normal(n)
    base[int(where * (n - 1))] = 0.37
    A = np.outer(base, np.concatenate([[1.0], rng.standard_normal(p - 1)]))
    Ad = fortran(torch.from_numpy(A).cuda())
    out = []
    for cls in (Solver, SolveKernels):
        with cls(n, p, 1e-10) as s:
            out.append(s.tsqr(Ad))
    Q, R = torch.empty_like(Ad), torch.full((p, p), float("nan"), dtype=torch.float64, device="cuda").t()
    st = torch.cuda.current_stream().cuda_stream
    assert lrp.lib().lrp_tsqr_noalloc(n, p, Ad.data_ptr(), n, Q.data_ptr(), n, R.data_ptr(), p, st) == 0
    torch.cuda.synchronize()
    out.append((Q, R))
    levels = _tree_r(A, p)[1]
    norms = np.linalg.norm(A, axis=0)
    for Qd, Rd in out:
        Qh, Rh = Qd.cpu().numpy(), Rd.cpu().numpy()
        left = np.linalg.norm(Rh[1:], axis=0) / norms
        print(f"  left over: {left.max() / EPS:.2f} eps, none in {np.mean(left[1:] < EPS / 64):.2f} of the columns")
        assert left.max() <= 8 * levels * EPS
        assert np.linalg.norm(Qh @ (Rh / norms) - A / norms, axis=0).max() <= 20.0 * levels * p * EPS
        assert np.linalg.norm(Qh.T @ Qh - np.eye(p)) <= 20.0 * levels * p * EPS
