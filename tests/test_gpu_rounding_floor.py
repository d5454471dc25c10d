"""FP64 solves whose index sets outgrow the numerical rank of the solution (1 or 2 wide bumps, caps 24
and 32): Q(I,:) is then singular to 1e-12 and the cross approximation multiplies the rounding of the
thin QR by its reciprocals, so a QR of other rounding moves these solutions by 4e-9 to 4e-6. They are
pinned to stored ones, formed with the column-by-column QR and full-length transforms: the statuses,
passes and ranks, and the solution through Gaussian sketches Om^T U diag(S) V^T Om'.

Tolerance: the steps after the QRs (core SVD, products, transforms back) are backward stable and not
amplified, c p eps with p = 32 and a modest c a pass, over up to 20 passes: 1e-12."""
import json
import os

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

with open(os.path.join(os.path.dirname(__file__), "golden", "fp64_rounding_floor.json")) as f:
    CASES = json.load(f)


@pytest.mark.parametrize("case", CASES, ids=[f"n{c['n']}-{c['bumps']}-{c['tol']}" for c in CASES])
def test_fp64_at_the_rounding_floor(case):
    import torch

    from paper_2607_06021_amd import Solver, fortran

    n = case["n"]
    print(f"rounding floor n={n} bumps={case['bumps']} cap={case['r_max']} tol={case['tol']}", flush=True)
    U, s, V, _ = workloads.bump_rhs(n, case["seed"], case["bumps"], case["width_lo"], case["width_hi"])
    dev = [fortran(torch.from_numpy(U).cuda()), torch.from_numpy(s).cuda(), fortran(torch.from_numpy(V).cuda())]
    with Solver(n, case["r_max"], case["tol"], maxiter=20) as sol:
        Uo, So, Vo, r, info = sol.solve(*dev)
    A = np.random.default_rng(771).standard_normal((n, 12)).T @ (Uo[:, :r] * So[:r]).cpu().numpy()
    B = np.random.default_rng(772).standard_normal((n, 12)).T @ Vo[:, :r].cpu().numpy()
    ref = np.array(case["sketch"])
    err = np.linalg.norm(A @ B.T - ref) / np.linalg.norm(ref)
    print(f"  status {info.status} passes {info.iters} rank {r}; sketched difference {err:.1e}")
    assert (info.status, info.iters, r) == (case["status"], case["iters"], case["rank"])
    assert err <= 1e-12
