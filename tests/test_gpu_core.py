"""The dense core step at every row class of its Jacobi and Householder kernels: one pass on forced
index sets of sizes around the multiples of 16, square and of both rectangular shapes, against the
oracle's pass (sets, rank, branch, relative error <= 1e-10 as in every FP64 comparison). The
right-hand side has 64 random columns, so every sampled core is full and far from singular."""
import numpy as np
import pytest

import workloads
from oracle import crossdeim as cd
from test_gpu_solve import compare_fp64, gpu_solve

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (2, 1), (4, 5), (8, 9), (15, 16), (16, 16), (17, 16), (31, 33), (32, 32), (33, 32), (37, 37),
         (47, 48), (49, 48), (63, 64), (64, 64)]


def core_case(nI, nJ, n=150, cols=64):
    rng = np.random.default_rng(100 * nI + nJ)
    U, V = rng.standard_normal((n, cols)), rng.standard_normal((n, cols))
    s = np.exp(-0.05 * np.arange(cols))
    I = sorted(int(i) for i in rng.choice(n, nI, replace=False))
    J = sorted(int(j) for j in rng.choice(n, nJ, replace=False))
    return n, U, s, V, [(I, J)]


@pytest.mark.parametrize("nI,nJ", SIZES)
def test_core_sizes(nI, nJ):
    n, U, s, V, replay = core_case(nI, nJ)
    print(f"core {nI} x {nJ}", flush=True)
    o = cd.solve(n, U, s, V, 64, 1e-10, 1, replay=replay)
    compare_fp64(gpu_solve(n, U, s, V, 64, 1e-10, 1, replay=replay), o, f"core {nI}x{nJ}")


@pytest.mark.parametrize("n", [256, 257, 4097, 16641])
def test_rho_row_blocks(n):
    """rho, the indicator and the stop at 1, 2, 17 and 66 row blocks of 256 (one launch; sums with a
    remainder of 16 and of 64 blocks), against the oracle's values of every pass."""
    U, s, V = workloads.make(workloads.CONFIGS["n4095_r10_fp64"], 0, n=n)
    print(f"rho n={n}", flush=True)
    o = cd.solve(n, U, s, V, 32, 1e-10, 20)
    g = gpu_solve(n, U, s, V, 32, 1e-10, 20)
    assert any(np.isfinite(t["rho"]) for t in g["trace"])
    compare_fp64(g, o, f"rho n={n}")


@pytest.mark.parametrize("n", [65535, 65536])
def test_product_folded_into_q(n):
    """Both sides of the size from which the factors' products are taken above the leaves of the QR
    tree (the larger sizes and the column kernels: the n = 2^20 - 1 tests against stored values)."""
    U, s, V = workloads.make(workloads.CONFIGS["n4095_r10_fp64"], 1, n=n)
    print(f"fold n={n}", flush=True)
    o = cd.solve(n, U, s, V, 32, 1e-10, 20)
    compare_fp64(gpu_solve(n, U, s, V, 32, 1e-10, 20), o, f"fold n={n}")
