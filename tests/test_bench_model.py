"""bench.py's operation counts of the thin QR: where the factor products are folded into Q's formation
(n >= 65536) the leaves make rank columns of p reflectors, and only picked blocks of Q itself."""
import types

import pytest

from test_bench_host import _bench


def _trace(p, rank):
    return [dict(I_pre=list(range(p)), J_pre=list(range(p)), nI=p, nJ=p, rank=rank, indicator=float("inf"), rho=float("inf"))]


@pytest.mark.parametrize("n,p,rank", [(1048575, 50, 25), (1048575, 50, 50), (65536, 64, 10)])
def test_folded_formation_counts_rank_columns(n, p, rank):
    b = _bench()
    w = types.SimpleNamespace(n=n, r_max=64)
    info = types.SimpleNamespace(rank=rank)
    m = b.kernel_model(w, "fp64", _trace(p, rank), info, 1)
    m0 = b.kernel_model(w, "fp64", [], info, 1)
    leaves = 2 * 2 * n * p * rank
    rows = -(-n // 256) * 64
    rest = 2 * (2 * rows * p ** 2 - 2 * p ** 3 / 3) + 2 * p * (2 * 256 * p ** 2 - 2 * p ** 3 / 3)
    assert m["tsqr_apply"]["flops"] - m0["tsqr_apply"]["flops"] == pytest.approx(leaves + rest, rel=1e-12)
    assert m["tsqr_factor"]["flops"] - m0["tsqr_factor"]["flops"] == pytest.approx(2 * (2 * n * p ** 2 - 2 * p ** 3 / 3))


def test_unfolded_formation_counts_the_whole_q():
    b = _bench()
    m = b.kernel_model(types.SimpleNamespace(n=65535, r_max=64), "mixed", _trace(40, 20), types.SimpleNamespace(rank=20), 20)
    assert m["tsqr_apply"]["flops"] == m["tsqr_factor"]["flops"]
