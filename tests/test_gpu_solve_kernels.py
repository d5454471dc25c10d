"""The kernels that only FP64 solves take, by themselves: the column-by-column QR and the full-length
Bluestein FFTs, through lrp_tsqr and lrp_dst1 of a context that a test switches to them. The same
matrices, sizes and bounds as the panel QR's and the odd-half transforms' own tests."""
import pytest

import paper_2607_06021_amd as pkg
import test_gpu_dst_general as dst_general
import test_gpu_kernels as kernels
import test_gpu_panel_qr as panel_qr
from paper_2607_06021_amd import lrp

pytestmark = pytest.mark.gpu


class SolveKernels(lrp.Solver):
    def __init__(self, *args, **kw):
        super().__init__(*args, **kw)
        assert lrp.lib().lrp_test_solve_kernels(self._h, 1) == 0


@pytest.fixture(autouse=True)
def solve_kernels(monkeypatch):
    monkeypatch.setattr(pkg, "Solver", SolveKernels)


def test_switch_selects_other_kernels():
    """The two QRs agree to rounding but not in every bit."""
    import torch

    n, p = 5000, 45
    A = torch.randn((p, n), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1)).t()
    with lrp.Solver(n, p, 1e-10) as a, SolveKernels(n, p, 1e-10) as b:
        Ra, Rb, Rc = a.tsqr(A)[1], b.tsqr(A)[1], b.tsqr(A)[1]
    assert torch.equal(Rb, Rc) and not torch.equal(Ra, Rb)
    # both backward stable: |dA| <= 20 p eps per level (four levels), R about as well conditioned as A (kappa < 2)
    assert (Ra - Rb).norm() <= 2 * 2 * 20 * 4 * p * 2.0**-52 * A.norm()


@pytest.mark.parametrize("kind", ["rand", "zeros"])
@pytest.mark.parametrize("n,p,r_max", panel_qr.CASES)
def test_column_qr(n, p, r_max, kind):
    panel_qr.test_panel_qr(n, p, r_max, kind)


@pytest.mark.parametrize("n,p,kind", [(255, 5, "rand"), (4095, 64, "ill"), (65535, 64, "ill"), (65535, 20, "deficient"),
                                      (1023, 64, "fibers"), (63, 63, "rand"), (511, 63, "ill"), (16383, 33, "rand")])
def test_column_qr_householder(n, p, kind):
    kernels.test_tsqr_matches_householder(n, p, kind)


@pytest.mark.parametrize("n,cols", [(1024, 1), (1025, 33), (2046, 5), (2048, 2), (4094, 3), (4096, 64), (16382, 2),
                                    (16385, 35), (65534, 3), (100000, 5), (262142, 2), (700000, 2), (1500000, 1)])
def test_full_length_dst(n, cols):
    dst_general.test_dst_odd_half(n, cols)
