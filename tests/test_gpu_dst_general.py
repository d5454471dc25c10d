"""The DST-I at general n by the odd half of Bluestein's convolution (four-step sizes, n + 1 > 1024):
n + 1 just above a power of two (most padding) and just below one (least), odd column counts, more
column pairs than one round holds, and in FP32. Against the oracle; the tolerances of
test_gpu_kernels.py's DST tests (a few eps per butterfly level of the length-M transforms)."""
import math

import numpy as np
import pytest

from oracle import crossdeim as cd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cols", [(1024, 1), (1025, 33), (2046, 5), (2048, 2), (4094, 3), (4096, 64), (16382, 2),
                                    (16385, 35), (65534, 3), (100000, 5), (262142, 2)])
def test_dst_odd_half(n, cols):
    import torch

    from paper_2607_06021_amd import Solver, fortran

    print(f"dst general n={n} cols={cols}", flush=True)
    rng = np.random.default_rng(n + cols)
    X = rng.standard_normal((n, cols))
    scale = rng.standard_normal(cols)
    with Solver(n, 32, 1e-10) as s:
        Xd = fortran(torch.from_numpy(X).cuda())
        Y = s.dst1(Xd, scale=torch.from_numpy(scale).cuda(), mul=0.5)
        Y32 = s.dst1(Xd, precision="mixed")
        back = s.dst1(s.dst1(Xd))
        torch.cuda.synchronize()
        Y, Y32, back = Y.cpu().numpy(), Y32.cpu().numpy(), back.cpu().numpy()
    ref = cd.dst1(X)
    lg = math.log2(4 * (n + 1))
    assert np.abs(Y - 0.5 * ref * scale).max() <= 2e-15 * lg * np.abs(0.5 * ref * scale).max()
    assert np.abs(Y32 - ref).max() <= 2e-6 * lg * np.abs(ref).max()
    assert np.abs(back - X).max() <= 4e-15 * lg * np.abs(X).max()


@pytest.mark.parametrize("n", [4095, 8191, 16383, 32767, 131071, 524287])
@pytest.mark.parametrize("cols", [1, 63])
def test_dst_four_step_tiles(n, cols):
    """Two-pass transforms at n + 1 a power of two, each stage split and both tile widths."""
    import torch

    from paper_2607_06021_amd import Solver, fortran

    print(f"dst tiles n={n} cols={cols}", flush=True)
    rng = np.random.default_rng(n + cols)
    X = rng.standard_normal((n, cols))
    with Solver(n, 32, 1e-10) as s:
        Xd = fortran(torch.from_numpy(X).cuda())
        Y, Y32 = s.dst1(Xd), s.dst1(Xd, precision="mixed")
        torch.cuda.synchronize()
        Y, Y32 = Y.cpu().numpy(), Y32.cpu().numpy()
    ref = cd.dst1(X)
    lg = math.log2(2 * (n + 1))
    assert np.abs(Y - ref).max() <= 2e-15 * lg * np.abs(ref).max()
    assert np.abs(Y32 - ref).max() <= 2e-6 * lg * np.abs(ref).max()
