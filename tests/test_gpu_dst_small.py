"""General-n DSTs on both sides of the line between full-length and odd-half transforms (at most
1 MB of transform data a buffer, M <= 2^14 points in FP64 and 2^15 in FP32): the last column count of
the one and the first of the other per length, and power-of-two sizes with so few columns that the
narrowest tiles run, up to the largest, whose wide tiles are two columns. Against the oracle, with the tolerances of the other DST tests (a few eps per
butterfly level)"""
import math

import numpy as np
import pytest

from oracle import crossdeim as cd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,edge64,edge32", [(1024, 16, 32), (2046, 16, 32), (2048, 8, 16), (4094, 8, 16),
                                             (4096, 0, 8), (8190, 0, 8)])
def test_dst_at_the_line(n, edge64, edge32):
    import torch

    from paper_2607_06021_amd import Solver, fortran

    print(f"dst line n={n}", flush=True)
    X = np.random.default_rng(n).standard_normal((n, max(edge64, edge32) + 2))
    ref = cd.dst1(X)
    lg = math.log2(4 * (n + 1))
    with Solver(n, 32, 1e-10) as s:
        for prec, edge, tol in (("fp64", edge64, 2e-15 * lg), ("mixed", edge32, 2e-6 * lg)):
            for cols in {1, max(edge - 1, 1), max(edge, 1), edge + 1, edge + 2}:
                Y = s.dst1(fortran(torch.from_numpy(X[:, :cols].copy()).cuda()), precision=prec)
                torch.cuda.synchronize()
                err = np.abs(Y.cpu().numpy() - ref[:, :cols]).max() / np.abs(ref[:, :cols]).max()
                assert err <= tol, (prec, cols, err)


@pytest.mark.parametrize("n,cols", [(262143, 1), (524287, 1), (524287, 3), (1048575, 2), (1048575, 16),
                                    (2097151, 4), (4194303, 3), (8388607, 2)])
def test_dst_few_columns(n, cols):
    import torch

    from paper_2607_06021_amd import Solver, fortran

    print(f"dst few columns n={n} cols={cols}", flush=True)
    X = np.random.default_rng(n + cols).standard_normal((n, cols))
    ref = cd.dst1(X)
    lg = math.log2(2 * (n + 1))
    with Solver(n, max(2, cols // 2), 1e-10) as s:
        Xd = fortran(torch.from_numpy(X).cuda())
        for prec, tol in (("fp64", 2e-15 * lg), ("mixed", 2e-6 * lg)):
            Y = s.dst1(Xd, precision=prec)
            torch.cuda.synchronize()
            assert np.abs(Y.cpu().numpy() - ref).max() <= tol * np.abs(ref).max(), prec
