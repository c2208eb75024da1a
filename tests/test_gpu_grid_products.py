"""The grid's products U = X O and V = X^T U in both tile sizes (64 x 64 from 256
tiles on, 32 x 32 below), with odd rows, columns and reduction lengths.

One MM iteration of a grid solves (X^T X + M) beta = c per column, M from the
marginal fits beta0; the residual of that system is formed here in FP64.  Bar:
1e-8 ||c||.  The solver stops at 1e-12; over s steps its recurrence drifts from
the true residual by at most about s 2^-52 ||X^T X + M|| ||beta|| / ||c|| = 1e-9
(s = 1000, n p = 3e6, ||beta|| = 30, ||c|| = 2e4), and the rounding of beta0 moves a
weight by 1e-14 over the smallest difference, 1e-10.
"""
import numpy as np
import pytest

import flrgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def flr():
    import torch

    assert torch.cuda.is_available()
    import paper_1306_1970_amd as m

    return m


@pytest.fixture(scope="module")
def ctx(flr):
    c = flr.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,p,cols,dtype", [(33, 65, 2, flrgen.F64), (131, 4001, 33, flrgen.F32),
                                            (301, 8999, 130, flrgen.F32), (257, 9001, 129, flrgen.BF16),
                                            (1101, 2049, 257, flrgen.F64)])
def test_columns_solve_their_systems(flr, ctx, n, p, cols, dtype):
    inst = flrgen.small_instance(n, p, "chain", dtype=dtype, seed=n)
    l1 = np.linspace(0.3, 1.5, cols)
    l2 = np.linspace(1.2, 0.4, cols)
    print("grid n=%d p=%d columns=%d" % (n, p, cols), flush=True)
    prob = flr.Problem.from_instance(ctx, inst)
    st, beta, res = prob.solve_grid(l1, l2, tol=1e-14, inner_tol=1e-12, max_iter=1, max_cg=20 * p)
    prob.close()
    X = inst.X
    if dtype == flrgen.BF16:
        X = (X.astype(np.uint32) << 16).view(np.float32)
    X = X.astype(np.float64)
    c = X.T @ inst.y
    b0 = c / np.sum(X * X, axis=0)
    B = beta.T
    flow = (B[:-1] - B[1:]) * (l2 / (np.abs(b0[:-1] - b0[1:]) + inst.eps)[:, None])
    R = c[:, None] - X.T @ (X @ B) - l1 * (B / (np.abs(b0) + inst.eps)[:, None])
    R[:-1] -= flow
    R[1:] += flow
    rel = np.linalg.norm(R, axis=0) / np.linalg.norm(c)
    print("  residuals %.2g .. %.2g, %d .. %d PCG steps" % (rel.min(), rel.max(), min(r["cg_iters"] for r in res),
                                                            max(r["cg_iters"] for r in res)), flush=True)
    assert rel.max() <= 1e-8
