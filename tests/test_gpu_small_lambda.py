"""lambda1 small against lambda2: M = lambda1 A + lambda2 B comes close to singular,
and its solve inside PCG has to stay a usable preconditioner.

X = I, so Q = I + M and its smallest eigenvalue is at least 1: an iterate whose
residual is at most delta ||y|| is within delta ||y|| of the direct solve.  Bar:
that, plus the rounding of a residual evaluated in double precision, 4 ulp of
||Q||_inf max |beta|, both doubled for the reference's own.
"""
import numpy as np
import pytest
from scipy.linalg import solveh_banded

import flrgen

pytestmark = pytest.mark.gpu
INNER, EPS, L2 = 1e-10, 1e-8, 0.7


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


def _direct(y, e, bw, l1):
    """One MM iterate from y by a banded Cholesky solve; the iterate and ||Q||_inf."""
    p = y.size
    j, k = e[:, 0], e[:, 1]
    w = L2 / (np.abs(y[j] - y[k]) + EPS)
    ab = np.zeros((bw + 1, p))
    ab[bw - (k - j), k] = -w
    ab[bw] = 1.0 + l1 / (np.abs(y) + EPS) + np.bincount(j, w, p) + np.bincount(k, w, p)
    return solveh_banded(ab, y), 2.0 * ab[bw].max()


def _check(y, sol, ref, qnorm):
    err = np.max(np.abs(sol.beta - ref))
    bar = 2.0 * (INNER * np.linalg.norm(y) + 4 * 2.0 ** -53 * qnorm * np.max(np.abs(ref)))
    print("  err %.2g (bar %.2g), %d PCG steps" % (err, bar, sol.cg_iters), flush=True)
    assert err <= bar


@pytest.mark.parametrize("l1", [1e-12, 1e-17, 1e-30, 1e-300])
@pytest.mark.parametrize("p", [300, 1500])
def test_chain(flr, ctx, p, l1):
    rng = np.random.default_rng(p)
    y = flrgen.piecewise_beta(p, 20, 0.5, rng) + 0.1 * rng.standard_normal(p)
    y[p // 2:p // 2 + 3] = y[p // 2]  # equal neighbours: a weight of 1 / eps
    e = flrgen.chain_edges(p)
    print("chain p=%d lambda1=%g" % (p, l1), flush=True)
    ref, qnorm = _direct(y, e, 1, l1)
    prob = flr.Problem.flsa(ctx, y, e)
    s = prob.solve(l1, L2, tol=1e-14, inner_tol=INNER, max_iter=1, max_cg=20 * p)
    prob.close()
    assert s.cg_iters < 20 * p
    _check(y, s, ref, qnorm)


def _pcg_steps(y, e, bw, l1, eps, steps):
    """PCG steps of `steps` MM iterations on the CPU, M^-1 from scipy's banded Cholesky solve."""
    p, b, cg = y.size, y.copy(), 0
    j, k = e[:, 0], e[:, 1]
    nc = np.linalg.norm(y)
    for _ in range(steps):
        a = l1 / (np.abs(b) + eps)
        w = L2 / (np.abs(b[j] - b[k]) + eps)
        ab = np.zeros((bw + 1, p))
        ab[bw - (k - j), k] = -w
        ab[bw] = a + np.bincount(j, w, p) + np.bincount(k, w, p)

        def m(v):
            d = w * (v[j] - v[k])
            return a * v + np.bincount(j, d, p) - np.bincount(k, d, p)

        r = y - (b + m(b))
        z = solveh_banded(ab, r)
        q, rz = z.copy(), r @ z
        while True:
            v = q + m(q)
            nu = rz / (q @ v)
            b = b + nu * q
            r -= nu * v
            cg += 1
            if not np.linalg.norm(r) / nc > INNER:
                break
            z = solveh_banded(ab, r)
            rzn = r @ z
            q = z + rzn / rz * q
            rz = rzn
    return cg


@pytest.mark.parametrize("graph,p,l1,eps", [("lattice", 100, 1e-10, 1e-8), ("lattice", 100, 1e-8, 1e-10),
                                            ("lattice", 1600, 1e-10, 1e-8), ("allpairs", 60, 1e-5, 1e-8),
                                            ("allpairs", 60, 1e-5, 1e-11)])
def test_banded(flr, ctx, graph, p, l1, eps):
    # an explicit inverse of M rounds its small eigenvalues away here (up to 60 times the steps, or a numerical
    # failure), so the solve keeps the band factor.  The steps stay within a quarter of the CPU's: both
    # factorizations round, by different amounts.
    rng = np.random.default_rng(p)
    y = np.repeat(rng.uniform(-2, 2, p // 12 + 1), 12)[:p] + 0.1 * rng.standard_normal(p)
    e = flrgen.lattice_edges(int(p ** 0.5)) if graph == "lattice" else np.stack(np.triu_indices(p, 1), 1)
    e = np.asarray(e, dtype=np.int64)
    print("%s p=%d lambda1=%g eps=%g" % (graph, p, l1, eps), flush=True)
    cg = _pcg_steps(y, e, int((e[:, 1] - e[:, 0]).max()), l1, eps, 4)
    prob = flr.Problem.flsa(ctx, y, e)
    base = prob.footprint
    s = prob.solve(l1, L2, tol=1e-14, inner_tol=INNER, max_iter=4, eps=eps, max_cg=2000)
    print("  status %d, %d PCG steps (CPU %d)" % (s.status, s.cg_iters, cg), flush=True)
    assert s.status == flr.FLR_ERR_MAX_ITER  # all four MM steps ran
    assert s.cg_iters <= cg + max(5, cg // 4)
    assert prob.footprint == base
    prob.solve(0.3, L2, tol=1e-6)
    assert prob.footprint > base  # and where M is well conditioned the inverses are used
    prob.close()
