"""M^-1 of graphs with index bandwidth bw >= 2: the nested dense inverses of the
single solve and the blocked sweeps of the grid, at sizes where they can go
wrong: orders around one tile (64), segments with a short last one, separators
that straddle tiles, bandwidths at both ends of each block size of the sweeps
(W = bw + 1 = 16 .. 31, 32 .. 63, 64 .. 107) and just outside, orders that leave
a short last block; and one order whose inverses would pass 4 GB, where the single
solve keeps the band factor.

X = I, so Q = I + M is banded and every MM iterate follows from a banded
Cholesky solve.  Bar: 1e-8 of max |beta| (the FP64 bar of the parity tests), and
the PCG step count within 2 % (at least 5 steps) of a CPU run of the same
recurrence whose M^-1 is scipy's banded Cholesky solve.
"""
import numpy as np
import pytest
from scipy.linalg import solveh_banded

pytestmark = pytest.mark.gpu
INNER, EPS, L1, L2, STEPS = 1e-12, 1e-8, 0.3, 0.7, 2


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


def _case(p, bw):
    rng = np.random.default_rng(1000 * p + bw)
    y = np.repeat(rng.uniform(-2, 2, p // 9 + 1), 9)[:p] * (rng.random(p) < 0.7) + 0.3 * rng.standard_normal(p)
    y[p // 2] = y[p // 2 - 1]  # equal neighbours: a weight of 1 / eps
    j = np.arange(p - 1)
    e = [np.stack([j, j + 1], 1), np.stack([np.arange(p - bw), np.arange(bw, p)], 1)]
    k = rng.integers(0, p - 1, p // 3)  # and some edges of every length up to bw
    d = rng.integers(1, bw + 1, p // 3)
    keep = k + d < p
    e.append(np.stack([k[keep], k[keep] + d[keep]], 1))
    return y, np.unique(np.concatenate(e), axis=0).astype(np.int64)


def _reference(y, e, bw):
    """STEPS MM iterations by direct solves, and the PCG steps they take with M^-1 from a banded Cholesky solve."""
    p, b, cg = y.size, y.copy(), 0
    j, k = e[:, 0], e[:, 1]
    nc = np.linalg.norm(y)
    for _ in range(STEPS):
        a = L1 / (np.abs(b) + EPS)
        w = L2 / (np.abs(b[j] - b[k]) + EPS)
        ab = np.zeros((bw + 1, p))
        ab[bw - (k - j), k] = -w
        ab[bw] = a + np.bincount(j, w, p) + np.bincount(k, w, p)

        def m(v):
            d = w * (v[j] - v[k])
            return a * v + np.bincount(j, d, p) - np.bincount(k, d, p)

        x = b.copy()
        r = y - (x + m(x))
        z = solveh_banded(ab, r)
        q, rz = z.copy(), r @ z
        while True:
            v = q + m(q)
            nu = rz / (q @ v)
            x += nu * q
            r -= nu * v
            cg += 1
            if not np.linalg.norm(r) / nc > INNER:
                break
            z = solveh_banded(ab, r)
            rzn = r @ z
            q = z + rzn / rz * q
            rz = rzn
        ab[bw] += 1.0
        b = solveh_banded(ab, y)
    return b, cg


def _check(what, beta, n, ref, cg):
    err = np.max(np.abs(beta - ref)) / np.max(np.abs(ref))
    print("  %s: err %.2g, %d PCG steps (reference %d)" % (what, err, n, cg), flush=True)
    assert err <= 1e-8
    assert abs(n - cg) <= max(5, cg // 50)


@pytest.mark.parametrize("p,bw", [(4, 2), (63, 5), (64, 63), (65, 64), (129, 17), (1000, 999), (1600, 2), (1901, 43),
                                  (2300, 70), (4099, 64), (4900, 130), (250001, 3)])
def test_single(flr, ctx, p, bw):
    y, e = _case(p, bw)
    print("single p=%d bw=%d" % (p, bw), flush=True)
    ref, cg = _reference(y, e, bw)
    prob = flr.Problem.flsa(ctx, y, e)
    for _ in range(2):  # the second factorization overwrites the first one's
        s = prob.solve(L1, L2, tol=1e-14, inner_tol=INNER, max_iter=STEPS)
        _check("single", s.beta, s.cg_iters, ref, cg)
    prob.close()


@pytest.mark.parametrize("p,bw", [(40, 14), (16, 15), (47, 15), (321, 30), (64, 31), (333, 31), (500, 62), (64, 63),
                                  (449, 63), (777, 100), (640, 106), (500, 107)])
def test_grid(flr, ctx, p, bw):
    y, e = _case(p, bw)
    print("grid p=%d bw=%d" % (p, bw), flush=True)
    ref, cg = _reference(y, e, bw)
    prob = flr.Problem.flsa(ctx, y, e)
    for static in (False, True):
        st, beta, res = prob.solve_grid([L1, 2 * L1, L1], [L2, L2, L2], tol=1e-14, static=static, inner_tol=INNER,
                                        max_iter=STEPS)
        _check("column 0", beta[0], res[0]["cg_iters"], ref, cg)
        _check("column 2", beta[2], res[2]["cg_iters"], ref, cg)
    prob.close()
