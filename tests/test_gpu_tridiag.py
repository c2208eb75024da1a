"""The tridiagonal factor of M as a scan of Moebius maps and the block kernel's
variants: sizes at the edges of a solver block (256), of the one workgroup that
holds two (512), of two blocks per workgroup (128 blocks, an odd number of them),
of a grid chunk (2048) and of the two-level scan (more than 256 blocks), broken chains (no coupling at some indexes) and weights that
span sixteen decades.

X = I, so Q = I + M is tridiagonal and every MM iterate follows from a direct
elimination.  Bar: 1e-8 of max |beta| (the FP64 bar of the parity tests), and
the PCG step count within 2 % (at least 5 steps) of a CPU run of the same
recurrence whose M^-1 is scipy's banded Cholesky solve: a factor that is not
M's would need another number of steps.
"""
import numpy as np
import pytest
from scipy.linalg import solveh_banded

import flrgen

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


def _case(p, broken):
    rng = np.random.default_rng(p)
    y = flrgen.piecewise_beta(p, max(1, min(20, p // 4)), 0.5, rng) + 0.3 * rng.standard_normal(p)
    if p > 8:
        y[p // 2:p // 2 + 3] = y[p // 2]  # equal neighbours: a weight of 1 / eps
    e = flrgen.chain_edges(p)
    if broken:
        e = e[np.arange(e.shape[0]) % 7 != 3]
    return y, e


def _reference(y, e):
    """STEPS MM iterations by direct solves, and the PCG steps they take with M^-1 from a banded Cholesky solve."""
    p, b, cg = y.size, y.copy(), 0
    nc = np.linalg.norm(y)
    for _ in range(STEPS):
        a = 1.0 / (np.abs(b) + EPS)
        w = np.zeros(max(p - 1, 1))
        if e.size:
            w[e[:, 0]] = L2 / (np.abs(b[e[:, 0]] - b[e[:, 1]]) + EPS)
        w = w[:p - 1]
        ab = np.zeros((2, p))
        ab[1] = L1 * a
        ab[1, :-1] += w
        ab[1, 1:] += w
        ab[0, 1:] = -w

        def m(v):
            d = w * (v[1:] - v[:-1])
            out = L1 * a * v
            out[:-1] -= d
            out[1:] += d
            return out

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
        full = ab.copy()
        full[1] += 1.0
        b = solveh_banded(full, y)
    return b, cg


@pytest.mark.parametrize("p,broken", [(2, False), (9, True), (255, False), (256, True), (257, False), (512, True),
                                      (513, False), (2048, False), (2049, True), (5000, False), (32513, True),
                                      (32769, False), (66000, True)])
def test_scan_factor(flr, ctx, p, broken):
    y, e = _case(p, broken)
    print("chain p=%d broken=%s" % (p, broken), flush=True)
    ref, cg = _reference(y, e)
    prob = flr.Problem.flsa(ctx, y, e)
    s = prob.solve(L1, L2, tol=1e-14, inner_tol=INNER, max_iter=STEPS)
    st, beta, res = prob.solve_grid([L1, L1], [L2, L2], tol=1e-14, inner_tol=INNER, max_iter=STEPS)
    prob.close()
    scale = np.max(np.abs(ref))
    for got, n in ((s.beta, s.cg_iters), (beta[0], res[0]["cg_iters"]), (beta[1], res[1]["cg_iters"])):
        err = np.max(np.abs(got - ref)) / scale
        print("  err %.2g, %d PCG steps (reference %d)" % (err, n, cg), flush=True)
        assert err <= 1e-8
        assert abs(n - cg) <= max(5, cg // 50)
