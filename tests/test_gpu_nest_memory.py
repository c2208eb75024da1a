"""What a handle's memory is charged with.  Nested dense inverses: taken by the first solve that applies
them and by no other, never a reason to refuse a request or a solve, and given
back when a server's budget cannot hold it.  Without it a solve applies the
banded factor: same iterates to the FP64 bar of the parity tests (1e-8 of
max |beta|)."""
import numpy as np
import pytest

import flrgen

pytestmark = pytest.mark.gpu
OPTS = dict(inner_tol=1e-12, max_iter=2)


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


def _close(a, b):
    err = np.max(np.abs(a - b)) / np.max(np.abs(b))
    print("  difference %.2g" % err, flush=True)
    assert err <= 1e-8


def _served(flr, ctx, prob, budget):
    srv = flr.flr_server_create(ctx.h, budget, 1)
    t = flr.flr_server_submit(srv, prob.h, 0.3, 0.7, 1e-14, flr.default_opts(**OPTS))
    beta = np.zeros(prob.p)
    st, res = flr.flr_server_poll(srv, t, True, beta)
    flr.flr_server_destroy(srv)
    assert st == flr.FLR_ERR_MAX_ITER  # both MM steps ran
    return beta


@pytest.mark.parametrize("q", [20, 40])  # one segment; segments and separators
def test_budget_of_the_banded_factor_is_enough(flr, ctx, q):
    y = np.random.default_rng(q).standard_normal(q * q)
    prob = flr.Problem.flsa(ctx, y, flrgen.lattice_edges(q))
    base = prob.footprint
    prob.solve(0.3, 0.7, tol=1e-14, preconditioner=flr.FLR_PRECOND_TRIDIAG, max_iter=1)
    assert prob.footprint == base  # another preconditioner takes none of it
    print("q=%d: budget %d" % (q, base), flush=True)
    small = _served(flr, ctx, prob, base)
    assert prob.footprint == base
    solo = prob.solve(0.3, 0.7, tol=1e-14, **OPTS)
    full = prob.footprint
    assert full > base
    _close(small, solo.beta)
    assert np.array_equal(_served(flr, ctx, prob, full), solo.beta)
    assert np.array_equal(_served(flr, ctx, prob, base), small)  # accepted as before, and the memory given back
    assert prob.footprint == base
    again = prob.solve(0.3, 0.7, tol=1e-14, **OPTS)  # taken again, rotation captured again
    assert prob.footprint == full
    assert np.array_equal(again.beta, solo.beta)
    prob.close()


def test_slots_take_and_release_while_others_capture(flr, ctx):
    # four slots at once: fresh handles take the memory, then a small budget makes every one give it back, each
    # while the other slots capture their rotations; results as on a handle alone
    q = 34
    ys = [np.random.default_rng(k).standard_normal(q * q) for k in range(4)]
    probs = [flr.Problem.flsa(ctx, y, flrgen.lattice_edges(q)) for y in ys]
    base = [p.footprint for p in probs]
    o = flr.default_opts(**OPTS)
    got = {}
    for name, budget in (("large", 2 ** 34), ("small", sum(base))):
        srv = flr.flr_server_create(ctx.h, budget, 4)
        tickets = [flr.flr_server_submit(srv, p.h, 0.3, 0.7, 1e-14, o) for p in probs]
        betas = [np.zeros(p.p) for p in probs]
        for t, b in zip(tickets, betas):
            st, res = flr.flr_server_poll(srv, t, True, b)
            assert st == flr.FLR_ERR_MAX_ITER
        flr.flr_server_destroy(srv)
        got[name] = betas
        held = [p.footprint > f for p, f in zip(probs, base)]
        print("  %s budget: inverses held %s" % (name, held), flush=True)
        assert held == [name == "large"] * 4
    for p, big, small in zip(probs, got["large"], got["small"]):
        _close(small, big)
        assert np.array_equal(p.solve(0.3, 0.7, tol=1e-14, **OPTS).beta, big)
        p.close()


def test_solve_where_the_memory_is_not_free(flr, ctx):
    import torch

    p, bw = 200000, 2
    rng = np.random.default_rng(3)
    y = np.repeat(rng.uniform(-2, 2, p // 8), 8) + 0.3 * rng.standard_normal(p)
    j = np.arange(p - 1)
    e = np.concatenate([np.stack([j, j + 1], 1), np.stack([np.arange(p - bw), np.arange(bw, p)], 1)])
    prob = flr.Problem.flsa(ctx, y, e.astype(np.int64))
    base = prob.footprint
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    held = torch.empty(free - 2500 * 2 ** 20, dtype=torch.uint8, device="cuda:0")
    print("p=%d bw=%d: %d MiB left free" % (p, bw, torch.cuda.mem_get_info()[0] >> 20), flush=True)
    tight = prob.solve(0.3, 0.7, tol=1e-14, **OPTS)
    assert prob.footprint == base
    del held
    torch.cuda.empty_cache()
    s = prob.solve(0.3, 0.7, tol=1e-14, **OPTS)
    assert base + 2 ** 29 < prob.footprint < base + 3 * 2 ** 29  # 1184 segments; cut into 128 they took 3.1 GB
    _close(tight.beta, s.beta)
    prob.close()


@pytest.mark.parametrize("n,p", [(1000, 10000), (500, 5000), (200, 1000)])
def test_setup_scratch_is_not_kept(flr, ctx, n, p):
    # X, the vectors, the edges and ONE array of X^T u partials: at most 512 / 40 rows of p where the launch target
    # bounds the row panels (p = 10^4), 512 / 20 at p = 5000, and a panel per four rows anywhere
    X = np.random.default_rng(1).standard_normal((n, p)).astype(np.float32)
    prob = flr.Problem(ctx, X, flr.FLR_F32, np.ones(n), flrgen.chain_edges(p), use_tuned=False)
    pad = (p + 1023) // 1024 * 1024
    parts = min(-(-512 // (pad // 256)), n // 4) * pad * 8
    rest = n * pad * 4 + 16 * pad * 8 + 2 * p * 12 + (pad // 1024 + 1) * n * 8 + 65536
    print("  n=%d p=%d: footprint %d, bound %d" % (n, p, prob.footprint, rest + parts), flush=True)
    assert prob.footprint <= rest + parts
    prob.close()
