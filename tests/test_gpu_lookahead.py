"""Solves whose iterations are issued ahead of the stop test: after three solves of one kind and width the host no longer
waits for each test, so a solve that then ends sooner must give what it gives on a fresh context, to the bit, and count the
same iterations, products and preconditioner applies."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [64, 130, 97, 200, 71]            # the last cluster lies far from the others
STATS = ("pcg_solves", "pcg_iterations", "products", "products_reused", "precond_applies")


def _problem(lib, acc_fp32, tol=1e-4):
    rng = np.random.default_rng(5)
    off = np.concatenate([[0], np.cumsum(SIZES)])
    centres = np.array([[0.0, 0.0], [3.2, 0.0], [0.0, 3.2], [3.2, 3.2], [500.0, 500.0]])
    X = (np.repeat(centres, SIZES, axis=0) + 0.4 * rng.standard_normal((off[-1], 2))).astype(np.float32)
    y = rng.standard_normal(off[-1]).astype(np.float32)
    probes = 2.0 * rng.integers(0, 2, (off[-1], 8)) - 1.0

    def fresh():
        ctx = lib.Context(X, y, off, probes, 4, tol=tol, max_iter=200, acc_fp32=acc_fp32)
        ctx.nugpr_build_blocks(np.array([1.0, 1.0, 1.0, 1.0]))
        assert ctx.nugpr_precond_factor()[0] == 0
        return ctx
    return fresh, off, rng


@pytest.mark.parametrize("acc_fp32", [False, True])
@pytest.mark.parametrize("then", ["zero", "isolated", "one-live-column", "indefinite"])
@pytest.mark.parametrize("ncols", [1, 9])
def test_a_solve_that_ends_sooner_than_the_last_three(lib, ncols, then, acc_fp32):
    import torch
    from paper_2510_12128_amd import binding as B
    fresh, off, rng = _problem(lib, acc_fp32)
    n = int(off[-1])
    hard = [rng.standard_normal((n, ncols)).astype(np.float32) for _ in range(3)]
    b = rng.standard_normal((n, ncols)).astype(np.float32)
    if then == "zero":
        b[:] = 0.0
    elif then == "isolated":
        b[:off[-2]] = 0.0                # the preconditioner is this cluster's own inverse: one iteration
    elif then == "one-live-column":
        b[:off[-2], :max(1, ncols - 1)] = 0.0        # all but the last column are frozen early (the only one: isolated)
    theta = np.array([1.0, 1.0, 1.0, 0.1])          # too little noise for these clusters: K' is indefinite

    def last(ctx):
        if then == "indefinite":
            ctx.nugpr_build_blocks(theta)
        before = ctx.nugpr_stats_read()
        out = ctx.nugpr_pcg_solve(b)
        after = ctx.nugpr_stats_read()
        return out, {k: after[k] - before[k] for k in STATS}

    ctx = fresh()
    steps = []
    for h in hard:
        code, _, iters, _, _ = ctx.nugpr_pcg_solve(h)
        assert code == 0
        steps.append(iters.max())
    assert min(steps) >= 4
    got, counts = last(ctx)
    twice, _ = last(ctx)
    ref_ctx = fresh()
    want, ref_counts = last(ref_ctx)
    if then == "indefinite":
        assert want[0] == B.NUGPR_INDEFINITE
    elif then != "one-live-column" or ncols == 1:
        assert want[0] == 0 and ref_counts["pcg_iterations"] <= 2
    assert counts == ref_counts, (counts, ref_counts)
    for out in (got, twice):
        assert out[0] == want[0]
        assert torch.equal(out[1], want[1])
        for k in (2, 3, 4):
            assert np.array_equal(out[k], want[k]), k
    ctx.close()
    ref_ctx.close()
