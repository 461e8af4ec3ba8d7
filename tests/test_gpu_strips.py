"""The strip kernel at the edges of its tiles, item kinds and column groups, against a float64 product of the very
matrices it applies (exported entries), with element-wise rounding bounds.  The products run before the export that fills
in the tiles above the diagonals, over blocks whose upper tiles still hold another theta's values: a strip that read one
would be off by far more than rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = {
    "one-tile": [64, 64],
    "around-a-tile": [63, 65, 129],
    "tiny": [5, 3, 1],
    "many-tiles": [200, 257, 64, 90, 33, 640],
    # one for each: its points are shared out among many threads (16 a column at 33 columns, 256 at one)
    "few-representatives": [1700, 900],
    "wide-coupling": [150] * 11,         # 11 x 65 representatives: row groups of the coupling matrix of unequal size
    "many-short": [90 + k % 60 for k in range(240)],  # more than 512 strips of few tiles
    "long-strips": [1900, 1610],         # more than 10 tiles a strip on average
    "long-streamed": [4800, 4730],       # the same, and more than 128 MB of K_ii
    "short-streamed": [500 + k % 13 for k in range(130)],  # more than 128 MB in strips of few tiles
}


@pytest.mark.parametrize("acc_fp32", [False, True])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("name", list(SIZES))
def test_products_and_applies_at_tile_edges(lib, name, dense, acc_fp32):
    import torch
    from paper_2510_12128_amd import binding as B
    sizes = SIZES[name]
    rank = {"tiny": 1, "few-representatives": 1, "wide-coupling": 65}.get(name, 7)
    n, d, t = sum(sizes), 3, 32
    rng = np.random.default_rng(11)
    off = np.concatenate([[0], np.cumsum(sizes)])
    centre = np.repeat(np.arange(len(sizes)), sizes)[:, None] * 3.0
    X = (centre + rng.standard_normal((n, d))).astype(np.float32)
    W = rng.standard_normal((n, rank)).astype(np.float32) if dense else None
    ctx = lib.Context(X, rng.standard_normal(n).astype(np.float32), off, 2.0 * rng.integers(0, 2, (n, t)) - 1.0, rank,
                      W=W, acc_fp32=acc_fp32)
    nc = len(sizes)
    ctx.nugpr_build_blocks(np.array([2.0, 1.4, 0.8, 2.1, 0.3]))
    ctx.nugpr_export(B.EXPORT_C)                                # these fill in the upper tiles
    ctx.nugpr_export(B.EXPORT_K, 0)
    ctx.nugpr_build_blocks(np.array([1.2, 0.9, 1.5, 1.3, 0.2]))
    assert ctx.nugpr_precond_factor()[0] == 0
    runs = []
    for T in (1, 2, 9, 16, 17, 18, 33):
        V = torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda")
        runs.append((T, V, ctx.nugpr_matvec(V), ctx.nugpr_precond_apply(V)))
    C = ctx.nugpr_export(B.EXPORT_C).double()

    def blocks(what):
        return (ctx.nugpr_export(what, i).double() for i in range(nc))

    Ws = list(blocks(B.EXPORT_W))

    def coupled(f, V):
        S = torch.cat([f(Ws[i]).T @ V[off[i]:off[i + 1]] for i in range(nc)])
        P = f(C) @ S
        return torch.cat([f(Ws[i]) @ P[i * rank:(i + 1) * rank] for i in range(nc)])

    # fp64 mode: the result is rounded to fp32 once and the exported diagonal lacks what fp32 dropped of it (2^-25 each
    # way).  fp32 mode: chains of 16 terms, each of the (at most three) passes also rounds its result: 20 2^-24 a pass.
    eps = 60 * 2.0 ** -24 if acc_fp32 else 2.0 ** -23
    product = [(coupled(lambda a: a, V.double()), coupled(torch.abs, V.double().abs())) for _, V, _, _ in runs]
    for what, which in ((B.EXPORT_K, 2), (B.EXPORT_LINV, 3)):
        worst = [0.0] * len(runs)
        for i, M in enumerate(blocks(what)):
            for k, run in enumerate(runs):
                rows = slice(off[i], off[i + 1])
                v = run[1][rows].double()
                if which == 2:
                    want, bound = M @ v + product[k][0][rows], M.abs() @ v.abs() + product[k][1][rows]
                else:
                    want, bound = M.T @ (M @ v), M.abs().T @ (M.abs() @ v.abs())
                err = (run[which][rows].double() - want).abs() / bound.clamp_min(1e-300)
                worst[k] = max(worst[k], float(err.max()))
        assert max(worst) <= eps, (name, dense, acc_fp32, what, [(r[0], w) for r, w in zip(runs, worst)])
    ctx.close()
