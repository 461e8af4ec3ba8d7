"""The strip kernel at the edges of its tiles, item kinds and column groups, against a float64 product of the very
matrices it applies (exported entries), with element-wise rounding bounds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = {
    "one-tile": [64, 64],
    "around-a-tile": [63, 65, 129],
    "tiny": [5, 3, 1],
    "many-tiles": [200, 257, 64, 90, 33, 640],
    "few-representatives": [1700, 900],  # one for each: its points are shared out among up to 16 threads a column
    "wide-coupling": [150] * 11,         # 11 x 65 representatives: row groups of the coupling matrix of unequal size
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
    theta = np.array([1.2, 0.9, 1.5, 1.3, 0.2])
    ctx.nugpr_build_blocks(theta)
    assert ctx.nugpr_precond_factor()[0] == 0
    nc = len(sizes)
    C = ctx.nugpr_export(B.EXPORT_C).double()
    K = [ctx.nugpr_export(B.EXPORT_K, i).double() for i in range(nc)]
    Y = [ctx.nugpr_export(B.EXPORT_LINV, i).double() for i in range(nc)]
    Ws = [ctx.nugpr_export(B.EXPORT_W, i).double() for i in range(nc)]

    def product(f, V):
        S = torch.cat([f(Ws[i]).T @ V[off[i]:off[i + 1]] for i in range(nc)])
        P = f(C) @ S
        return torch.cat([f(K[i]) @ V[off[i]:off[i + 1]] + f(Ws[i]) @ P[i * rank:(i + 1) * rank] for i in range(nc)])

    def apply(f, V):
        return torch.cat([f(Y[i]).T @ (f(Y[i]) @ V[off[i]:off[i + 1]]) for i in range(nc)])

    # fp64 mode: the result is rounded to fp32 once and the exported diagonal lacks what fp32 dropped of it (2^-25 each
    # way).  fp32 mode: chains of 16 terms, each of the (at most three) passes also rounds its result: 20 2^-24 a pass.
    eps = 60 * 2.0 ** -24 if acc_fp32 else 2.0 ** -23
    for T in (1, 2, 9, 16, 17, 18, 33):
        V = torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda")
        for got, ref in ((ctx.nugpr_matvec(V), product), (ctx.nugpr_precond_apply(V), apply)):
            want, bound = ref(lambda a: a, V.double()), ref(torch.abs, V.double().abs())
            worst = float(((got.double() - want).abs() / bound.clamp_min(1e-300)).max())
            assert worst <= eps, (name, dense, acc_fp32, T, ref.__name__, worst)
    ctx.close()
