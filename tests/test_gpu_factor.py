"""The factorisation at the edges of its tiles (64), blocks (128), tree levels and shared sums, against float64 on the exported
matrices: backward error of L, residual of the stored inverse, log det."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = {
    "one-tile": [64, 1, 63],
    "around-a-block": [65, 127, 128, 129, 191, 192, 193],
    "around-a-level": [256, 257, 320, 385, 513, 575],
    # few block rows and many columns: the sums of a block are shared by several workgroups
    "one-long": [2113],
    "long-and-short": [1665, 70, 1024, 3, 1471],
    "uneven-many": [64 * (1 + k % 7) + k for k in range(70)],          # more clusters than lanes look at in one go
    # enough blocks for launches of whole blocks of 128 (test_factor_routes.py): odd and even numbers of tiles, ragged last ones
    "whole-blocks": [513, 575, 641, 769, 833, 1025] * 10,
    "whole-blocks-shared-sums": [1025] * 20 + [1087] * 20 + [1000] * 14 + [513, 70, 1],
}


@pytest.mark.parametrize("name", list(SIZES))
def test_factor_and_inverse_at_block_edges(lib, name):
    import torch
    from paper_2510_12128_amd import binding as B
    sizes = SIZES[name]
    n, d = sum(sizes), 3
    rng = np.random.default_rng(5)
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = rng.standard_normal((n, d)).astype(np.float32)
    ctx = lib.Context(X, rng.standard_normal(n).astype(np.float32), off, 2.0 * rng.integers(0, 2, (n, 2)) - 1.0, 1)
    for theta in (np.array([2.0, 1.4, 0.8, 2.1, 0.3]), np.array([1.2, 0.9, 1.5, 1.3, 0.2])):      # the second time over what the first left
        ctx.nugpr_build_blocks(theta)
        code, logdet, bad = ctx.nugpr_precond_factor()
        assert code == 0 and bad == -1
        want = 0.0
        V = torch.randn(n, 3, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
        Z = ctx.nugpr_precond_apply(V)
        for i, b in enumerate(sizes):
            K = ctx.nugpr_export(B.EXPORT_K, i).double()
            L = ctx.nugpr_export(B.EXPORT_L, i).double()
            Y = ctx.nugpr_export(B.EXPORT_LINV, i).double()
            # element-wise backward error of a Cholesky factorisation of order b: (b + 1) u |L| |L|^T, u = 2^-24; what goes
            # through a block's explicit inverse also meets the condition number of the block's factor, at these theta at most
            # sqrt(1 + 128 alpha / sigma^2) = 31, in both of its uses: 64 u
            u = 2.0 ** -24
            err = (L @ L.T - K).abs() / (L.abs() @ L.abs().T)
            assert float(err.max()) <= (b + 1 + 64) * u, (name, i, float(err.max()) / u)
            # residual of an inverse by blocks, likewise relative to |Y| |L|
            res = (Y @ L - torch.eye(b, device=L.device, dtype=L.dtype)).abs() / (Y.abs() @ L.abs()).clamp_min(1.0)
            assert float(res.max()) <= (b + 1 + 64) * u, (name, i, float(res.max()) / u)
            # the apply takes its second half from the mirror image of Y: fp64 sums over b terms, rounded to fp32
            v = V[off[i]:off[i + 1]].double()
            ref = Y.T @ (Y @ v)
            bound = 2.0 ** -24 * ref.abs() + 2 * b * 2.0 ** -53 * (Y.abs().T @ (Y.abs() @ v.abs()))
            assert float(((Z[off[i]:off[i + 1]].double() - ref).abs() / bound).max()) <= 1.0, (name, i)
            want -= 2.0 * float(torch.log(Y.diagonal()).sum())
        assert abs(logdet - want) <= 1e-12 * n + 1e-10 * abs(want)
    ctx.close()


@pytest.mark.parametrize("alpha,noise", [(2e38, 0.5e38), (1.5e38, 0.3e38), (1e37, 2e36), (1e-36, 2e-37), (4e-38, 1e-38), (3e-38, 0.6e-38)])
def test_factor_at_the_ends_of_the_number_range(lib, alpha, noise):
    """Pivots whose reciprocal is subnormal (above 2^126) or that are subnormal themselves."""
    import torch
    from paper_2510_12128_amd import binding as B
    sizes = [70, 200, 129]
    n = sum(sizes)
    rng = np.random.default_rng(5)
    X = rng.standard_normal((n, 3)).astype(np.float32)
    ctx = lib.Context(X, np.zeros(n, np.float32), np.concatenate([[0], np.cumsum(sizes)]), 2.0 * rng.integers(0, 2, (n, 2)) - 1.0, 1)
    ctx.nugpr_build_blocks(np.array([2.0, 1.4, 0.8, alpha, noise]))
    code, logdet, bad = ctx.nugpr_precond_factor()
    assert code == 0 and bad == -1
    u, unit = 2.0 ** -24, 2.0 ** -149
    for i, b in enumerate(sizes):
        K, L, Y = (ctx.nugpr_export(w, i).double() for w in (B.EXPORT_K, B.EXPORT_L, B.EXPORT_LINV))
        # the bounds of the test above; subnormal entries are rounded to whole units in each of b steps, and the roundings go twice
        # through a block's inverse and factor, whose condition number is at most sqrt(1 + 128 alpha / sigma^2) = 26 here
        LL = L.abs() @ L.abs().T
        assert float(((L @ L.T - K).abs() - 2 * 26 * b * unit).div(LL).max()) <= (b + 1 + 64) * u
        res = (Y @ L - torch.eye(b, device=L.device, dtype=L.dtype)).abs() / (Y.abs() @ L.abs()).clamp_min(1.0)
        assert float(res.max()) <= (b + 1 + 64) * u
    ctx.close()


@pytest.mark.parametrize("scale", [1.0, 1e12, 1e-12])
@pytest.mark.parametrize("name", ["around-a-block", "around-a-level", "long-and-short", "whole-blocks"])
def test_factor_of_blocks_with_a_wide_spread(lib, name, scale):
    """Entries from the scale of the variances down to the smallest that fp32 holds, every one held to its own size."""
    import torch
    from paper_2510_12128_amd import binding as B
    sizes = SIZES[name]
    n, d = sum(sizes), 20
    rng = np.random.default_rng(6)
    X = rng.standard_normal((n, d)).astype(np.float32)
    ctx = lib.Context(X, np.zeros(n, np.float32), np.concatenate([[0], np.cumsum(sizes)]), 2.0 * rng.integers(0, 2, (n, 2)) - 1.0, 1)
    ctx.nugpr_build_blocks(np.array([0.5] * d + [1.0 * scale, 0.1 * scale]))
    assert ctx.nugpr_precond_factor()[0] == 0
    u, unit = 2.0 ** -24, 2.0 ** -149
    low = 0
    for i, b in enumerate(sizes):
        K, L, Y = (ctx.nugpr_export(w, i).double() for w in (B.EXPORT_K, B.EXPORT_L, B.EXPORT_LINV))
        low += int(((K > 2.0 ** -126 * scale) & (K < 2.0 ** -100 * scale)).sum())
        # element by element: (b + 1) u |L| |L|^T and what the explicit inverses of 128 x 128 blocks add (condition number below 4 at this
        # spread: 64 u is more than enough); subnormal entries and intermediates are off by whole units in each of b steps, which
        # meet entries of L or Y of up to max(1, s), s = sqrt(alpha + sigma^2) or 1 / sigma
        LL = L.abs() @ L.abs().T
        big = 4.0 * b * unit * max(1.0, float(L.abs().max()), float(Y.abs().max())) ** 2
        assert float(((L @ L.T - K).abs() - big).div(LL + unit).max()) <= (b + 1 + 64) * u, (name, i)
        # the inverse: Y21 = -Y22 (L21 Y11), each product off by b u of its terms' magnitudes, so Y L by that of |Y| |L| |Y| |L|
        G = Y.abs() @ L.abs()
        res = (Y @ L - torch.eye(b, device=L.device, dtype=L.dtype)).abs()
        assert float((res - big).div(G @ G + unit).max()) <= (b + 1 + 64) * u, (name, i)
    assert low > 1000
    ctx.close()
