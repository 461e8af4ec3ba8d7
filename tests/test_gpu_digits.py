"""Products and applies that take the integer matrix cores (fp64 mode, more than 17 columns, many strips), against float64
products of the exported matrices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# 802 strips, 17 and more tiles each on average in their triangles; and short ones, whose triangles keep the fp64 instructions
SIZES = {"long": [2112] * 24 + [2049, 70, 5], "short": [64, 65, 200, 130] * 70}


def _context(lib, sizes, rank=5):
    n, t = sum(sizes), 32
    rng = np.random.default_rng(21)
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = (np.repeat(np.arange(len(sizes)), sizes)[:, None] * 2.5 + rng.standard_normal((n, 3))).astype(np.float32)
    ctx = lib.Context(X, np.zeros(n, np.float32), off, 2.0 * rng.integers(0, 2, (n, t)) - 1.0, rank)
    ctx.nugpr_build_blocks(np.array([1.5, 1.1, 0.9, 1.3, 0.2]))
    assert ctx.nugpr_precond_factor()[0] == 0
    return ctx, off, rng


@pytest.mark.parametrize("name", list(SIZES))
def test_products_and_applies_in_digits(lib, name):
    import torch
    from paper_2510_12128_amd import binding as B
    sizes, rank = SIZES[name], 5
    ctx, off, rng = _context(lib, sizes, rank)
    n = off[-1]
    runs = []
    for T in (18, 32, 33):
        V = torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda")
        V[::3] *= 1e-4                                              # small values beside large ones
        V[:, T - 1] = 0.0
        runs.append((V, ctx.nugpr_matvec(V), ctx.nugpr_precond_apply(V)))
    C = ctx.nugpr_export(B.EXPORT_C).double()
    Ws = [ctx.nugpr_export(B.EXPORT_W, i).double() for i in range(len(sizes))]
    # A row of products is off by half a unit of 2^-30 of its largest entry for each of its entries (2^-31, largest below 2^31) times the
    # vector's values, and by 2^-39 of the vector's largest for each entry; places that are left out come to less.  Then the result
    # is rounded to fp32, and the exported diagonal lacks up to 2^-25 of itself.
    def bound(M, v):
        A, x = M.abs(), v.abs()
        return 2.0 ** -30 * A.max(1, keepdim=True).values * x.sum(0) + 2.0 ** -37 * A.sum(1, keepdim=True) * x.max(0).values

    for V, Q, Z in runs:
        v = V.double()
        S = torch.cat([Ws[i].T @ v[off[i]:off[i + 1]] for i in range(len(sizes))])
        P, dP = C @ S, bound(C, S)
        for i in (0, 1, len(sizes) - 3, len(sizes) - 2, len(sizes) - 1):
            rows, r = slice(off[i], off[i + 1]), slice(i * rank, (i + 1) * rank)
            K, Y = ctx.nugpr_export(B.EXPORT_K, i).double(), ctx.nugpr_export(B.EXPORT_LINV, i).double()
            want = K @ v[rows] + Ws[i] @ P[r]
            off_diagonal = K - torch.diag(K.diagonal())
            limit = bound(off_diagonal, v[rows]) + Ws[i] @ dP[r] + 2.0 ** -24 * want.abs() + 2.0 ** -24 * K.diagonal()[:, None] * v[rows].abs()
            assert float(((Q[rows].double() - want).abs() - limit).max()) <= 0.0, (name, V.shape[1], i)
            u = Y @ v[rows]
            want = Y.T @ u
            limit = bound(Y.T, u) + Y.abs().T @ bound(Y, v[rows]) + 2.0 ** -24 * want.abs() + 1e-14 * (Y.abs().T @ u.abs())
            assert float(((Z[rows].double() - want).abs() - limit).max()) <= 0.0, (name, V.shape[1], i)
        assert bool((Q[:, -1] == 0).all()) and bool((Z[:, -1] == 0).all())
    ctx.close()


def test_scales_and_values_that_are_not_finite(lib):
    """Powers of two pass exactly, and a NaN or infinity stays in its column."""
    import torch
    ctx, off, rng = _context(lib, SIZES["long"])
    V = torch.as_tensor(rng.standard_normal((off[-1], 33)), dtype=torch.float32, device="cuda")
    scale = torch.as_tensor(2.0 ** rng.integers(-60, 60, 33), dtype=torch.float32, device="cuda")
    for f in (ctx.nugpr_matvec, ctx.nugpr_precond_apply):
        clean = f(V)
        assert torch.equal(f(V), clean)
        assert torch.equal(f(V * scale), clean * scale)
        for bad in (float("nan"), float("inf")):
            W = V.clone()
            W[off[3] + 7, 0] = bad
            W[off[4], 20] = bad
            got = f(W)
            for col, cluster in ((0, 3), (20, 4)):
                assert not bool(torch.isfinite(got[off[cluster]:off[cluster + 1], col]).any())
            keep = [c for c in range(33) if c not in (0, 20)]
            assert torch.equal(got[:, keep], clean[:, keep])
    ctx.close()
