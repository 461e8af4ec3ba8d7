"""Products and applies of 18 to 33 columns on many strips (fp64 mode), component by component against float64 products of the
exported matrices: every entry is held to its own size, whatever stands beside it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# 828 strips, 16.9 tiles each on average in their triangles; and 700 short ones
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
def test_products_and_applies_of_many_columns(lib, name):
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
    # Matrices are stored in fp32 and meet the vectors in fp64: what is left is the rounding of the result to fp32, the sums in fp64
    # (2113 terms and two passes at most: 2^-40 of the terms' magnitudes), and what the exported diagonal lacks (up to 2^-25 of itself).
    for V, Q, Z in runs:
        v = V.double()
        S = torch.cat([Ws[i].T @ v[off[i]:off[i + 1]] for i in range(len(sizes))])
        P, dP = C @ S, C.abs() @ S.abs()
        for i in (0, 1, len(sizes) - 3, len(sizes) - 2, len(sizes) - 1):
            rows, r = slice(off[i], off[i + 1]), slice(i * rank, (i + 1) * rank)
            K, Y = ctx.nugpr_export(B.EXPORT_K, i).double(), ctx.nugpr_export(B.EXPORT_LINV, i).double()
            want = K @ v[rows] + Ws[i] @ P[r]
            limit = 2.0 ** -24 * (want.abs() + K.diagonal()[:, None] * v[rows].abs()) + 2.0 ** -40 * (K.abs() @ v[rows].abs() + Ws[i] @ dP[r])
            assert float(((Q[rows].double() - want).abs() - limit).max()) <= 0.0, (name, V.shape[1], i)
            u = Y @ v[rows]
            want = Y.T @ u
            limit = 2.0 ** -24 * want.abs() + 2.0 ** -40 * (Y.abs().T @ (Y.abs() @ v[rows].abs()))
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


@pytest.mark.parametrize("T", [17, 18, 33])
def test_columns_of_the_operator_and_values_of_every_size(lib, T):
    """Unit vectors give the columns of K' to the bit, however small an entry is beside its neighbours; and rows far from a value
    that is a billion times the others keep their own."""
    import torch
    from paper_2510_12128_amd import binding as B
    sizes = SIZES["long"]
    ctx, off, rng = _context(lib, sizes)
    n, i = off[-1], 2
    rows = slice(off[i], off[i + 1])
    K, Y = ctx.nugpr_export(B.EXPORT_K, i).double(), ctx.nugpr_export(B.EXPORT_LINV, i).double()
    at = torch.as_tensor(rng.choice(sizes[i], T, replace=False), device="cuda")
    E = torch.zeros(n, T, device="cuda")
    E[off[i] + at, torch.arange(T, device="cuda")] = 1.0
    Q, Z = ctx.nugpr_matvec(E)[rows].double(), ctx.nugpr_precond_apply(E)[rows].double()
    other = torch.ones_like(Q, dtype=torch.bool)
    other[at, torch.arange(T, device="cuda")] = False                # (the exported diagonal is rounded)
    assert torch.equal(Q[other], K[:, at][other])
    e = E[rows].double()
    limit = 2.0 ** -24 * (Y.T @ (Y @ e)).abs() + 2.0 ** -40 * (Y.abs().T @ (Y.abs() @ e))
    assert float(((Z - Y.T @ (Y @ e)).abs() - limit).max()) <= 0.0
    V = torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda")
    V[off[i] + at, torch.arange(T, device="cuda")] *= 1e9
    Q = ctx.nugpr_matvec(V)[rows].double()
    C, Ws = ctx.nugpr_export(B.EXPORT_C).double(), [ctx.nugpr_export(B.EXPORT_W, k).double() for k in range(len(sizes))]
    S = torch.cat([Ws[k].T @ V[off[k]:off[k + 1]].double() for k in range(len(sizes))])
    v, r = V[rows].double(), slice(i * 5, i * 5 + 5)
    want = K @ v + Ws[i] @ (C[r] @ S)
    limit = 2.0 ** -24 * (want.abs() + K.diagonal()[:, None] * v.abs()) + 2.0 ** -40 * (K.abs() @ v.abs() + Ws[i] @ (C[r].abs() @ S.abs()))
    assert float(((Q - want).abs() - limit).max()) <= 0.0
    ctx.close()


def test_static_product_beside_products_and_applies_of_the_same_context(lib):
    """The product with scratch of its own overlaps calls that use the context's workspace, on another stream."""
    import torch
    ctx, off, rng = _context(lib, [2048] * 26, rank=1)               # 832 strips of 16.5 tiles, and small enough for the static buffer
    n, T = off[-1], 18
    V, W = (torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda") for _ in range(2))
    want = [ctx.nugpr_matvec(V), ctx.nugpr_matvec(W), ctx.nugpr_precond_apply(W)]
    assert torch.equal(ctx.nugpr_matvec_static(V), want[0])
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = [[], [], []]
    for _ in range(8):
        with torch.cuda.stream(side):
            got[0].append(ctx.nugpr_matvec_static(V))
        got[1].append(ctx.nugpr_matvec(W))
        got[2].append(ctx.nugpr_precond_apply(W))
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert all(torch.equal(x, w) for x in g)
    ctx.close()
