"""Clusters so far apart that most of the coupling matrix vanishes in fp32: its products pass over the tiles without a value."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("acc_fp32", [False, True])
def test_products_where_most_of_the_coupling_vanishes(lib, acc_fp32):
    import torch
    from paper_2510_12128_amd import binding as B
    nc, b, rank, t = 40, 130, 128, 32                   # 80 x 80 tiles of coupling, five an item
    n = nc * b
    rng = np.random.default_rng(4)
    off = np.arange(nc + 1) * b
    centres = np.stack([6.0 * (np.arange(nc) % 4), 500.0 * (np.arange(nc) // 4)], 1)
    X = (np.repeat(centres, b, axis=0) + 0.5 * rng.standard_normal((n, 2))).astype(np.float32)
    ctx = lib.Context(X, np.sin(X).sum(1).astype(np.float32), off, 2.0 * rng.integers(0, 2, (n, t)) - 1.0, rank, acc_fp32=acc_fp32)
    Ws = [ctx.nugpr_export(B.EXPORT_W, i).double() for i in range(nc)]
    eps = 60 * 2.0 ** -24 if acc_fp32 else 2.0 ** -23   # as at the edges of the strip kernel's tiles
    # no tile between the groups, all of them, none again: every assembly says anew which tiles hold a value
    for ell, share in ((1.5, (0.001, 0.2)), (400.0, (0.9, 1.0)), (1.5, (0.001, 0.2))):
        ctx.nugpr_build_blocks(np.array([ell, ell, 1.3, 0.2]))
        Vs = [torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda") for T in (1, 17, 33)]
        got = [ctx.nugpr_matvec(V) for V in Vs]
        C = ctx.nugpr_export(B.EXPORT_C).double()
        assert share[0] <= float((C != 0).double().mean()) <= share[1]
        K = [ctx.nugpr_export(B.EXPORT_K, i).double() for i in range(nc)]
        for V, g in zip(Vs, got):
            def product(f, v):
                P = f(C) @ torch.cat([Ws[i].T @ v[off[i]:off[i + 1]] for i in range(nc)])
                return torch.cat([f(K[i]) @ v[off[i]:off[i + 1]] + Ws[i] @ P[i * rank:(i + 1) * rank] for i in range(nc)])
            err = (g.double() - product(lambda a: a, V.double())).abs() / product(torch.abs, V.double().abs())
            assert float(err.max()) <= eps, (ell, V.shape[1])
    ctx.close()


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("acc_fp32", [False, True])
def test_values_that_are_not_finite_reach_every_row(lib, acc_fp32, dense):
    """A NaN or infinity among the vector rows meets every row of the coupling matrix, zeros included: 0 times it is NaN."""
    import torch
    nc, b, rank = 40, 130, 128
    n = nc * b
    rng = np.random.default_rng(4)
    centres = np.stack([6.0 * (np.arange(nc) % 4), 500.0 * (np.arange(nc) // 4)], 1)
    X = (np.repeat(centres, b, axis=0) + 0.5 * rng.standard_normal((n, 2))).astype(np.float32)
    ctx = lib.Context(X, np.zeros(n, np.float32), np.arange(nc + 1) * b, 2.0 * rng.integers(0, 2, (n, 32)) - 1.0, rank, acc_fp32=acc_fp32)
    theta = np.array([1.5, 1.5, 1.3, 0.2])
    ctx.nugpr_build_blocks(theta)
    if dense:
        ctx.nugpr_set_nystrom_basis(theta)
    for T in (1, 2, 17, 33):
        V = torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda")
        clean = ctx.nugpr_matvec(V)
        assert bool(torch.isfinite(clean).all())
        for at, col, bad in ((0, 0, float("nan")), (n - 1, T - 1, float("inf")), (7 * b + 129, T // 2, -float("inf")), (39 * b, T - 1, float("nan"))):
            W = V.clone()
            W[at, col] = bad
            got = ctx.nugpr_matvec(W)
            keep = [c for c in range(T) if c != col]
            assert torch.equal(got[:, keep], clean[:, keep]), (T, at)
            assert not bool(torch.isfinite(got[:, col]).any()), (T, at, int(torch.isfinite(got[:, col]).sum()))
    ctx.close()


def test_training_step_where_most_of_the_coupling_vanishes(lib):
    """Both matrices of a pair assembly against an assembly of their own each: entries differ by a rounding to fp32 (2^-25), whose
    difference over 2 h = 2e-3 is 1.5e-5 of a term of the loss at most."""
    nc, b, rank, t = 40, 130, 128, 16
    n = nc * b
    rng = np.random.default_rng(4)
    centres = np.stack([5.0 * (np.arange(nc) % 4), 500.0 * (np.arange(nc) // 4)], 1)
    X = (np.repeat(centres, b, axis=0) + 0.5 * rng.standard_normal((n, 2))).astype(np.float32)
    probes = 2.0 * rng.integers(0, 2, (n, t)) - 1.0
    phi = np.log(np.array([1.2, 1.3, 1.0, 0.2]))
    grads = []
    for no_shortcuts in (False, True):
        ctx = lib.Context(X, np.sin(X).sum(1).astype(np.float32), np.arange(nc + 1) * b, probes, rank, no_shortcuts=no_shortcuts)
        o = ctx.nugpr_train_step(phi, np.zeros(4), np.zeros(4), 0)
        assert o["code"] == 0
        grads.append(np.asarray(o["grad"]))
        ctx.close()
    assert np.abs(grads[0] - grads[1]).max() <= 1.5e-5 * np.linalg.norm(grads[1])
