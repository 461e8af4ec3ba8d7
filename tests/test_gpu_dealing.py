"""Uneven clusters, whose strips the dies get in lists of different lengths: every strip is run once, for one system and for
several side by side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = {
    "one-large": [1500] + [40] * 30,             # larger than an eighth of the whole: cut
    "fewer-than-dies": [700, 300, 90],
    "one": [130],
    "spread": [int(64 * 1.13 ** k) + k % 3 for k in range(26)],
    "large-and-tiny": [1000] * 7 + [5] * 57,
}


@pytest.mark.parametrize("name", list(SIZES))
def test_products_and_applies_of_uneven_clusters(lib, name):
    import torch
    from paper_2510_12128_amd import binding as B
    sizes = SIZES[name]
    n, t, rank = sum(sizes), 16, 3
    rng = np.random.default_rng(5)
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = (np.repeat(np.arange(len(sizes)), sizes)[:, None] * 4.0 + 0.5 * rng.standard_normal((n, 2))).astype(np.float32)
    y, probes = np.sin(X).sum(1).astype(np.float32), 2.0 * rng.integers(0, 2, (n, t)) - 1.0
    theta = np.array([0.9, 1.1, 1.0, 0.3])
    side, alone = (lib.Context(X, y, off, probes, rank, max_iter=cap) for cap in (1024, 4096))   # (alone: one system at a time)
    for ctx in (side, alone):
        ctx.nugpr_build_blocks(theta)
        assert ctx.nugpr_precond_factor()[0] == 0
    pts = (X[rng.integers(0, n, 4 * (t + 1))] + 0.3).astype(np.float32)
    one, four = alone.nugpr_predict(theta, pts), side.nugpr_predict(theta, pts)
    assert four["code"] == 0 and np.array_equal(np.asarray(one["var"]), np.asarray(four["var"]))
    for T in (1, 17):
        V = torch.as_tensor(rng.standard_normal((n, T)), dtype=torch.float32, device="cuda")
        got = [side.nugpr_matvec(V), side.nugpr_precond_apply(V), side.nugpr_split_apply(V)]
        v = V.double()
        K, Y, W = ([side.nugpr_export(what, i).double() for i in range(len(sizes))] for what in (B.EXPORT_K, B.EXPORT_LINV, B.EXPORT_W))
        C = side.nugpr_export(B.EXPORT_C).double()

        def blocks(f, x):
            return torch.cat([f(i) @ x[off[i]:off[i + 1]] for i in range(len(sizes))])

        def coupled(x):
            P = C @ blocks(lambda i: W[i].T, x)
            return torch.cat([W[i] @ P[i * rank:(i + 1) * rank] for i in range(len(sizes))])

        want = [blocks(lambda i: K[i], v) + coupled(v), blocks(lambda i: Y[i].T, blocks(lambda i: Y[i], v))]
        u = blocks(lambda i: Y[i].T, v)
        want.append(blocks(lambda i: Y[i], blocks(lambda i: K[i], u) + coupled(u)))
        # the result in fp32 and the diagonal's part that its export lacks: 2^-24 each; the relation Y K Y^T = I, which the third uses,
        # holds to the fp32 factor's backward error (cond(K) = 100 at most here)
        for g, w, eps in zip(got, want, (2.0 ** -22, 2.0 ** -22, 1e-4)):
            assert float((g.double() - w).norm() / w.norm()) <= eps
    side.close()
    alone.close()
