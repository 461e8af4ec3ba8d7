"""Solves side by side (both sides of a central difference; blocks of test points) against one after the other: the same results
to the bit and the same counts.  A context whose iteration cap leaves room for one system's logs only takes them one after the
other."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ALONE, SHARE = 4096, 1024            # iteration caps: one system at a time; the largest with four side by side
STATS = ("loss_evals", "pcg_solves", "pcg_iterations", "pcg_iterations_max", "products", "products_reused", "precond_applies", "assembly_passes",
         "matrices_assembled", "factorisations")


def _contexts(lib, sizes, t, caps, acc_fp32, iso, spacing=4.0):
    rng = np.random.default_rng(3)
    off = np.concatenate([[0], np.cumsum(sizes)])
    d = 2
    centres = np.stack([spacing * (np.arange(len(sizes)) % 3), spacing * (np.arange(len(sizes)) // 3)], 1)
    X = (np.repeat(centres, sizes, axis=0) + 0.5 * rng.standard_normal((off[-1], d))).astype(np.float32)
    y = np.sin(X).sum(1).astype(np.float32)
    probes = 2.0 * rng.integers(0, 2, (off[-1], t)) - 1.0 if t else None
    return X, [lib.Context(X, y, off, probes, 3, tol=1e-6, max_iter=cap, acc_fp32=acc_fp32, isotropic=iso) for cap in caps]


@pytest.mark.parametrize("acc_fp32", [False, True])
@pytest.mark.parametrize("name,sizes,t,iso,spacing", [
    ("one-cluster", [70], 4, False, 4.0),
    ("ragged", [64, 130, 97, 3, 200, 71], 8, False, 4.0),
    ("ragged-iso-33", [64, 130, 97, 65], 32, True, 3.0),
    ("close", [128, 129, 127], 16, False, 3.8),          # several iterations, the sides of a difference need not take as many
    ("largest", [1024] * 32, 4, False, 7.0),             # 32768 points
])
def test_training_step_side_by_side(lib, name, sizes, t, iso, spacing, acc_fp32):
    _, (alone, over, four) = _contexts(lib, sizes, t, (ALONE, SHARE + 1, SHARE), acc_fp32, iso, spacing)
    phi = np.log(np.array([0.9, 1.0, 0.3] if iso else [0.9, 1.1, 1.0, 0.3]))
    zero = np.zeros_like(phi)
    runs = []
    for ctx in (alone, over, four):
        outs = []
        p, m, v = phi, zero, zero
        for k in range(3):                                # Adam moves on: from the second step the solver issues iterations ahead
            ctx.nugpr_stats_read(reset=True)
            o = ctx.nugpr_train_step(p, m, v, k)
            p, m, v = o["log_theta"], o["adam_m"], o["adam_v"]
            outs.append((o["code"], o["nll0"], o["grad"].tolist(), p.tolist(), {k: x for k, x in ctx.nugpr_stats_read().items() if k in STATS}))
        V = np.random.default_rng(1).standard_normal((sum(sizes), 3)).astype(np.float32)
        outs.append(ctx.nugpr_matvec(V).cpu().numpy().tolist())          # the blocks that are in force afterwards
        runs.append(outs)
    assert runs[0][0][0] == 0
    assert runs[1] == runs[0]
    assert runs[2] == runs[0]
    for ctx in (alone, over, four):
        ctx.close()


def test_timed_launches_count_systems(lib):
    """The timing of the product launch counts a launch once for every system it serves, so that time over launches is that of a
    product.  With a cap of one iteration no product is issued in vain."""
    _, (ctx,) = _contexts(lib, [64, 130, 97], 4, (1,), False, False, 30.0)
    phi = np.log(np.array([0.9, 1.1, 1.0, 0.3]))
    ctx.nugpr_profile_enable(True)
    ctx.nugpr_stats_read(reset=True)
    ctx.nugpr_train_step(phi, np.zeros(4), np.zeros(4), 0)
    ms, launches = ctx.nugpr_profile_read()
    stats = ctx.nugpr_stats_read()
    assert stats["loss_evals"] == 9 and ms > 0
    assert launches == stats["products"] == 5              # the base loss; two for each lengthscale (the others reuse its product)
    ctx.close()


@pytest.mark.parametrize("acc_fp32", [False, True])
@pytest.mark.parametrize("sizes,t,spacing", [([64, 130, 97, 3, 200, 71], 4, 4.0), ([128, 129, 127], 16, 3.8)])
def test_prediction_side_by_side(lib, sizes, t, spacing, acc_fp32):
    X, (alone, over, four) = _contexts(lib, sizes, t, (ALONE, SHARE + 1, SHARE), acc_fp32, False, spacing)
    theta = np.array([0.9, 1.1, 1.0, 0.3])
    T = t + 1
    rng = np.random.default_rng(7)
    ctxs = (alone, over, four)
    for ctx in ctxs:
        ctx.nugpr_build_blocks(theta)
        assert ctx.nugpr_precond_factor()[0] == 0
    for m in (1, T, T + 1, 2 * T, 3 * T - 1, 4 * T, 5 * T + 2, 7 * T):
        pts = (X[rng.integers(0, len(X), m)] + 0.3 * rng.standard_normal((m, 2))).astype(np.float32)
        pts[::5] += 1e4                                   # out of reach of everything: zero right-hand sides
        for var in (True, False):
            for ctx in ctxs:
                ctx.nugpr_stats_read(reset=True)
            outs = [ctx.nugpr_predict(theta, pts, variance=var) for ctx in ctxs]
            assert outs[0]["code"] == 0
            counts = [{k: x for k, x in ctx.nugpr_stats_read().items() if k in STATS} for ctx in ctxs]
            assert counts[0]["pcg_solves"] == 1 + (-(-m // T) if var else 0)
            assert counts[1] == counts[0] and counts[2] == counts[0], m
            for o in outs[1:]:
                assert o["code"] == 0
                assert np.array_equal(np.asarray(o["mean"]), np.asarray(outs[0]["mean"]))
                if var:
                    assert np.array_equal(np.asarray(o["var"]), np.asarray(outs[0]["var"]))
    for ctx in ctxs:
        ctx.close()


@pytest.mark.parametrize("at", [0, 7, 10, 19, 29])
def test_prediction_up_to_the_block_with_a_bad_point(lib, at):
    """A test point that is not a number ends a prediction at its block: the blocks ahead of it have been written, in the same
    set of launches or not."""
    from paper_2510_12128_amd import binding as B
    X, ctxs = _contexts(lib, [64, 130, 97, 3, 200, 71], 4, (ALONE, SHARE), False, False)
    theta = np.array([0.9, 1.1, 1.0, 0.3])
    T = 5
    rng = np.random.default_rng(7)
    pts = (X[rng.integers(0, len(X), 6 * T)] + 0.3 * rng.standard_normal((6 * T, 2))).astype(np.float32)
    outs = []
    for ctx in ctxs:
        ctx.nugpr_build_blocks(theta)
        assert ctx.nugpr_precond_factor()[0] == 0
        good = ctx.nugpr_predict(theta, pts)
        bad = pts.copy()
        bad[at] = np.nan
        o = ctx.nugpr_predict(theta, bad)
        assert good["code"] == 0 and o["code"] == B.NUGPR_NOT_FINITE
        ahead = at // T * T
        for k in ("mean", "var"):
            assert np.array_equal(o[k][:ahead], good[k][:ahead])
            assert not o[k][ahead:].any()
        outs.append(o)
        ctx.close()
    for k in ("mean", "var"):
        assert np.array_equal(outs[0][k], outs[1][k])


@pytest.mark.parametrize("acc_fp32", [False, True])
@pytest.mark.parametrize("sizes,spacing", [([1000] * 24, 5.5), ([1024] * 16, 5.0), ([300] * 40, 5.0)], ids=["24x1000", "16x1024", "40x300"])
def test_two_column_groups_side_by_side(lib, sizes, spacing, acc_fp32):
    """33 columns, two column groups, and as many triangular strips as make one system alone and several side by side take
    different instantiations of the strip kernel."""
    X, ctxs = _contexts(lib, sizes, 32, (ALONE, SHARE), acc_fp32, False, spacing)
    theta = np.array([0.9, 1.1, 1.0, 0.3])
    rng = np.random.default_rng(9)
    pts = (X[rng.integers(0, len(X), 6 * 33)] + 0.3 * rng.standard_normal((6 * 33, 2))).astype(np.float32)
    outs = []
    for ctx in ctxs:
        step = ctx.nugpr_train_step(np.log(theta), np.zeros(4), np.zeros(4), 0)
        post = ctx.nugpr_predict(theta, pts)
        assert step["code"] == 0 and post["code"] == 0 and post["max_iters_used"] >= 3
        outs.append((step["nll0"], step["grad"].tolist(), post["mean"].tolist(), post["var"].tolist()))
        ctx.close()
    assert outs[0] == outs[1]


@pytest.mark.parametrize("t", [0, 4, 32])
def test_workspace_for_one_system(lib, monkeypatch, t):
    """Less workspace, by the three more sets of seven vector blocks: the same results, one system at a time; less than that is
    refused."""
    from paper_2510_12128_amd import binding as B
    sizes = [64, 130, 97, 3, 200, 71]
    n = sum(sizes)
    whole = B.load_library()
    less, whole_bytes = [0], 0

    class Smaller:
        def __getattr__(self, name):
            return getattr(whole, name)

        def nugpr_workspace_bytes(self, problem):
            nonlocal whole_bytes
            whole_bytes = whole.nugpr_workspace_bytes(problem)
            return whole_bytes - less[0]

    monkeypatch.setattr(B, "load_library", lambda: Smaller())
    phi = np.log(np.array([0.9, 1.1, 1.0, 0.3]))
    outs = []
    for less[0] in (0, 3 * 7 * 8 * n * (t + 1)):
        X, (ctx,) = _contexts(lib, sizes, t, (SHARE,), False, False)
        o = ctx.nugpr_train_step(phi, np.zeros(4), np.zeros(4), 0)
        p = ctx.nugpr_predict(np.exp(phi), X[:5 * (t + 1)])
        assert o["code"] == 0 and p["code"] == 0
        outs.append((o["nll0"], o["grad"].tolist(), p["mean"].tolist(), p["var"].tolist()))
        ctx.close()
    assert outs[0] == outs[1]
    less[0] = whole_bytes - 4 * sum((64 * (-(-b // 64))) ** 2 for b in sizes)          # room for one of the matrices
    with pytest.raises(B.NugprError):
        _contexts(lib, sizes, t, (SHARE,), False, False)
