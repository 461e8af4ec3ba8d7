"""GPU parity: every step of the HIP path against the fp64 CPU oracle, element by
element on the same seeded inputs, called through the C ABI (ctypes binding).

Tolerances (the spec bar is 1e-4 relative on solves, loss and gradients):
  assembled entries       2e-6 relative + 1e-7 absolute (fp32 storage of an fp64 value;
                          the exponent argument carries ~|arg| * 6e-8 relative error)
  products / applies      1e-5 of the output's max norm (fp32 accumulation over <= 4096 terms)
  solves, loss, gradient  1e-4 relative, as stated.
"""
import numpy as np
import pytest

from oracle import nugpr_oracle as O
from paper_2510_12128_amd import inputs as I
from paper_2510_12128_amd import binding as B
from conftest import record_metric

pytestmark = pytest.mark.gpu


def make_ctx(lib, w, **kw):
    return lib.Context(w.X, w.y, w.offsets, w.probes, w.rank, tol=kw.pop("tol", w.tol),
                       max_iter=kw.pop("max_iter", w.max_iter), isotropic=w.isotropic, **kw)


def small_ragged(seed=3, t=8, **kw):
    # several tiles per cluster, ragged tails (sizes not multiples of 64), three RHS widths
    args = dict(n_clusters=4, sizes=[200, 70, 129, 64], d=3, rank=8, t=t, seed=seed, ell=1.5,
                spacing=4.5, sigma_blob=0.3, tol=1e-6, max_iter=100)
    args.update(kw)
    return I.make_small(**args)


CASES = {
    "ragged-t8": lambda: small_ragged(t=8),
    "ragged-t16": lambda: small_ragged(seed=4, t=16),
    "ragged-t32": lambda: small_ragged(seed=5, t=32, sizes=[300, 65, 257], spacing=6.5),
    # cluster sizes whose last 64-column tile is more than half full, exactly half full, and one column wide:
    # the strips of a diagonal block walk their tiles in a rotating order and read the upper ones transposed
    "ragged-halves": lambda: small_ragged(seed=6, t=16, sizes=[104, 242, 160, 321], spacing=6.0),
    # 17 x 128 representatives: the coupling matrix has 34 tile rows in 12 groups (eleven of 3, one of 1), so
    # its strips pair up over super-blocks of unequal size, rotate through several tiles, and four column
    # slabs stay empty
    "many-reps": lambda: I.make_small(n_clusters=17, sizes=[130 + (7 * i) % 23 for i in range(17)], d=3, rank=128,
                                      t=16, seed=9, ell=1.5, spacing=7.0, sigma_blob=0.5, tol=1e-6, max_iter=100),
    "tiny": lambda: I.make_small(n_clusters=3, sizes=[8, 12, 5], d=2, rank=2, t=4, seed=7, ell=1.5,
                                 spacing=3.5, sigma_blob=0.3, tol=1e-6, max_iter=50),
    "iso-d1": lambda: I.make_small(n_clusters=2, sizes=[90, 40], d=1, rank=3, t=3, seed=8, ell=0.8,
                                   spacing=4.0, sigma_blob=0.4, isotropic=True, tol=1e-6, max_iter=50),
    "C1": lambda: I.make_config("C1"),
    "C1-wide": lambda: I.make_config("C1", "wide"),
}


def oracle_problem(w):
    return O.Problem(w.X, w.y, w.offsets, w.probes, w.rank)


def relmax(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


@pytest.mark.parametrize("case", ["ragged-t8", "many-reps", "tiny", "iso-d1", "C1-wide"])
def test_build_blocks_matches_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    # theta-independent pieces: bit-exact (integer decisions / copies)
    reps = ctx.nugpr_export(B.EXPORT_REPS).cpu().numpy()
    assert np.array_equal(reps.astype(np.float64), prob.reps)
    for i in range(w.n_clusters):
        Wi = ctx.nugpr_export(B.EXPORT_W, i).cpu().numpy()
        assert np.array_equal(Wi.astype(np.float64), prob.Ws[i]), f"W of cluster {i}"
    ctx.nugpr_build_blocks(w.theta)
    blocks, Cm = prob.assemble(w.theta)
    for i in range(w.n_clusters):
        Ki = ctx.nugpr_export(B.EXPORT_K, i).cpu().numpy().astype(np.float64)
        np.testing.assert_allclose(Ki, blocks[i], rtol=2e-6, atol=1e-7)
        assert np.array_equal(Ki, Ki.T)
    Cg = ctx.nugpr_export(B.EXPORT_C).cpu().numpy().astype(np.float64)
    r = w.rank
    Coff = Cm.copy()
    for i in range(w.n_clusters):
        Coff[i * r:(i + 1) * r, i * r:(i + 1) * r] = 0.0
    np.testing.assert_allclose(Cg, Coff, rtol=2e-6, atol=1e-7)
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t16", "ragged-t32", "ragged-halves", "many-reps", "tiny", "iso-d1",
                                  "C1-wide"])
def test_matvec_matches_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    op = prob.operator(w.theta)
    rng = np.random.default_rng(11)
    for ncols in sorted({1, 2, w.n_probes + 1}):
        D = rng.standard_normal((w.n, ncols)).astype(np.float32)
        Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
        ref = op(D.astype(np.float64))
        assert relmax(Q, ref) < 1e-5, (ncols, relmax(Q, ref))
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-halves", "many-reps"])
def test_upper_tiles_are_left_out_by_products_and_filled_in_for_the_export(lib, case):
    """The assembly leaves out the upper tiles of the K_ii (and of the coupling matrix, when its strips pair up): the
    products of every width read the lower ones only, right after the first assembly and over the upper tiles that an
    export of the blocks before has left, and the export must see the full blocks after every assembly."""
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    rng = np.random.default_rng(12)
    for scale in (1.0, 1.3):
        theta = w.theta.copy()
        theta[:-2] *= scale
        ctx.nugpr_build_blocks(theta)
        op = prob.operator(theta)
        for ncols in (w.n_probes + 1, 1, 2):              # matrix cores and vector ALU, vector ALU only, both
            D = rng.standard_normal((w.n, ncols)).astype(np.float32)
            Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
            assert relmax(Q, op(D.astype(np.float64))) < 1e-5, (scale, ncols)
        blocks, Cm = prob.assemble(theta)
        for i in range(w.n_clusters):
            Ki = ctx.nugpr_export(B.EXPORT_K, i).cpu().numpy().astype(np.float64)
            np.testing.assert_allclose(Ki, blocks[i], rtol=2e-6, atol=1e-7)
            assert np.array_equal(Ki, Ki.T)
        Cg = ctx.nugpr_export(B.EXPORT_C).cpu().numpy().astype(np.float64)
        assert np.array_equal(Cg, Cg.T)
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t32", "tiny", "iso-d1", "C1-wide"])
def test_precond_factor_and_apply_match_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    code, logdetM, bad = ctx.nugpr_precond_factor()
    assert code == 0 and bad == -1
    fac = O.Factor(prob, w.theta)
    assert abs(logdetM - fac.logdetM) <= 1e-5 * abs(fac.logdetM) + 1e-4
    for i in range(w.n_clusters):
        Li = ctx.nugpr_export(B.EXPORT_L, i).cpu().numpy().astype(np.float64)
        assert relmax(Li, fac.Ls[i]) < 2e-5, ("L", i, relmax(Li, fac.Ls[i]))
        Yi = ctx.nugpr_export(B.EXPORT_LINV, i).cpu().numpy().astype(np.float64)
        ref = np.linalg.inv(fac.Ls[i])
        assert relmax(Yi, ref) < 1e-4, ("Linv", i, relmax(Yi, ref))
    Bg = ctx.nugpr_export(B.EXPORT_B).cpu().numpy().astype(np.float64)
    assert relmax(Bg, fac.B) < 5e-5        # B = L Z inherits the fp32 factor's error
    assert np.array_equal(Bg[:, 0], w.y.astype(np.float64))
    rng = np.random.default_rng(12)
    R = rng.standard_normal((w.n, w.n_probes + 1)).astype(np.float32)
    Z = ctx.nugpr_precond_apply(R).cpu().numpy().astype(np.float64)
    ref = fac.apply(R.astype(np.float64))
    assert relmax(Z, ref) < 1e-4, relmax(Z, ref)
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t16", "ragged-t32", "ragged-halves", "many-reps", "tiny", "iso-d1",
                                  "C1", "C1-wide"])
def test_pcg_solve_and_mll_match_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    code, logdetM, bad = ctx.nugpr_precond_factor()
    assert code == 0
    fac = O.Factor(prob, w.theta)
    ref = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
    Bg = ctx.nugpr_export(B.EXPORT_B)
    code, X, iters, alpha, beta = ctx.nugpr_pcg_solve(Bg)
    assert code == 0, code
    Xg = X.cpu().numpy().astype(np.float64)
    for c in range(w.n_probes + 1):
        err = np.linalg.norm(Xg[:, c] - ref["X"][:, c]) / np.linalg.norm(ref["X"][:, c])
        assert err < 1e-4, (c, err)
    assert np.all(np.abs(iters.astype(np.int64) - ref["iters"]) <= 2)
    # residual of the solve against the oracle's operator
    res = np.linalg.norm(prob.operator(w.theta)(Xg) - fac.B, axis=0) / np.linalg.norm(fac.B, axis=0)
    assert res.max() < 20 * w.tol + 2e-6
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == 0
    record_metric("mll:" + w.name, solve_err=float(max(np.linalg.norm(Xg[:, c] - ref["X"][:, c]) /
                  np.linalg.norm(ref["X"][:, c]) for c in range(w.n_probes + 1))),
                  nll_err=float(abs(out["nll"] - ref["nll"]) / abs(ref["nll"])), iters=int(iters.max()))
    for key in ("quad", "logdet", "nll"):
        assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
    ctx.close()


# Gradient bar: 1e-4 of the gradient norm.  The 25-point case adds the floor that fp32
# STORAGE of the covariance entries imposes whatever the arithmetic: an entry rounding of
# 2^-24 moves each probe's quadratic form by ~1e-6, which the difference quotient
# multiplies by 1/(2h) = 500, while this case's whole gradient is only ~8.
GRAD_FLOOR = {"tiny": 1e-3}


# ragged-t32: 33 columns (two column groups); ragged-halves / many-reps: pair assembly with the lower-only coupling
# matrix and strips that pair up over super-blocks of unequal size
@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t32", "ragged-halves", "many-reps", "tiny", "iso-d1", "C1",
                                  "C1-wide"])
def test_train_step_gradient_matches_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    phi0 = np.log(w.theta)
    p = phi0.shape[0]
    out = ctx.nugpr_train_step(phi0, np.zeros(p), np.zeros(p), 0)
    assert out["code"] == 0, out["code"]
    phi, m, v, step, nll0, g = O.train_step(prob, phi0, np.zeros(p), np.zeros(p), 0, w.fd_step, w.tol,
                                            w.max_iter, lr=w.lr)
    assert abs(out["nll0"] - nll0) <= 1e-4 * abs(nll0)
    gerr = np.linalg.norm(out["grad"] - g) / np.linalg.norm(g)
    print("gradient rel err", gerr, "gpu", out["grad"], "oracle", g, flush=True)
    record_metric("grad:" + w.name, grad_err=float(gerr), nll0_err=float(abs(out["nll0"] - nll0) / abs(nll0)),
                  gnorm=float(np.linalg.norm(g)))
    assert np.linalg.norm(out["grad"] - g) <= 1e-4 * np.linalg.norm(g) + GRAD_FLOOR.get(case, 0.0), gerr
    assert out["step"] == 1
    np.testing.assert_allclose(out["log_theta"], phi, rtol=0, atol=2e-3 * w.lr + 1e-9)
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-t16", "C1"])
def test_train_step_operator_shortcuts_agree_with_fresh_assembly(lib, case):
    # Section 3.3, eqs. (linear2) / (linear3): the output-scale and noise evaluations may reuse the blocks
    # assembled at theta_0 (default) or assemble anew (NUGPR_NO_SHORTCUTS); both must match the oracle,
    # which always assembles in fp64
    w = CASES[case]()
    prob = oracle_problem(w)
    phi0 = np.log(w.theta)
    p = phi0.shape[0]
    _, _, _, _, nll0, g = O.train_step(prob, phi0, np.zeros(p), np.zeros(p), 0, w.fd_step, w.tol, w.max_iter, lr=w.lr)
    grads = {}
    for no_sc in (False, True):
        ctx = make_ctx(lib, w, no_shortcuts=no_sc)
        out = ctx.nugpr_train_step(phi0, np.zeros(p), np.zeros(p), 0)
        assert out["code"] == 0
        assert abs(out["nll0"] - nll0) <= 1e-4 * abs(nll0)
        assert np.linalg.norm(out["grad"] - g) <= 1e-4 * np.linalg.norm(g) + GRAD_FLOOR.get(case, 0.0)
        grads[no_sc] = out["grad"]
        ctx.close()
    # the two hyperparameters the shortcut serves (the last two entries of theta)
    err_sc = np.abs(grads[False][-2:] - g[-2:]).max() / np.linalg.norm(g)
    err_fresh = np.abs(grads[True][-2:] - g[-2:]).max() / np.linalg.norm(g)
    print("alpha / sigma^2 gradient error: shortcut", err_sc, "fresh assembly", err_fresh, flush=True)
    record_metric("shortcut:" + w.name, err_shortcut=float(err_sc), err_fresh=float(err_fresh))
    np.testing.assert_allclose(grads[False][:-2], grads[True][:-2], rtol=0, atol=1e-9 * np.linalg.norm(g))


# Prediction bar: the mean to 1e-4 of the largest mean; the variance to 1e-4 of the prior
# variance alpha (it is alpha minus a quadratic form of that size, so the quadratic form's
# 1e-4 relative accuracy is what can be asked of the difference).
@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t32", "tiny", "iso-d1", "C1", "C1-wide"])
def test_predict_matches_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    # more test points than one batch holds, with a ragged last batch
    m = 2 * (w.n_probes + 1) + 3
    Xt = I.test_points(w, m, seed=5)
    # a theta other than the preconditioner's: prediction after training steps
    theta = w.theta * (1.0 + 0.04 * np.cos(np.arange(w.theta.shape[0])))
    ref = O.predict(prob, fac, theta, Xt, w.tol, w.max_iter)
    out = ctx.nugpr_predict(theta, Xt)
    assert out["code"] == 0
    alpha = theta[-2]
    err_mean = float(np.max(np.abs(out["mean"] - ref["mean"])) / np.max(np.abs(ref["mean"])))
    err_var = float(np.max(np.abs(out["var"] - ref["var"])) / alpha)
    record_metric("predict:" + w.name, err_mean=err_mean, err_var=err_var, m=m,
                  iters=int(out["max_iters_used"]))
    assert err_mean < 1e-4, err_mean
    assert err_var < 1e-4, err_var
    assert abs(out["max_iters_used"] - int(np.max(ref["iters"]))) <= 2
    # mean only: the same means, no variance solves
    out2 = ctx.nugpr_predict(theta, Xt, variance=False)
    assert out2["var"] is None
    assert np.max(np.abs(out2["mean"] - out["mean"])) <= 1e-12 * np.max(np.abs(out["mean"]))
    # the loss path still works on the same context afterwards (its right-hand sides are untouched)
    refl = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
    got = ctx.nugpr_mll(w.theta)
    assert abs(got["nll"] - refl["nll"]) <= 1e-4 * abs(refl["nll"])
    # scores on the host side of the boundary
    yt = np.sin(Xt.astype(np.float64).sum(axis=1))
    assert abs(B.nugpr_rmse(out["mean"], yt) - O.rmse(ref["mean"], yt)) < 1e-4
    ctx.close()


def test_predict_edge_cases(lib):
    w = small_ragged(seed=10, t=4)
    ctx = make_ctx(lib, w)
    Xt = I.test_points(w, 3, seed=1)
    with pytest.raises(B.NugprError) as e:          # needs the factor
        ctx.nugpr_predict(w.theta, Xt)
    assert e.value.code == B.NUGPR_ERR_STATE
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0
    out = ctx.nugpr_predict(w.theta, np.zeros((0, w.d), dtype=np.float32))     # no test points
    assert out["code"] == 0 and out["mean"].shape == (0,)
    with pytest.raises(B.NugprError):
        ctx.nugpr_predict(w.theta, np.zeros((2, w.d + 1), dtype=np.float32))
    # a training input as the test point.  K_* is exact while K' is approximated, so the joint
    # matrix need not be positive semi-definite: the variance is below the prior (K'^-1 is
    # positive definite) but can come out slightly negative, in the oracle as well.
    prob = oracle_problem(w)
    fac = O.Factor(prob, w.theta)
    one = w.X[[17]]
    ref = O.predict(prob, fac, w.theta, one, w.tol, w.max_iter)
    out = ctx.nugpr_predict(w.theta, one)
    assert abs(out["mean"][0] - ref["mean"][0]) < 1e-4 * max(abs(ref["mean"][0]), 1.0)
    assert abs(out["var"][0] - ref["var"][0]) < 1e-4 * w.theta[-2]
    assert out["var"][0] < w.theta[-2]
    ctx.close()


# ---- the paper's own loss machinery (Section 3.1): split operator, Pade log-determinant, forward differences
@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t32", "tiny", "iso-d1", "C1-wide"])
def test_split_operator_matches_oracle_with_and_without_the_identity_relation(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    prob = oracle_problem(w)
    fac = O.Factor(prob, w.theta)
    rng = np.random.default_rng(21)
    D = rng.standard_normal((w.n, w.n_probes + 1)).astype(np.float32)
    theta2 = w.theta * (1.0 + 0.05 * np.sin(1.0 + np.arange(w.theta.shape[0])))
    for no_shortcuts in (False, True):
        ctx = make_ctx(lib, w, no_shortcuts=no_shortcuts)
        ctx.nugpr_build_blocks(w.theta)
        assert ctx.nugpr_precond_factor()[0] == 0
        # stored blocks = factored blocks: eq. (linear1) applies (or is switched off)
        A0 = O.split_operator(prob.operator(w.theta), fac.Ls, prob.offsets)
        got = ctx.nugpr_split_apply(D).cpu().numpy().astype(np.float64)
        ref = A0(D.astype(np.float64))
        e0 = relmax(got, ref)
        # blocks of another theta under the same factor: the general route
        ctx.nugpr_build_blocks(theta2)
        A2 = O.split_operator(prob.operator(theta2), fac.Ls, prob.offsets)
        got2 = ctx.nugpr_split_apply(D[:, :2]).cpu().numpy().astype(np.float64)
        e2 = relmax(got2, A2(D[:, :2].astype(np.float64)))
        record_metric("split:" + w.name, no_shortcuts=int(no_shortcuts), err_same_theta=e0, err_other_theta=e2)
        # the factor and its inverse are fp32: 1e-4 is the bar of the solves they take part in
        assert e0 < 1e-4 and e2 < 1e-4, (e0, e2)
        ctx.close()


@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t32", "tiny", "iso-d1", "C1", "C1-wide"])
def test_pade_loss_matches_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w, logdet_pade=True)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    theta2 = w.theta * (1.0 + 0.03 * np.cos(np.arange(w.theta.shape[0])))
    for th in (w.theta, theta2):
        ref = O.mll(prob, fac, th, w.tol, w.max_iter, logdet="pade")
        out = ctx.nugpr_mll(th)
        assert out["code"] == 0
        record_metric("pade:" + w.name, nll_err=abs(out["nll"] - ref["nll"]) / abs(ref["nll"]),
                      logdet_err=abs(out["logdet"] - ref["logdet"]) / abs(ref["logdet"]),
                      iters=int(out["max_iters_used"]), oracle_iters=int(ref["iters"].max()))
        for key in ("quad", "logdet", "nll"):
            assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
        assert abs(out["max_iters_used"] - int(ref["iters"].max())) <= 2
    ctx.close()


@pytest.mark.parametrize("case,pade", [("ragged-t8", False), ("ragged-t8", True), ("iso-d1", True), ("C1", False),
                                       ("C1", True)])
def test_forward_difference_step_matches_oracle(lib, case, pade):
    w = CASES[case]()
    print("case", w.name, "pade", pade, flush=True)
    rel_step, thr, cap = 0.04, 2e-2, 6
    prob = oracle_problem(w)
    phi = np.log(w.theta)
    p = phi.shape[0]
    ref = O.train_step_forward(prob, phi, np.zeros(p), np.zeros(p), 0, rel_step, thr, cap, w.tol, w.max_iter,
                               logdet="pade" if pade else "slq")
    phi_o, m_o, v_o, step_o, nll_o, g_o, halv_o = ref
    results = {}
    for no_shortcuts in (False, True):
        ctx = make_ctx(lib, w, fd_step=rel_step, fd_forward=True, fd_threshold=thr, fd_max_halvings=cap,
                       logdet_pade=pade, no_shortcuts=no_shortcuts)
        out = ctx.nugpr_train_step(phi, np.zeros(p), np.zeros(p), 0)
        assert out["code"] == 0
        results[no_shortcuts] = (out, ctx.nugpr_fd_halvings().astype(np.int64))
        ctx.close()
    for no_shortcuts, (out, halv) in results.items():
        assert abs(out["nll0"] - nll_o) <= 1e-4 * abs(nll_o)
        gerr = float(np.linalg.norm(out["grad"] - g_o) / np.linalg.norm(g_o))
        record_metric("forward:" + w.name, pade=int(pade), no_shortcuts=int(no_shortcuts), grad_err=gerr,
                      halvings=halv.tolist(), oracle_halvings=halv_o.tolist())
        # The halving count is a decision taken on floating-point quotients: where both sides took the
        # same number of halvings the quotient itself is compared; where they differ by the one step a
        # marginal comparison can cost, both quotients are valid answers of the rule and agree to the
        # threshold the rule itself applies.
        same = halv == halv_o
        assert np.all(np.abs(halv - halv_o) <= 1), (halv, halv_o)
        scale = np.linalg.norm(g_o)
        assert np.all(np.abs(out["grad"] - g_o)[same] <= 1e-4 * scale), (out["grad"], g_o)
        assert np.all(np.abs(out["grad"] - g_o)[~same] <= 2 * thr * np.abs(g_o)[~same] + 1e-4 * scale)
        assert same.sum() >= p - 1
        if np.all(same):
            np.testing.assert_allclose(out["log_theta"], phi_o, rtol=0, atol=2e-4)
    # with and without the linear relations: the same function
    a, b = results[False][0], results[True][0]
    assert np.linalg.norm(a["grad"] - b["grad"]) <= 1e-4 * np.linalg.norm(b["grad"])


# ---- SPD compensation K'' of eqs. (krep), (kypp)
COMP_CASES = dict(CASES)
COMP_CASES["indefinite"] = lambda: small_ragged(seed=12, t=4)        # K' has a negative eigenvalue, K'' has none
COMP_CASES["rank1"] = lambda: I.make_small(n_clusters=5, sizes=[70, 64, 130, 20, 33], d=2, rank=1, t=6, seed=41,
                                            ell=1.0, spacing=0.8, sigma_blob=0.8, noise=0.05, tol=1e-8, max_iter=60)


# couplings beyond the dense host eigen-solve (n_c r > 512): lambda_0 comes from the Lanczos process on the device
COMP_CASES["C2-x0.3"] = lambda: I.make_config("C2", scale=0.3)                    # 10 x 64 = 640 representatives
# strongly overlapping clusters with a wide lengthscale: lambda_0 is 2e-6 alpha and the device iteration stops at its
# step cap with an estimate inside [lambda_0, lambda_0 + 2e-7] (accepted: positive semi-definiteness bounds the error)
COMP_CASES["overlap-640"] = lambda: I.make_small(n_clusters=10, sizes=[150 + (11 * i) % 37 for i in range(10)], d=4,
                                                 rank=64, t=8, seed=21, ell=1.5, spacing=3.0, sigma_blob=0.8, tol=1e-6,
                                                 max_iter=300)
COMP_CASES["many-reps-close"] = lambda: I.make_small(n_clusters=17, sizes=[130 + (7 * i) % 23 for i in range(17)], d=3,
                                                     rank=128, t=16, seed=9, ell=1.5, spacing=2.0, sigma_blob=0.5,
                                                     tol=1e-6, max_iter=100)     # 2176 representatives, clusters touching


@pytest.mark.parametrize("case", ["ragged-t8", "tiny", "iso-d1", "C1", "indefinite", "rank1", "many-reps", "C2-x0.3",
                                  "overlap-640", "many-reps-close"])
def test_compensated_operator_loss_and_gradient_match_oracle(lib, case):
    w = COMP_CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w, compensate=True)
    prob = O.Problem(w.X, w.y, w.offsets, w.probes, w.rank, compensate=True)
    ctx.nugpr_build_blocks(w.theta)
    blocks, Cm = prob.assemble(w.theta)
    lam0 = O.compensation_lambda(Cm)
    big = w.n_clusters * w.rank > 512
    steps = ctx.nugpr_compensation_steps()
    assert (steps > 0) == big
    # dense host eigen-solve: to rounding; Lanczos on the device: to its stopping tolerance (and from above)
    lam_err = ctx.nugpr_compensation_lambda() - lam0
    record_metric("lambda0:" + case, n_reps=w.n_clusters * w.rank, lambda0=lam0, err=float(lam_err), lanczos_steps=steps)
    capped = steps >= 150
    assert abs(lam_err) <= (1e-10 if big else 1e-11) * max(1.0, w.theta[-2]) or (capped and 0.0 <= lam_err <= 1e-6), lam_err
    Cg = ctx.nugpr_export(B.EXPORT_C).cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(Cg, Cm - lam0 * np.eye(Cm.shape[0]), rtol=2e-6, atol=1e-7)
    op = prob.operator(w.theta)
    rng = np.random.default_rng(31)
    for ncols in sorted({1, w.n_probes + 1}):
        D = rng.standard_normal((w.n, ncols)).astype(np.float32)
        Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
        assert relmax(Q, op(D.astype(np.float64))) < 1e-5
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    theta2 = w.theta * (1.0 + 0.03 * np.cos(np.arange(w.theta.shape[0])))
    iters_at = []
    for th in (w.theta, theta2):
        ref = O.mll(prob, fac, th, w.tol, w.max_iter)
        out = ctx.nugpr_mll(th)
        assert out["code"] == 0, out
        for key in ("quad", "logdet", "nll"):
            assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
        assert abs(out["max_iters_used"] - int(ref["iters"].max())) <= 2
        iters_at.append(int(out["max_iters_used"]))
    # Section 3.3: with the factor of the SAME theta the preconditioned system has at most n_c r + 1
    # distinct eigenvalues, so CG needs at most that many iterations (one more allowed for rounding)
    assert iters_at[0] <= w.n_clusters * w.rank + 2
    phi = np.log(w.theta)
    step = ctx.nugpr_train_step(phi, np.zeros(ctx.p), np.zeros(ctx.p), 0)
    g = O.fd_gradient(prob, fac, phi, w.fd_step, w.tol, w.max_iter)
    gerr = float(np.linalg.norm(step["grad"] - g) / np.linalg.norm(g))
    record_metric("compensated:" + w.name, lambda0=lam0, nll_err=abs(out["nll"] - ref["nll"]) / abs(ref["nll"]),
                  grad_err=gerr, iters=int(out["max_iters_used"]))
    assert gerr < max(1e-4, GRAD_FLOOR.get(case, 0.0)), gerr
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-t8", "iso-d1", "C1", "indefinite", "many-reps", "C2-x0.3"])
def test_factor_of_the_compensated_blocks_matches_oracle(lib, case):
    """NUGPR_PRECOND_COMPENSATED: the factor of the diagonal blocks of K'' (eq. (kypp)) as preconditioner.  Factor,
    inverse, log det M, right-hand sides, preconditioner apply, loss and gradient against the oracle's
    Factor(compensated_blocks=True); fewer iterations than with the factor of K_diag."""
    w = COMP_CASES[case]()
    print("case", w.name, flush=True)
    prob = O.Problem(w.X, w.y, w.offsets, w.probes, w.rank, compensate=True)
    plain = make_ctx(lib, w, compensate=True)
    plain.nugpr_build_blocks(w.theta)
    assert plain.nugpr_precond_factor()[0] == 0
    it_plain = plain.nugpr_mll(w.theta)["max_iters_used"]
    plain.close()
    ctx = make_ctx(lib, w, compensate=True, precond_compensated=True)
    ctx.nugpr_build_blocks(w.theta)
    code, logdetM, bad = ctx.nugpr_precond_factor()
    assert code == 0 and bad == -1
    fac = O.Factor(prob, w.theta, compensated_blocks=True)
    assert abs(logdetM - fac.logdetM) <= 1e-5 * abs(fac.logdetM) + 1e-4
    for i in range(min(w.n_clusters, 6)):
        Li = ctx.nugpr_export(B.EXPORT_L, i).cpu().numpy().astype(np.float64)
        assert relmax(Li, fac.Ls[i]) < 2e-5, ("L", i, relmax(Li, fac.Ls[i]))
    rng = np.random.default_rng(12)
    R = rng.standard_normal((w.n, w.n_probes + 1)).astype(np.float32)
    Z = ctx.nugpr_precond_apply(R).cpu().numpy().astype(np.float64)
    assert relmax(Z, fac.apply(R.astype(np.float64))) < 2e-4
    ref = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == 0, out
    for key in ("quad", "logdet", "nll"):
        assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
    assert abs(out["max_iters_used"] - int(ref["iters"].max())) <= 2
    assert out["max_iters_used"] <= it_plain
    phi = np.log(w.theta)
    step = ctx.nugpr_train_step(phi, np.zeros(ctx.p), np.zeros(ctx.p), 0)
    assert step["code"] == 0
    g = O.fd_gradient(prob, fac, phi, w.fd_step, w.tol, w.max_iter)
    gerr = float(np.linalg.norm(step["grad"] - g) / np.linalg.norm(g))
    record_metric("precond-compensated:" + w.name, nll_err=abs(out["nll"] - ref["nll"]) / abs(ref["nll"]), grad_err=gerr,
                  iters=int(out["max_iters_used"]), iters_with_the_factor_of_K_diag=int(it_plain))
    assert gerr < max(1e-4, GRAD_FLOOR.get(case, 0.0)), gerr
    ctx.close()


def test_factor_of_the_compensated_blocks_needs_the_one_hot_basis(lib):
    w = COMP_CASES["ragged-t8"]()
    with pytest.raises(B.NugprError):
        make_ctx(lib, w, precond_compensated=True)                  # without NUGPR_COMPENSATE
    ctx = make_ctx(lib, w, compensate=True, precond_compensated=True)
    ctx.nugpr_build_blocks(w.theta)
    ctx.nugpr_set_nystrom_basis(w.theta)
    ctx.nugpr_build_blocks(w.theta)
    with pytest.raises(B.NugprError) as err:
        ctx.nugpr_precond_factor()
    assert err.value.code == B.NUGPR_ERR_STATE
    ctx.close()


def test_compensation_makes_an_indefinite_problem_solvable(lib):
    w = COMP_CASES["indefinite"]()
    plain = make_ctx(lib, w)
    plain.nugpr_build_blocks(w.theta)
    assert plain.nugpr_precond_factor()[0] == 0
    assert plain.nugpr_mll(w.theta)["code"] == B.NUGPR_INDEFINITE
    plain.close()
    comp = make_ctx(lib, w, compensate=True)
    comp.nugpr_build_blocks(w.theta)
    assert comp.nugpr_precond_factor()[0] == 0
    out = comp.nugpr_mll(w.theta)
    assert out["code"] == 0 and np.isfinite(out["nll"])
    # prediction runs on the compensated operator as well
    prob = O.Problem(w.X, w.y, w.offsets, w.probes, w.rank, compensate=True)
    fac = O.Factor(prob, w.theta)
    Xt = I.test_points(w, 7, seed=2)
    ref = O.predict(prob, fac, w.theta, Xt, w.tol, w.max_iter)
    got = comp.nugpr_predict(w.theta, Xt)
    assert np.max(np.abs(got["mean"] - ref["mean"])) <= 1e-4 * np.max(np.abs(ref["mean"]))
    assert np.max(np.abs(got["var"] - ref["var"])) <= 1e-4 * w.theta[-2]
    comp.close()
    big = I.make_config("C2", scale=0.3)             # n_c r = 10 x 64 = 640 > 512: the device route, fp64 mode only
    with pytest.raises(B.NugprError) as e:
        make_ctx(lib, big, compensate=True, acc_fp32=True)
    assert e.value.code == B.NUGPR_ERR_INVALID


# ---- fp32 arithmetic mode (NUGPR_ACC_FP32): fp32 vector blocks and fp32 matrix-core accumulation.
# Products and solves meet the same bars; the finite-difference gradient is NOT held to 1e-4 in this
# mode (accumulation rounding of ~1e-7 of the loss is divided by 2h), which is why it is not the default:
# the test records its error and bounds it loosely.
@pytest.mark.parametrize("case", ["ragged-t8", "ragged-t32", "tiny", "iso-d1", "C1"])
def test_fp32_mode_matches_oracle(lib, case):
    w = CASES[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w, acc_fp32=True)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    op = prob.operator(w.theta)
    rng = np.random.default_rng(41)
    for ncols in sorted({1, 2, w.n_probes + 1}):
        D = rng.standard_normal((w.n, ncols)).astype(np.float32)
        Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
        assert relmax(Q, op(D.astype(np.float64))) < 2e-5
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    R = rng.standard_normal((w.n, w.n_probes + 1)).astype(np.float32)
    Z = ctx.nugpr_precond_apply(R).cpu().numpy().astype(np.float64)
    assert relmax(Z, fac.apply(R.astype(np.float64))) < 2e-4
    A = O.split_operator(op, fac.Ls, prob.offsets)
    S = ctx.nugpr_split_apply(R).cpu().numpy().astype(np.float64)
    assert relmax(S, A(R.astype(np.float64))) < 2e-4
    ref = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == 0
    for key in ("quad", "logdet", "nll"):
        assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
    Xt = I.test_points(w, w.n_probes + 3, seed=8)
    pref = O.predict(prob, fac, w.theta, Xt, w.tol, w.max_iter)
    pgot = ctx.nugpr_predict(w.theta, Xt)
    assert pgot["code"] == 0
    assert np.max(np.abs(pgot["mean"] - pref["mean"])) <= 1e-4 * np.max(np.abs(pref["mean"]))
    assert np.max(np.abs(pgot["var"] - pref["var"])) <= 1e-4 * w.theta[-2]
    phi = np.log(w.theta)
    step = ctx.nugpr_train_step(phi, np.zeros(ctx.p), np.zeros(ctx.p), 0)
    g = O.fd_gradient(prob, fac, phi, w.fd_step, w.tol, w.max_iter)
    gerr = float(np.linalg.norm(step["grad"] - g) / np.linalg.norm(g))
    record_metric("fp32mode:" + w.name, nll_err=abs(out["nll"] - ref["nll"]) / abs(ref["nll"]), grad_err=gerr)
    assert gerr < 1e-3, gerr
    ctx.close()
    # the Pade route in the same mode
    pctx = make_ctx(lib, w, acc_fp32=True, logdet_pade=True)
    pctx.nugpr_build_blocks(w.theta)
    assert pctx.nugpr_precond_factor()[0] == 0
    pr = O.mll(prob, fac, w.theta, w.tol, w.max_iter, logdet="pade")
    po = pctx.nugpr_mll(w.theta)
    assert po["code"] == 0 and abs(po["nll"] - pr["nll"]) <= 1e-4 * abs(pr["nll"])
    pctx.close()


# ---- degenerate and extreme shapes: no probes, one cluster, rank = cluster size (exact covariance),
# the largest dimension, a dimension that is no multiple of the matrix-core depth, clusters of one point
DEGENERATE = {
    "no-probes": (lambda: I.make_small(n_clusters=3, sizes=[70, 64, 30], d=2, rank=4, t=0, seed=51, ell=1.5, spacing=4.0,
                                       sigma_blob=0.3, tol=1e-8, max_iter=60), False),
    "one-cluster": (lambda: I.make_small(n_clusters=1, sizes=[150], d=3, rank=5, t=4, seed=52, ell=1.2, tol=1e-8,
                                         max_iter=60), False),
    "rank-is-size": (lambda: I.make_small(n_clusters=3, sizes=[12, 12, 12], d=2, rank=12, t=4, seed=53, ell=1.5,
                                          spacing=2.0, sigma_blob=0.5, tol=1e-8, max_iter=80), False),
    "d64": (lambda: I.make_small(n_clusters=2, sizes=[80, 50], d=64, rank=3, t=4, seed=54, ell=8.0, spacing=3.0,
                                 sigma_blob=0.5, tol=1e-8, max_iter=60), True),
    "d7-tiny-clusters": (lambda: I.make_small(n_clusters=3, sizes=[65, 1, 2], d=7, rank=1, t=3, seed=55, ell=2.5,
                                              spacing=3.0, sigma_blob=0.5, tol=1e-8, max_iter=60), True),
    "singletons": (lambda: I.make_small(n_clusters=6, sizes=[1, 1, 1, 1, 1, 1], d=2, rank=1, t=2, seed=56, ell=1.0,
                                        spacing=1.5, sigma_blob=0.1, tol=1e-10, max_iter=60), False),
}


@pytest.mark.parametrize("case", sorted(DEGENERATE))
def test_degenerate_shapes_match_oracle(lib, case):
    mk, compensate = DEGENERATE[case]       # the strongly coupled ones are only definite with the compensation
    w = mk()
    print("case", case, w.name, flush=True)
    ctx = make_ctx(lib, w, compensate=compensate)
    prob = O.Problem(w.X, w.y, w.offsets, w.probes, w.rank, compensate=compensate)
    ctx.nugpr_build_blocks(w.theta)
    blocks, Cm = prob.assemble(w.theta)
    for i in range(w.n_clusters):
        Ki = ctx.nugpr_export(B.EXPORT_K, i).cpu().numpy().astype(np.float64)
        np.testing.assert_allclose(Ki, blocks[i], rtol=2e-6, atol=1e-7)
    op = prob.operator(w.theta)
    rng = np.random.default_rng(61)
    D = rng.standard_normal((w.n, w.n_probes + 1)).astype(np.float32)
    Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
    assert relmax(Q, op(D.astype(np.float64))) < 1e-5
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    if case == "rank-is-size":
        # every point is a representative: K' is the exact covariance (Section 3.3)
        ell, alpha, s2 = O.split_theta(w.theta, w.d)
        Kex = O.rbf(prob.X, prob.X, ell, alpha) + s2 * np.eye(w.n)
        assert relmax(Q, Kex @ D.astype(np.float64)) < 1e-5
    code, X, iters, _, _ = ctx.nugpr_pcg_solve(fac.B.astype(np.float32))
    assert code == 0
    Xo = O.pcg(op, fac.apply, fac.B.astype(np.float32).astype(np.float64), w.tol, w.max_iter)[0]
    Xg = X.cpu().numpy().astype(np.float64)
    for c in range(w.n_probes + 1):
        assert np.linalg.norm(Xg[:, c] - Xo[:, c]) <= 1e-4 * np.linalg.norm(Xo[:, c]), c
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == 0
    if w.n_probes > 0:
        ref = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
        for key in ("quad", "logdet", "nll"):
            assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]) + 1e-9, (key, out[key], ref[key])
        if case == "one-cluster":
            # the preconditioner is the operator itself: one iteration in exact arithmetic, one more
            # here to take the fp32 factor's 1e-6 residual below the 1e-8 tolerance
            assert out["max_iters_used"] <= 2
    else:
        # no probes: the quadratic term is exact, the log-determinant is the preconditioner's part alone
        quad = float(prob.y @ O.pcg(op, fac.apply, prob.y[:, None].copy(), w.tol, w.max_iter)[0][:, 0])
        assert abs(out["quad"] - quad) <= 1e-4 * abs(quad)
        assert abs(out["logdet"] - fac.logdetM) <= 1e-5 * abs(fac.logdetM) + 1e-4
    Xt = I.test_points(w, 5, seed=3)
    pref = O.predict(prob, fac, w.theta, Xt, w.tol, w.max_iter)
    pgot = ctx.nugpr_predict(w.theta, Xt)
    assert np.max(np.abs(pgot["mean"] - pref["mean"])) <= 1e-4 * max(np.max(np.abs(pref["mean"])), 1e-12)
    assert np.max(np.abs(pgot["var"] - pref["var"])) <= 1e-4 * w.theta[-2]
    ctx.close()


def test_user_supplied_representatives_and_dense_basis(lib):
    # reps and W given by the caller (Section 3.3 leaves their choice open): soft, normalised weights instead of
    # the default one-hot basis, so the dense W^T D and W P products run instead of their one-hot forms
    w = small_ragged(seed=3, t=8)
    rng = np.random.default_rng(71)
    r = w.rank
    reps, Ws = [], []
    for i in range(w.n_clusters):
        Xi = w.X[w.offsets[i]:w.offsets[i + 1]].astype(np.float64)
        Ri = Xi[rng.choice(Xi.shape[0], r, replace=False)]
        d2 = ((Xi[:, None, :] - Ri[None, :, :]) ** 2).sum(-1)
        Wi = np.exp(-0.5 * d2 / 0.3 ** 2)
        Wi /= Wi.sum(axis=1, keepdims=True)
        reps.append(Ri.astype(np.float32))
        Ws.append(Wi.astype(np.float32))
    reps = np.concatenate(reps)
    W = np.concatenate(Ws)
    prob = O.Problem(w.X, w.y, w.offsets, w.probes, r, reps=reps, Ws=[x.astype(np.float64) for x in Ws])
    assert np.linalg.eigvalsh(prob.dense(w.theta))[0] > 0.0
    ctx = make_ctx(lib, w, reps=reps, W=W)
    assert np.array_equal(ctx.nugpr_export(B.EXPORT_REPS).cpu().numpy(), reps)
    for i in range(w.n_clusters):
        assert np.array_equal(ctx.nugpr_export(B.EXPORT_W, i).cpu().numpy(), Ws[i])
    ctx.nugpr_build_blocks(w.theta)
    op = prob.operator(w.theta)
    rng2 = np.random.default_rng(72)
    for ncols in (1, w.n_probes + 1):
        D = rng2.standard_normal((w.n, ncols)).astype(np.float32)
        Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
        assert relmax(Q, op(D.astype(np.float64))) < 1e-5
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    ref = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == 0
    for key in ("quad", "logdet", "nll"):
        assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
    A = O.split_operator(op, fac.Ls, prob.offsets)
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0           # stored blocks = factored blocks: eq. (linear1) route
    R = rng2.standard_normal((w.n, w.n_probes + 1)).astype(np.float32)
    S = ctx.nugpr_split_apply(R).cpu().numpy().astype(np.float64)
    assert relmax(S, A(R.astype(np.float64))) < 1e-4
    phi = np.log(w.theta)
    step = ctx.nugpr_train_step(phi, np.zeros(ctx.p), np.zeros(ctx.p), 0)
    g = O.fd_gradient(prob, fac, phi, w.fd_step, w.tol, w.max_iter)
    gerr = float(np.linalg.norm(step["grad"] - g) / np.linalg.norm(g))
    record_metric("user-basis", nll_err=abs(out["nll"] - ref["nll"]) / abs(ref["nll"]), grad_err=gerr)
    assert gerr < 1e-4, gerr
    ctx.close()


@pytest.mark.parametrize("case", ["ragged-t16", "overlap", "r128"])
def test_nystrom_basis_matches_oracle(lib, case):
    # Section 3.3 fixes the basis only at rank one; nugpr_set_nystrom_basis builds W_i = k(X_i, R_i) k(R_i, R_i)^-1
    # on the device.  The basis is an input of the method (theta independent once built): the oracle is handed
    # the library's W, after it has been compared with the formula evaluated in numpy
    w = {"ragged-t16": lambda: small_ragged(seed=4, t=16),
         # clusters moved together: the one-hot K' is indefinite here, the Nystrom one is not
         "overlap": lambda: I.make_config("C1", "wide", centre_shrink=2.0),
         "r128": lambda: I.make_small(n_clusters=5, sizes=[200, 131, 128, 260, 190], d=3, rank=128, t=8, seed=33, ell=1.2,
                                      spacing=4.0, sigma_blob=0.9, tol=1e-6, max_iter=100)}[case]()
    print("case", w.name, flush=True)
    ctx = make_ctx(lib, w)
    theta_b = w.theta * (1.0 + 0.02 * np.sin(np.arange(w.theta.shape[0])))      # the basis point: not the evaluation point
    ctx.nugpr_set_nystrom_basis(theta_b)
    plain = oracle_problem(w)
    ell, alpha, _ = O.split_theta(theta_b, w.d)
    Ws = []
    for i in range(w.n_clusters):
        Wi = ctx.nugpr_export(B.EXPORT_W, i).cpu().numpy().astype(np.float64)
        Xi = plain.X[w.offsets[i]:w.offsets[i + 1]]
        Ri = plain.reps[i * w.rank:(i + 1) * w.rank]
        Krr = O.rbf(Ri, Ri, ell, alpha) + 1e-4 * alpha * np.eye(w.rank)
        ref = np.linalg.solve(Krr, O.rbf(Ri, Xi, ell, alpha)).T
        # the weights themselves are ill-conditioned (kernel matrix of nearby points); what is well defined is
        # what they are used for: the interpolated kernel rows W_i Krr against k(X_i, R_i)
        assert relmax(Wi @ Krr, ref @ Krr) < 1e-4, ("W", i, relmax(Wi @ Krr, ref @ Krr))
        Ws.append(Wi)
    prob = O.Problem(w.X, w.y, w.offsets, w.probes, w.rank, Ws=Ws)
    if case == "overlap":
        assert np.linalg.eigvalsh(plain.dense(w.theta))[0] < 0 < np.linalg.eigvalsh(prob.dense(w.theta))[0]
    ctx.nugpr_build_blocks(w.theta)
    op = prob.operator(w.theta)
    rng = np.random.default_rng(81)
    for ncols in (1, w.n_probes + 1):
        D = rng.standard_normal((w.n, ncols)).astype(np.float32)
        Q = ctx.nugpr_matvec(D).cpu().numpy().astype(np.float64)
        assert relmax(Q, op(D.astype(np.float64))) < 1e-5
    with pytest.raises(B.NugprError) as e:            # a new basis needs a new factorisation call
        ctx.nugpr_mll(w.theta)
    assert e.value.code == B.NUGPR_ERR_STATE
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    ref = O.mll(prob, fac, w.theta, w.tol, w.max_iter)
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == 0
    for key in ("quad", "logdet", "nll"):
        assert abs(out[key] - ref[key]) <= 1e-4 * abs(ref[key]), (key, out[key], ref[key])
    phi = np.log(w.theta)
    step = ctx.nugpr_train_step(phi, np.zeros(ctx.p), np.zeros(ctx.p), 0)
    assert step["code"] == 0
    g = O.fd_gradient(prob, fac, phi, w.fd_step, w.tol, w.max_iter)
    gerr = float(np.linalg.norm(step["grad"] - g) / np.linalg.norm(g))
    record_metric("nystrom:" + case, nll_err=abs(out["nll"] - ref["nll"]) / abs(ref["nll"]), grad_err=gerr,
                  iters=int(out["max_iters_used"]))
    assert gerr < 1e-4, gerr
    ctx.close()


def test_stale_factor_is_reused_across_theta(lib):
    # Section 3.2: the factor of theta_0 preconditions K(theta') too; eq. (logdet) stays exact
    w = small_ragged(seed=11, t=16)
    ctx = make_ctx(lib, w)
    prob = oracle_problem(w)
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0
    fac = O.Factor(prob, w.theta)
    theta2 = w.theta * np.array([1.05, 0.97, 1.02, 1.1, 0.9])
    ref = O.mll(prob, fac, theta2, w.tol, w.max_iter)
    out = ctx.nugpr_mll(theta2)
    assert out["code"] == 0
    assert abs(out["nll"] - ref["nll"]) <= 1e-4 * abs(ref["nll"])
    assert abs(out["logdet_precond"] - fac.logdetM) <= 1e-5 * abs(fac.logdetM) + 1e-4
    ctx.close()


def test_error_paths(lib):
    w = small_ragged(seed=10, t=4)
    ctx = make_ctx(lib, w)
    # call order
    with pytest.raises(B.NugprError) as e:
        ctx.nugpr_mll(w.theta)
    assert e.value.code == B.NUGPR_ERR_STATE
    with pytest.raises(B.NugprError) as e:
        ctx.nugpr_build_blocks(np.array([1.0, -1.0, 1.0, 1.0, 0.1]))
    assert e.value.code == B.NUGPR_ERR_INVALID
    # max_iter = 1: not converged, results still written
    w2 = small_ragged(seed=10, t=4)
    ctx2 = make_ctx(lib, w2, max_iter=1, tol=1e-9)
    ctx2.nugpr_build_blocks(w2.theta)
    assert ctx2.nugpr_precond_factor()[0] == 0
    code, X, iters, _, _ = ctx2.nugpr_pcg_solve(ctx2.nugpr_export(B.EXPORT_B))
    assert code == B.NUGPR_NOT_CONVERGED and iters.max() == 1
    assert np.isfinite(X.cpu().numpy()).all()
    ctx.close()
    ctx2.close()


def test_nan_in_the_targets_is_reported_not_iterated_on(lib):
    # a NaN in y poisons <b, b> and <b, M^-1 b> of column 0: the solve must say so (and end), the other
    # columns are unaffected
    w = small_ragged(seed=10, t=4)
    y = w.y.copy()
    y[37] = np.nan
    ctx = lib.Context(w.X, y, w.offsets, w.probes, w.rank, tol=w.tol, max_iter=w.max_iter)
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0           # the factor does not involve y
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == B.NUGPR_NOT_FINITE and np.isnan(out["nll"])
    assert out["max_iters_used"] <= w.max_iter
    step = ctx.nugpr_train_step(np.log(w.theta), np.zeros(ctx.p), np.zeros(ctx.p), 0)
    assert step["code"] == B.NUGPR_NOT_FINITE
    # an infinite entry in a caller's right-hand side: same status from the solver itself
    Bg = ctx.nugpr_export(B.EXPORT_B).clone()
    Bg[:, 0] = 1.0
    Bg[5, 2] = float("inf")
    code, X, iters, _, _ = ctx.nugpr_pcg_solve(Bg)
    assert code == B.NUGPR_NOT_FINITE
    Xh = X.cpu().numpy()
    assert np.isfinite(Xh[:, [0, 1, 3, 4]]).all()        # the clean columns were solved
    ctx.close()
    # NaN / Inf in X: found when the blocks are assembled, reported by the factorisation and the train step
    for row, val in ((int(w.offsets[2]) + 3, np.nan), (int(w.offsets[1]) + 40, np.inf)):
        X2 = w.X.copy()
        X2[row, 1] = val
        ctx2 = lib.Context(X2, w.y, w.offsets, w.probes, w.rank, tol=w.tol, max_iter=w.max_iter)
        ctx2.nugpr_build_blocks(w.theta)
        assert ctx2.nugpr_precond_factor()[0] == B.NUGPR_NOT_FINITE
        with pytest.raises(B.NugprError) as e:          # no valid factor: a loss cannot be asked for
            ctx2.nugpr_mll(w.theta)
        assert e.value.code == B.NUGPR_ERR_STATE
        assert ctx2.nugpr_train_step(np.log(w.theta), np.zeros(ctx2.p), np.zeros(ctx2.p), 0)["code"] == B.NUGPR_NOT_FINITE
        ctx2.close()
    # clean inputs on a fresh context after all that: the flag does not stick to the library
    ctx3 = make_ctx(lib, w)
    ctx3.nugpr_build_blocks(w.theta)
    assert ctx3.nugpr_precond_factor()[0] == 0 and ctx3.nugpr_mll(w.theta)["code"] == 0
    ctx3.close()


def test_not_positive_definite_block_is_reported(lib):
    # duplicate points with (numerically) no noise: the second cluster's block is singular
    # (a short lengthscale keeps the first cluster's block close to alpha*I, so only the
    # cluster of identical points, K = alpha 1 1^T + 1e-12 I, loses definiteness in fp32)
    w = I.make_small(n_clusters=2, sizes=[70, 66], d=2, rank=2, t=2, seed=13, spacing=4.0, sigma_blob=0.3,
                     ell=0.02, tol=1e-6, max_iter=20)
    w.X[70:] = w.X[70]
    theta = w.theta.copy()
    theta[-1] = 1e-12
    ctx = make_ctx(lib, w)
    ctx.nugpr_build_blocks(theta)
    code, logdetM, bad = ctx.nugpr_precond_factor()
    assert code == B.NUGPR_NOT_PD and bad == 1
    ctx.close()


def test_indefinite_operator_is_reported(lib):
    # overlapping clusters with a wide lengthscale: the uncompensated K' is not SPD (Section 3.3)
    w = I.make_small(n_clusters=4, sizes=[64, 70, 80, 66], d=2, rank=2, t=4, seed=43, ell=1.5, halfwidth=3.0,
                     tol=1e-8, max_iter=200)
    prob = oracle_problem(w)
    assert np.linalg.eigvalsh(prob.dense(w.theta)).min() < 0
    ctx = make_ctx(lib, w)
    ctx.nugpr_build_blocks(w.theta)
    assert ctx.nugpr_precond_factor()[0] == 0
    out = ctx.nugpr_mll(w.theta)
    assert out["code"] == B.NUGPR_INDEFINITE
    ctx.close()
