"""Kernel branches at the sizes where they can go wrong: the edges of tiles,
the remainders, the smallest and largest sizes that a dispatch rule sends each
way."""
import numpy as np
import pytest

import coxsim
import oracle
from tests.gpu_helpers import device_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
import paper_2010_16114_amd as P  # noqa: E402


def _bits(a, b):
    np.testing.assert_array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8))


@pytest.mark.parametrize("p", [1, 17, 257, 32767, 32785])
def test_epilogue_column_blocks(p):
    """The proximal epilogue with one thread per column (up to 7 vectors) and
    with 16 or 8 (from 8 on; 16 or 32 columns per workgroup) takes each vector's
    step and l1 norm the same way, so a step of 7 of 8 vectors agrees with the
    step of all 8 bit for bit: a last block of one column, fewer columns than a
    block, both sides of the width where the block grows."""
    d = coxsim.genotype_problem(200, p, min(p, 8), 0.3, 900 + p, days=True)
    cox, M = device_problem(d, "int8", ldx=208, max_batch=8)
    lams = coxsim.lambda_grid(0.9 * oracle.lambda_max(M, d.time, d.event), 8, 0.05)
    sigma = 1.0 / (2.0 * (np.sqrt(d.n) + np.sqrt(d.p)) ** 2)
    rng = np.random.Generator(np.random.PCG64(p))
    beta = (rng.normal(0, 0.05, (8, p)) * (rng.random((8, p)) < 0.3)).astype(np.float32)
    b8, b7 = torch.from_numpy(beta).cuda(), torch.from_numpy(beta[:7].copy()).cuda()
    o8 = cox.prox_step(b8, lams, sigma)
    o7 = cox.prox_step(b7, lams[:7], sigma)
    assert (b7.cpu().numpy() != beta[:7]).any()
    _bits(b8[:7].cpu().numpy(), b7.cpu().numpy())
    _bits(o8[:7], o7)


@pytest.mark.parametrize("n,p,B", [(130, 40, 9), (700, 65, 64), (3001, 257, 20)])
def test_small_matrix_core_splits(n, p, B, monkeypatch):
    """With fewer blocks than compute units the eta update shares a block's
    stages among workgroups and the X~' R pass splits its subjects: one stage per
    share, more shares than stages, a ragged last stage.  The sums are exact
    integers, so both agree bit for bit with the unsplit shapes."""
    d = coxsim.genotype_problem(n, p, 4, 0.3, 700 + n, days=True)
    cox, M = device_problem(d, "fp8", ldx=(n + 15) // 16 * 16, max_batch=B)
    lams = coxsim.lambda_grid(oracle.lambda_max(M, d.time, d.event), B, 0.01)
    sigma = 1.0 / (2.0 * (np.sqrt(n) + np.sqrt(p)) ** 2)
    out = []
    for xv, ev in ((14, 2), (15, 8), (15, 11)):
        monkeypatch.setenv("COXHIP_MFMA_VARIANT", str(xv))
        monkeypatch.setenv("COXHIP_ETA_VARIANT", str(ev))
        beta, _, obj, _ = cox.fit_path(lams, max_iter=10, tol=0.0, step=sigma)
        out.append((beta.cpu().numpy(), obj))
    assert (out[0][0] != 0).any()
    for beta, obj in out[1:]:
        _bits(beta, out[0][0])
        _bits(obj, out[0][1])


@pytest.mark.parametrize("n,B,ties", [(1, 9, "none"), (7, 16, "none"), (17, 17, "days"), (255, 33, "all"),
                                      (257, 48, "none"), (4099, 64, "days"), (4113, 20, "long"), (9001, 40, "none")])
def test_batched_risk_rows(n, B, ties):
    """The batched risk-set passes (state in rows of 16, 32, 48 or 64 vectors, 32,
    16, 10 or 8 tiles to a workgroup) at the edges of their tiles: fewer subjects
    than a tile, tie groups inside a tile, over many tiles and workgroups, over all
    subjects, and tied censored subjects.  Losses to the batched tests' 1e-12.  The
    gradient differs from the oracle's by the residual's rounding to q = max|r| /
    2^22 (at most q / 2 a subject) and the FP32 output: s_j sum_i |g_ij - mu_j| q / 2
    + 2^-23 |g_j| for the SNPs, FP32 rounding alone for the covariates."""
    p, q = 37, 3
    d = coxsim.genotype_problem(max(n, 30), p, 3, 0.4, 4000 + n)
    rng = np.random.Generator(np.random.PCG64(n))
    G = d.G[:, :n].copy()
    time = {"none": rng.random(n), "days": rng.integers(1, 40, n).astype(float), "all": np.ones(n),
            "long": np.where(rng.random(n) < 0.7, 5.0, rng.random(n) * 10)}[ties]
    event = (rng.random(n) < 0.5).astype(np.int32)
    event[0] = 1
    ldx = (n + 15) // 16 * 16
    X = torch.zeros((p, ldx), dtype=torch.int8)
    X[:, :n] = torch.from_numpy(G)
    Z = rng.normal(size=(q, n)).astype(np.float32)
    cox = P.Cox(X.cuda(), time, event, xtype=P.X_INT8, n=n, center=torch.from_numpy(d.mu).cuda(),
                scale=torch.from_numpy(d.s).cuda(), max_batch=B)
    cox.set_covariates(torch.from_numpy(Z).cuda())
    beta = (rng.normal(0, 0.2, (B, p + q)) * (rng.random((B, p + q)) < 0.5)).astype(np.float32)
    loss, grad = cox.loss_grad(torch.from_numpy(beta).cuda())
    only, _ = cox.loss_grad(torch.from_numpy(beta).cuda(), want_grad=False)
    _bits(loss, only)
    grad = grad.cpu().numpy()
    Xs = (G.astype(np.float64) - d.mu[:, None].astype(np.float64)) * d.s[:, None].astype(np.float64)
    full = np.concatenate([Xs, Z.astype(np.float64)])
    M = oracle.Matrix.dense(full)
    for b in range(B):
        negL, gl = oracle.loss_grad(M, time, event, beta[b].astype(np.float64))
        go = -gl  # the oracle gives the gradient of L
        assert loss[b] == pytest.approx(negL, rel=1e-12, abs=1e-12 * n), b
        r = oracle.loglik(full.T @ beta[b].astype(np.float64), time, event)[1]
        tol = 2.0**-23 * np.abs(go) + 1e-12 * n
        tol[:p] += np.abs(Xs).sum(axis=1) * np.abs(r).max() * 2.0**-23
        assert (np.abs(grad[b] - go) <= tol).all(), (b, np.abs(grad[b] - go).max())


@pytest.mark.parametrize("n,lead", [(1000, 0), (1009, 48), (2040, 112), (2040, 0), (40, 16), (130, 64)])
def test_whole_line_loads(n, lead):
    """The X~' R shapes that load whole 128-byte lines of X (13 to 15) agree bit for
    bit with a shape that loads 64-byte pieces from the column's start (8), for
    columns that start anywhere in a line: ldx 0, 16, 48, 112 bytes past a multiple
    of 128, X itself `lead` bytes into a line, less than a stage of subjects."""
    p, B = 530, 16
    d = coxsim.genotype_problem(n, p, 4, 0.3, 7000 + n + lead, days=True)
    ldx = (n + 15) // 16 * 16
    buf = torch.full((p * ldx + 256,), 0x40, dtype=torch.uint8)  # the bytes around X and its padding are not zero
    X = buf[lead:lead + p * ldx].view(p, ldx)
    X[:, :n] = torch.from_numpy(coxsim.FP8_E4M3_CODE[d.G])
    dev = buf.cuda()
    X = dev[lead:lead + p * ldx].view(p, ldx)
    assert X.data_ptr() % 128 == lead
    cox = P.Cox(X, d.time, d.event, xtype=P.X_FP8_E4M3, n=n, center=torch.from_numpy(d.mu).cuda(),
                scale=torch.from_numpy(d.s).cuda(), max_batch=B)
    lams = coxsim.lambda_grid(0.8 * cox.lambda_max(), B, 0.05)
    sigma = 1.0 / (2.0 * (np.sqrt(n) + np.sqrt(p)) ** 2)
    out = []
    for xv in (8, 13, 14, 15):
        with pytest.MonkeyPatch.context() as mp:
            mp.setenv("COXHIP_MFMA_VARIANT", str(xv))
            mp.setenv("COXHIP_ETA_VARIANT", "2")
            beta, _, obj, _ = cox.fit_path(lams, max_iter=6, tol=0.0, step=sigma)
        out.append((beta.cpu().numpy(), obj))
    assert (out[0][0] != 0).any()
    for beta, obj in out[1:]:
        _bits(beta, out[0][0])
        _bits(obj, out[0][1])


@pytest.mark.parametrize("n,p,B", [(33000, 130, 64), (131100, 65, 9), (66000, 200, 20), (33000, 64, 40), (1000, 1000, 64),
                                   (513, 63, 16), (129, 700, 33)])
def test_dense_product_blocks(n, p, B, monkeypatch):
    """The one-pass dense X~ beta of the matrix cores (512, 256 or 128 subjects per
    block; whole rounds of blocks and a last one split over columns; odd and even
    numbers of 64-column stages) against the FP64 vector passes: the losses agree to
    the batched tests' 1e-12, and a vector with a NaN stays alone in its loss."""
    d = coxsim.genotype_problem(n, p, 4, 0.5, 8100 + n, days=True)
    cox, _ = device_problem(d, "int8", ldx=(n + 15) // 16 * 16, max_batch=B)
    rng = np.random.Generator(np.random.PCG64(n + p))
    scale = 10.0 ** rng.uniform(-6, 0, (B, 1))
    beta = torch.from_numpy((0.2 * scale * rng.normal(size=(B, p))).astype(np.float32)).cuda()
    beta[1] = 0.0
    loss, _ = cox.loss_grad(beta, want_grad=False)
    monkeypatch.setenv("COXHIP_NO_MFMA", "1")
    ref, _ = cox.loss_grad(beta, want_grad=False)
    monkeypatch.delenv("COXHIP_NO_MFMA")
    np.testing.assert_allclose(loss, ref, rtol=1e-12)
    beta[B // 2, p // 2] = float("nan")
    with pytest.raises(P.CoxError):
        cox.loss_grad(beta, want_grad=False)


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("ties", [False, True])
def test_small_risk_sets(n, ties):
    """The risk-set phases in one launch (up to 4,096 subjects, four tiles of 1,024)
    and just above in five: loss and adjoint in FP64 against the oracle's.  Both sum
    at most n terms of one sign in FP64, so 1e-12 of the loss and of each residual's
    parts (delta and w c, at most 1 + |r|) covers the rounding many times over."""
    rng = np.random.Generator(np.random.PCG64(31 * n + ties))
    time = rng.integers(1, 50, n).astype(float) if ties else rng.random(n)
    event = (rng.random(n) < 0.6).astype(np.int32)
    event[-1] = 1
    eta = rng.normal(0, 1.5, (3, n))
    cox = P.Cox(torch.zeros((1, (n + 15) // 16 * 16), device="cuda"), time, event, n=n, max_batch=3)
    et = torch.from_numpy(eta).cuda().requires_grad_(True)
    loss = P.BreslowNLL.apply(et, cox)
    loss.sum().backward()
    for b in range(3):
        L, r = oracle.loglik(eta[b], time, event)
        assert float(loss[b].detach()) == pytest.approx(-L, rel=1e-12, abs=1e-12 * n)
        assert (np.abs(et.grad[b].cpu().numpy() + r) <= 1e-12 * (1 + np.abs(r))).all()


@pytest.mark.parametrize("storage,p,B", [("f32", 40, 1), ("fp8", 127, 2), ("int8", 2100, 1), ("f32", 5000, 3),
                                         ("fp8", 9000, 8)])
def test_eta_update_stages(storage, p, B):
    """The eta update's column groups staged through LDS, 128 columns at a time
    with 8 loads in flight: lists of fewer columns than groups, of part stages and
    of several stages per group, held to the parity tests' bars (1e-5 of max|beta|,
    1e-6 in the objective) after steps that each hang on the one before."""
    d = coxsim.genotype_problem(1500, p, 5, 0.3, 6000 + p, days=True)
    cox, M = device_problem(d, storage, ldx=1504, max_batch=B)
    lams = coxsim.lambda_grid(oracle.lambda_max(M, d.time, d.event), B + 1, 0.02)[1:]
    sigma = 1.0 / (2.0 * (np.sqrt(d.n) + np.sqrt(d.p)) ** 2)
    beta, _, obj, _ = cox.fit_path(lams, max_iter=20, tol=0.0, step=sigma)
    beta = beta.cpu().numpy()
    for b in range(B):
        bo, tr, _, _ = oracle.fit(M, d.time, d.event, lams[b], sigma, max_iter=20)
        assert np.abs(beta[b] - bo).max() <= 1e-5 * np.abs(bo).max()
        assert obj[b] == pytest.approx(tr[-1], rel=1e-6)


@pytest.mark.parametrize("r", [1, 4, 13, 21, 24, 29, 32, 33, 46, 51, 56, 64])
@pytest.mark.parametrize("m,n,pad", [(65, 130, 2), (255, 513, 0), (1, 5, 0), (514, 256, 0)])
def test_nmf_rank_quads(r, m, n, pad):
    """Every instance of the NMF contractions (1 to 16 quads of the rank; 64, 128
    or 256 rows or columns per workgroup with ragged ends; aligned rows and not).
    The multiplicative update only adds and multiplies nonnegative FP64 numbers and
    divides once, so three iterations from positive factors carry at most
    3 (2 (m + n) + 2 r + 3) roundings of 1.2e-16, under 2e-12 here."""
    rng = np.random.default_rng(100 * r + m)
    X = rng.random((m, n)).astype(np.float32)
    Xd = torch.zeros((m, n + pad), dtype=torch.float32)
    Xd[:, :n] = torch.from_numpy(X)
    Vt0, W0 = 0.1 + rng.random((r, m)), 0.1 + rng.random((r, n))
    Vt, W = torch.from_numpy(Vt0).cuda(), torch.from_numpy(W0).cuda()
    nmf = P.NMF(Xd.cuda(), r, n=n)
    nmf.run(Vt, W, P.NMF_MULTIPLICATIVE, 3)
    Vo, Wo, _ = oracle.nmf_run(X, Vt0, W0, P.NMF_MULTIPLICATIVE, 3)
    np.testing.assert_allclose(Vt.cpu().numpy(), Vo, rtol=1e-11)
    np.testing.assert_allclose(W.cpu().numpy(), Wo, rtol=1e-11)


@pytest.mark.parametrize("n,M", [(257, 1), (1025, 8), (4095, 3), (4096, 32), (4097, 9), (8200, 33), (4099, 64), (4101, 65),
                                 (12300, 129), (5000, 200)])
def test_refit_blocks(n, M):
    """The refit's passes over the design (chunks of 4,096 positions, columns in
    groups of 4 and 8, eta in blocks of 256), the Gram tiles (16, 32 and 64 columns
    and their ragged last ones) and the factor's blocks of 32: at the Newton solution
    both sides solve the same FP64 equations, so coefficients, errors and likelihood
    agree to the refit tests' 1e-8 (1e-12 for the likelihood)."""
    rng = np.random.Generator(np.random.PCG64(17 * n + M))
    X = rng.normal(size=(M, n)).astype(np.float32)
    eta = 0.3 * X[:min(M, 5)].sum(axis=0)
    time = np.ceil(200 * rng.exponential(np.exp(-eta)))
    event = (rng.random(n) < 0.7).astype(np.int32)
    ldx = (n + 15) // 16 * 16
    Xd = torch.zeros((M, ldx), dtype=torch.float32)
    Xd[:, :n] = torch.from_numpy(X)
    cox = P.Cox(Xd.cuda(), time, event, n=n)
    coef, se, pv, L, it, st = cox.refit(np.arange(M), gtol=1e-9)
    assert st == P.OK
    Mo = oracle.Matrix.dense(X.astype(np.float64))
    b, cov, _, conv = oracle.newton(Mo, time, event, np.arange(M), gtol=1e-11, maxit=100)
    assert conv
    np.testing.assert_allclose(coef, b, rtol=1e-8, atol=1e-9)
    np.testing.assert_allclose(se, np.sqrt(np.diag(cov)), rtol=1e-8)
    assert L == pytest.approx(oracle.loglik(oracle.xbeta(Mo, b), time, event)[0], rel=1e-12)


def test_sums_longer_than_int32_holds(monkeypatch):
    """From 2^23 subjects (columns) on the int8 limbs' int32 sums could wrap: they are
    taken in shares, in the shapes too that do not split otherwise (X~' R 14, eta update
    2).  2^23 + 512 tied subjects, 256 of them events: every censored residual is -256/n,
    held as -128 q (lowest limb -128), against a column of twos.  2^24 + 64 equal columns,
    whose equal steps have the top limb 64: one ISTA step moves them all, and a warm
    start takes the dense product over them.  The gradient is off by at most q / 2 a
    subject (q = max|r| / 2^22) and the FP32 output; the step and with it eta by 2^-22 of
    themselves, the objective (at most 4 in size of its derivative's terms) by 1e-6."""
    monkeypatch.setenv("COXHIP_MFMA_VARIANT", "14")
    monkeypatch.setenv("COXHIP_ETA_VARIANT", "2")
    B, ev = 9, 256
    n = 2**23 + 512
    X = torch.zeros((2, n), dtype=torch.int8, device="cuda")
    X[0, ev:] = 2
    event = np.zeros(n, np.int32)
    event[:ev] = 1
    cox = P.Cox(X, np.ones(n), event, xtype=P.X_INT8, max_batch=B)
    loss, grad = cox.loss_grad(torch.zeros((B, 2), device="cuda"))
    np.testing.assert_allclose(loss, ev * np.log(n), rtol=1e-12)
    want = 2.0 * (n - ev) * ev / n
    np.testing.assert_allclose(grad[:, 0].cpu().numpy(), want, rtol=2.0**-23, atol=2.0 * (n - ev) * 2.0**-23)
    np.testing.assert_array_equal(grad[:, 1].cpu().numpy(), 0.0)
    cox.close()
    del cox, X, grad
    n, p = 16, 2**24 + 64
    X = torch.zeros((p, n), dtype=torch.int8, device="cuda")
    X[:, 0] = 2
    time = np.arange(n, 0, -1.0)  # subject 0 leaves last: it is in every risk set
    cox = P.Cox(X, time, np.ones(n, np.int32), xtype=P.X_INT8, max_batch=B)

    def negL(eta0):
        e = np.exp(np.r_[eta0, np.zeros(n - 1)])
        return np.log(np.cumsum(e)).sum() - eta0

    g = 2.0 * (1.0 - (1.0 / np.arange(1, n + 1)).sum())
    lams = np.linspace(0.5, 0.1, B) * abs(g)
    step = 1.0 / (2.0 * p * abs(g))
    beta, _, obj, _ = cox.fit_path(lams, max_iter=1, tol=0.0, step=step)
    want = np.sign(g) * step * (abs(g) - lams)
    f1 = np.array([negL(2.0 * p * b) + l * p * abs(b) for b, l in zip(want, lams)])
    assert (np.abs(f1 - negL(0.0)) > 0.1).all()  # the step matters
    np.testing.assert_allclose(beta[:, ::p - 1].cpu().numpy(), np.repeat(want[:, None], 2, 1), rtol=1e-6)
    np.testing.assert_allclose(obj, f1, rtol=1e-6)
    _, _, warm, _ = cox.fit_path(lams, max_iter=0, tol=0.0, step=step, beta=beta)
    np.testing.assert_allclose(warm, f1, rtol=1e-6)


def test_eta_shapes_are_timed_on_a_filled_list(tmp_path, monkeypatch):
    """A batch warm-started where nothing moves (lambda above lambda_max, beta 0) has an
    empty change list, on which every shape of the eta update takes no time: none is
    kept or stored.  The next fit, whose first steps move most columns, is timed."""
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("COXHIP_TUNE_CACHE", str(cache))
    for v in ("COXHIP_MFMA_VARIANT", "COXHIP_ETA_VARIANT"):
        monkeypatch.delenv(v, raising=False)
    B = 16
    d = coxsim.genotype_problem(1000, 600, 4, 0.3, 77, days=True)
    cox, _ = device_problem(d, "int8", ldx=1008, max_batch=B)
    lm = cox.lambda_max()
    sigma = 1.0 / (2.0 * cox.opnorm2()[0])
    beta, _, _, _ = cox.fit_path(lm * np.linspace(3.0, 2.0, B), max_iter=20, tol=0.0, step=sigma,
                                 beta=torch.zeros((B, 600), device="cuda"))
    assert not beta.any()
    assert cox.mfma_tuning()["eta_variant"] == -1 and '"eta|' not in cache.read_text()
    lams = coxsim.lambda_grid(lm, B, 0.01)
    beta, _, obj, _ = cox.fit_path(lams, max_iter=5, tol=0.0, step=sigma)
    t = cox.mfma_tuning()
    assert t["eta_variant"] >= 0 and all(m > 0 for m in t["eta_ms"][:P.ETA_VARIANTS])
    assert '"eta|' in cache.read_text()
    monkeypatch.setenv("COXHIP_ETA_VARIANT", "0")  # the shape that serves meanwhile: the same integer sums
    again, _, oagain, _ = cox.fit_path(lams, max_iter=5, tol=0.0, step=sigma)
    _bits(again.cpu().numpy(), beta.cpu().numpy())
    _bits(oagain, obj)


def test_tune_cache_keeps_layouts_apart(tmp_path, monkeypatch):
    """A shape timed for columns on whole 128-byte lines is not taken from the cache for
    columns that are not, nor for an X that starts inside a line, and is for its own."""
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("COXHIP_TUNE_CACHE", str(cache))
    for v in ("COXHIP_MFMA_VARIANT", "COXHIP_ETA_VARIANT"):
        monkeypatch.delenv(v, raising=False)
    B, n, p = 16, 500, 130
    d = coxsim.genotype_problem(n, p, 4, 0.3, 78, days=True)
    timed = []
    for ldx, lead in ((512, 0), (528, 0), (512, 16), (512, 0)):
        buf = torch.zeros(p * ldx + 256, dtype=torch.uint8)
        buf[lead:lead + p * ldx].view(p, ldx)[:, :n] = torch.from_numpy(coxsim.FP8_E4M3_CODE[d.G])
        X = buf.cuda()[lead:lead + p * ldx].view(p, ldx)
        cox = P.Cox(X, d.time, d.event, xtype=P.X_FP8_E4M3, n=n, max_batch=B)
        cox.loss_grad(torch.zeros((B, p), device="cuda"))
        timed.append(any(cox.mfma_tuning()["xtr_ms"]))
    assert timed == [True, True, True, False]
    assert cache.read_text().count('"xtr|') == 3


@pytest.mark.parametrize("storage,n,p,B", [("f32", 60000, 40, 64), ("fp8", 60000, 400, 64), ("int8", 2000, 20000, 64),
                                           ("fp8", 30000, 1000, 33), ("f32", 1000, 2000, 64), ("fp8", 200000, 64, 16)])
def test_workspace_of_a_handle(storage, n, p, B):
    """What a handle holds on the device: five B x n FP64 arrays of state and the FP32
    residual, four column groups of eta updates (two from 128 x 1,024 rows on) and the
    dense X beta's partial sums, four B x p FP64 arrays and the split sums of X'r, and on the
    matrix cores three limbs per vector, row and column and five rounds of 256 x 256
    sums per vector padded to 16.  Everything else is small beside it: 5% and the 64 MB that the
    column groups of any batch may take."""
    up = lambda a, m: (a + m - 1) // m * m  # noqa: E731
    one = storage != "f32"
    X = torch.zeros((p, up(n, 16)), dtype=torch.int8 if storage == "int8" else torch.uint8 if one else torch.float32)
    time = np.arange(n, 0, -1.0)
    event = (np.arange(n) % 5 == 0).astype(np.int32)
    Xd = X.cuda()
    torch.cuda.synchronize()
    held = P.device_bytes()
    cox = P.Cox(Xd, time, event, n=n, max_batch=B)
    got = P.device_bytes() - held
    pad, rs, nslab = up(B, 16), up(n, 8192), up(n, 1024) // 1024
    wgs, chunks = -(-p // (64 if one else 16)), rs // 8192
    nsplit = min(chunks, max(1, -(-12288 // wgs)))
    gemv = max(8 * max(1, min(-(-2048 // nslab), -(-p // 256))), 4 * max(1, min(-(-2048 // (up(n, 4096) // 4096)), -(-p // 64))))
    limit = 8 * 5 * B * n + 4 * B * rs + 8 * (max(1, min(4, 512 // nslab)) * B + gemv) * n + 8 * (4 + nsplit) * B * p
    if one:
        limit += 3 * pad * (rs + up(p, 64)) + 8 * 5 * 256 * 256 * pad
    assert got <= 1.05 * limit + 64 * 2**20, (got, limit)
    cox.close()
    assert P.device_bytes() == held


@pytest.mark.parametrize("q,B", [(16, 16), (17, 9), (17, 48), (33, 40), (64, 16), (64, 64)])
def test_batched_risk_rows_many_covariates(q, B):
    """Covariates beside the batched form: Z' r takes them 16 at a time and reuses its
    LDS between the chunks, Z beta holds up to 64 x 64 coefficients there; whole, ragged
    and last chunks, rows of 16, 48 and 64 vectors.  Losses to the batched tests'
    1e-12; gradients of the covariates to FP32 rounding, of the SNPs to the residual's
    22 bits as well (s_j sum_i |g_ij - mu_j| q / 2)."""
    n, p = 1203, 21
    d = coxsim.genotype_problem(n, p, 3, 0.4, 5000 + q, days=True)
    cox, _ = device_problem(d, "int8", ldx=1216, max_batch=B)
    rng = np.random.Generator(np.random.PCG64(100 * q + B))
    Z = rng.normal(size=(q, n)).astype(np.float32)
    cox.set_covariates(torch.from_numpy(Z).cuda())
    beta = (rng.normal(0, 0.1, (B, p + q)) * (rng.random((B, p + q)) < 0.7)).astype(np.float32)
    loss, grad = cox.loss_grad(torch.from_numpy(beta).cuda())
    grad = grad.cpu().numpy()
    Xs = (d.G.astype(np.float64) - d.mu[:, None].astype(np.float64)) * d.s[:, None].astype(np.float64)
    full = np.concatenate([Xs, Z.astype(np.float64)])
    M = oracle.Matrix.dense(full)
    for b in range(B):
        negL, gl = oracle.loss_grad(M, d.time, d.event, beta[b].astype(np.float64))
        assert loss[b] == pytest.approx(negL, rel=1e-12), b
        r = oracle.loglik(full.T @ beta[b].astype(np.float64), d.time, d.event)[1]
        tol = 2.0**-23 * np.abs(gl) + 1e-12 * n
        tol[:p] += np.abs(Xs).sum(axis=1) * np.abs(r).max() * 2.0**-23
        assert (np.abs(grad[b] + gl) <= tol).all(), (b, np.abs(grad[b] + gl).max())


@pytest.mark.parametrize("n,p,B,bad", [(33000, 130, 64, (5, 40)), (700, 300, 20, (0,)), (513, 63, 33, (32, 31)),
                                       (131100, 65, 16, (15,))])
def test_dense_product_keeps_nonfinite_vectors_apart(n, p, B, bad):
    """A vector with a NaN or an infinity makes the call return NUMERIC; the loss and
    gradient of every other vector, which the call has written all the same, equal those of a
    clean call bit for bit, in each launch of 32 vectors (blocks of 256 subjects) or 16
    (blocks of 512)."""
    d = coxsim.genotype_problem(n, p, 4, 0.5, 8200 + n, days=True)
    cox, _ = device_problem(d, "fp8", ldx=(n + 15) // 16 * 16, max_batch=B)
    rng = np.random.Generator(np.random.PCG64(n + p))
    beta = torch.from_numpy((0.1 * rng.normal(size=(B, p))).astype(np.float32)).cuda()
    loss, grad = cox.loss_grad(beta)
    for k, b in enumerate(bad):
        beta[b, p // 2] = float("inf") if k else float("nan")
    got, ggot = np.zeros(B), torch.zeros_like(beta)
    st = P.lib().cox_loss_grad(cox._h, beta.data_ptr(), B, P._np_ptr(got), ggot.data_ptr())
    assert st == P.ERR_NUMERIC and not np.isfinite(got[list(bad)]).any()
    good = np.setdiff1d(np.arange(B), bad)
    _bits(got[good], loss[good])
    _bits(ggot.cpu().numpy()[good], grad.cpu().numpy()[good])


@pytest.mark.parametrize("n,M", [(3000, 257), (20000, 300), (30000, 384), (45000, 385), (9000, 400), (40000, 130)])
def test_refit_gram_tiles(n, M):
    """The Gram terms' four kinds of 128 x 128 tiles side by side (full ones off the
    diagonal from 257 columns on, a last column of tiles of 1 to 128 columns, those on the
    diagonal) at two to about forty chunks of rows each, for both terms (event times
    without ties).  At the refit's coefficients a Newton step of the same equations in
    NumPy's FP64 is no longer than the refit tests' 1e-8, and the errors are the root of
    that information's inverse to 1e-8."""
    rng = np.random.Generator(np.random.PCG64(19 * n + M))
    X = rng.normal(size=(M, n)).astype(np.float32)
    eta = 0.3 * X[:5].sum(axis=0)
    time = rng.exponential(np.exp(-eta))
    event = (rng.random(n) < 0.7).astype(np.int32)
    ldx = (n + 15) // 16 * 16
    Xd = torch.zeros((M, ldx), dtype=torch.float32)
    Xd[:, :n] = torch.from_numpy(X)
    cox = P.Cox(Xd.cuda(), time, event, n=n)
    coef, se, _, L, _, st = cox.refit(np.arange(M), gtol=1e-7)
    assert st == P.OK
    order = np.argsort(-time, kind="stable")
    D, ev = X[:, order].astype(np.float64), event[order].astype(np.float64)
    w = np.exp(coef @ D)
    W = np.cumsum(w)
    wc = w * np.cumsum((ev / W)[::-1])[::-1]
    at = ev > 0
    mean = (np.cumsum(D * w, axis=1) / W)[:, at]
    H = (D * wc) @ D.T - mean @ mean.T
    step = np.linalg.solve(H, D @ (ev - wc))
    assert np.abs(step).max() <= 1e-8 * np.abs(coef).max()
    np.testing.assert_allclose(se, np.sqrt(np.diag(np.linalg.inv(H))), rtol=1e-8)
    assert L == pytest.approx((np.log(w[at]) - np.log(W[at])).sum(), rel=1e-11)


@pytest.mark.parametrize("storage,B", [("f32", 8), ("f32", 9), ("f32", 16), ("f32", 23), ("f32", 64), ("int8", 20)])
def test_vector_eta_update_groups(storage, B):
    """The vector form's eta update takes every full group of 8 vectors in one launch, a rest
    of 1 to 7 in another; with tolerances that stop vectors at different steps, groups whose
    vectors have all stopped among them.  Each vector's fit is its own: it matches the same
    fit alone, whose FP64 sums differ in their order only (1e-11 of the largest
    coefficient over the steps), up to the FP32 rounding of the result."""
    n, p = 1500, 300
    rng = np.random.Generator(np.random.PCG64(900 + B))
    if storage == "f32":
        X = rng.normal(size=(p, n)).astype(np.float32)
    else:
        X = rng.integers(-3, 4, size=(p, n)).astype(np.int8)  # not allele counts: the vector form
    time = rng.exponential(np.exp(-0.2 * X[:4].sum(axis=0).astype(np.float64)))
    event = (rng.random(n) < 0.6).astype(np.int32)
    xtype = P.X_F32 if storage == "f32" else P.X_INT8
    Xd = torch.from_numpy(X).cuda()
    cox = P.Cox(Xd, time, event, xtype=xtype, n=n, max_batch=B)
    one = P.Cox(Xd, time, event, xtype=xtype, n=n, max_batch=1)
    step = 1.0 / (2.0 * cox.opnorm2()[0])
    lams = coxsim.lambda_grid(cox.lambda_max(), B, 0.05)
    beta, iters, obj, _ = cox.fit_path(lams, max_iter=40, tol=1e-4, lag=2, step=step)
    beta = beta.cpu().numpy()
    assert len(set(np.asarray(iters).tolist())) > 1 or B < 16
    for b in range(B):
        alone, it, f, _ = one.fit_path([lams[b]], max_iter=40, tol=1e-4, lag=2, step=step)
        alone = alone.cpu().numpy()[0]
        assert it[0] == iters[b], b
        assert (np.abs(beta[b] - alone) <= 2.0**-23 * np.abs(alone) + 1e-11 * np.abs(alone).max()).all(), b
        assert obj[b] == pytest.approx(f[0], rel=1e-12), b
