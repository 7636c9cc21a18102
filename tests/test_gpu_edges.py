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
