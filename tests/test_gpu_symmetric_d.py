"""Symmetric mode with a D that is not symmetric (GPU; through the C ABI): C is formed above
the diagonal and mirrored, so only D's upper triangle counts, in every arithmetic."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_19163_amd import zf as _zf
    _zf.lib()
    return _zf


@pytest.mark.parametrize("prec", ["bf16x3", "bf16", "fp32", "fp64", "emu", "crt"])
@pytest.mark.parametrize("n", [1, 33, 200])
def test_upper_triangle_of_d_counts(zf, prec, n):
    rng = np.random.default_rng(n)
    A = torch.from_numpy(rng.standard_normal((n, 40))).cuda()
    D = rng.standard_normal((n, n))
    up = np.triu(D) + np.triu(D, 1).T
    kw = dict(sym=True, alpha=0.5, beta=-1.5, gamma=0.25)
    if prec in ("emu", "crt"):
        kw["slices"] = 7 if prec == "emu" else 14
    C, s = zf.t_gemm(prec, A, A, D=torch.from_numpy(D).cuda(), **kw)
    U, t = zf.t_gemm(prec, A, A, D=torch.from_numpy(up).cuda(), **kw)
    assert torch.equal(C, C.T) and torch.equal(C, U) and s == t
