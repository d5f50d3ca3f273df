"""Overflow in the products of a residual (GPU; through the C ABI): the norm of elements that
are infinite is infinite, not NaN, in the symmetric mode too, which leaves out the elements
below the diagonal of a diagonal block."""
import math

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


@pytest.mark.parametrize("prec", ["bf16x3", "bf16", "fp32"])
@pytest.mark.parametrize("n", [1, 33, 200])
def test_norm_of_infinite_products(zf, prec, n):
    """Elements 2^66, exact in every format: each product is beyond the FP32 range."""
    A = torch.full((n, 40), 2.0 ** 66, dtype=torch.float64, device="cuda")
    C, s = zf.t_gemm(prec, A, A, sym=True, kblocked=prec != "fp32")
    assert bool((C == math.inf).all())
    assert s == math.inf


@pytest.mark.parametrize("n", [100, 400])
def test_history_of_an_overflow(zf, n):
    """A guess of 2^70 I: ||Z0^T S Z0 - I|| overflows FP32 in the first evaluation."""
    S = torch.full((n, n), 0.5, dtype=torch.float64, device="cuda")
    S.fill_diagonal_(1.0)
    Z0 = torch.eye(n, dtype=torch.float64, device="cuda") * 2.0 ** 70
    out = zf.refine_batched([S], [Z0], raise_on_error=False)
    assert out.rc == zf.ERR_NONFINITE
    assert out.results[0].hist == [math.inf]


@pytest.mark.parametrize("kw", [dict(), dict(refine="off"), dict(precision="fp64", refine="off")])
def test_message_of_a_failed_solve(zf, monkeypatch, kw):
    """The one-kernel solve names the arithmetic and the sweep as separate launches do."""
    S = torch.eye(90, dtype=torch.float64, device="cuda")
    S[4, 7] = S[7, 4] = float("nan")
    said = []
    for limit in ("0", "320"):
        monkeypatch.setenv("ZF_TEAM_MAX", limit)
        with pytest.raises(zf.ZFError) as e:
            zf.refine(S, **kw)
        assert e.value.code == zf.ERR_NONFINITE
        said.append(str(e.value))
    assert said[0] == said[1]
    assert ("FP64" if "precision" in kw else "BF16x3") + " sweep 0" in said[0]
