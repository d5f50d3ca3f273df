"""The stop test run by the last block of the residual product (GPU).

Err is the norm of the FP64 partials of every block, summed in one fixed order whatever
block comes last: equal inputs give equal bits.  The orders below have from 21 to 1275
blocks, both sides of the 512 that one pass of the summing wave covers.
"""
import numpy as np
import pytest
import torch

from paper_2404_19163_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_19163_amd import zf as _zf
    _zf.lib()
    return _zf


@pytest.mark.parametrize("precision,n", [("fp64", 330), ("fp64", 1000), ("fp64", 1500),
                                         ("bf16x3", 330), ("bf16x3", 1000), ("bf16x3", 2100)])
def test_err_is_the_norm_in_one_order(zf, precision, n):
    """hist[0] against the norm of I - S / g, formed on the CPU in FP64: within the products'
    error, n u64 |S| / g for FP64 and (3 n u32 + 3 2^-16) |S| / g for the pairs, plus the
    pairs' own rounding 2^-16; a second call gives the same history."""
    S = inputs.overlap_gaussian(n, 1.0, 3)
    kw = dict(order=2, precision=precision, refine="off")
    Sd = torch.from_numpy(S).cuda()
    r = zf.refine(Sd, None, **kw)
    g = np.max(np.sum(np.abs(S), axis=1))
    ref = np.linalg.norm(np.eye(n) - S / g)
    rel = n * 2.0 ** -52 if precision == "fp64" else 3 * n * 2.0 ** -24 + 6 * 2.0 ** -16
    assert abs(r.hist[0] - ref) <= rel * np.linalg.norm(np.abs(S)) / g + 1e-13 * ref
    assert list(zf.refine(Sd, None, **kw).hist) == list(r.hist)
    if precision == "fp64":
        assert r.final_rms in (zf.residual(Sd, r.Z), r.hist[-2] / np.sqrt(n))


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n", [200, 700])
def test_residual_of_bad_values(zf, n, bad):
    S = torch.eye(n, dtype=torch.float64, device="cuda")
    Z = S.clone()
    assert zf.residual(S, Z) == 0.0
    Z[n // 2, 3] = bad
    assert not np.isfinite(zf.residual(S, Z))
    Z[n // 2, 3] = 0.0
    assert zf.residual(S, Z) == 0.0
