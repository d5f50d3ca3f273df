"""Padding, transposing, splitting and unpadding of the operands (GPU).

Integer matrices small enough that every product and sum is exact in each arithmetic
(entries of magnitude <= 3, sums below 2^16): the results must equal the integers.  Orders
around the 8-row, 32-, 64- and 128-column pieces the kernels move, and operands whose first
element is only 8-byte aligned.
"""
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


def _cuda(a, offset):
    """A contiguous CUDA copy that starts `offset` elements into its storage."""
    buf = torch.zeros(a.size + offset, dtype=torch.float64, device="cuda")
    v = buf[offset:].view(*a.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    return v


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("n", [1, 5, 31, 33, 64, 127, 130, 257, 1025])
def test_congruence_of_integers_is_exact(zf, precision, n, offset):
    rng = np.random.default_rng(n)
    Z = rng.integers(-3, 4, (n, n)) * (rng.random((n, n)) < min(1.0, 40.0 / n))
    H = np.diag(rng.integers(-3, 4, n))
    H[0, n - 1] = H[n - 1, 0] = 2
    ref = (Z.T @ H @ Z).astype(np.float64)
    got = zf.congruence(_cuda(H.astype(np.float64), offset), _cuda(Z.astype(np.float64), offset),
                        precision=precision)
    assert np.array_equal(got.cpu().numpy(), ref)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", [1, 31, 33, 64, 127, 200, 1000])
def test_residual_of_integers(zf, n, offset):
    """The residual's sum of squares is an exact integer: one square root and one division."""
    rng = np.random.default_rng(n)
    Z = np.eye(n) + np.roll(np.diag(rng.integers(-2, 3, n)), 1, axis=1)
    S = np.diag(rng.integers(1, 4, n)).astype(np.float64)
    ref = np.sqrt(np.sum((np.eye(n) - Z.T @ S @ Z) ** 2)) / np.sqrt(n)
    Sd, Zd = _cuda(S, offset), _cuda(Z, offset)
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    zf.residual_noalloc(Sd, Zd, out)
    assert out.item() == pytest.approx(ref, rel=1e-15)
    assert zf.residual(Sd, Zd) == out.item()
