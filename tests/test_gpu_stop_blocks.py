"""The stop test over many blocks, and the residual it reports (GPU; through the C ABI).

The last block sums the norm partials in passes of 512: forced tile edges give counts on
both sides of one and of two passes.  Err must be the norm of the residual formed on the
CPU in FP64 within the products' error, and the reported residual that of the returned Z.
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


def _blocks(n, edge):
    t = (n + 127) // 128 * 128 // edge
    if edge == 32:  # quarters of 64-wide tiles, those below the diagonal counted too
        t //= 2
        return 4 * (t * (t + 1) // 2)
    return t * (t + 1) // 2


@pytest.mark.parametrize("precision,n,edge,blocks", [
    ("fp64", 900, 32, 544), ("fp64", 1200, 32, 840), ("fp64", 1400, 32, 1012),
    ("fp64", 1500, 32, 1200), ("bf16x3", 2000, 64, 528), ("bf16x3", 2900, 64, 1081)])
def test_err_over_many_blocks(zf, monkeypatch, precision, n, edge, blocks):
    """hist[0] against the norm of I - S / g: within n u64 |S| / g for FP64 and
    (3 n u32 + 6 2^-16) |S| / g for the pairs; a second call gives the same history."""
    assert _blocks(n, edge) == blocks
    monkeypatch.setenv("ZF_F64_SYM_TILE", str(edge))
    monkeypatch.setenv("ZF_X3_SYM_TILE", str(edge))
    S = inputs.overlap_gaussian(n, 1.0, 3)
    Sd = torch.from_numpy(S).cuda()
    kw = dict(order=2, precision=precision, refine="off", max_sweeps=30)
    r = zf.refine(Sd, None, **kw)
    g = np.max(np.sum(np.abs(S), axis=1))
    ref = np.linalg.norm(np.eye(n) - S / g)
    rel = n * 2.0 ** -52 if precision == "fp64" else 3 * n * 2.0 ** -24 + 6 * 2.0 ** -16
    assert abs(r.hist[0] - ref) <= rel * np.linalg.norm(np.abs(S)) / g + 1e-13 * ref
    assert list(zf.refine(Sd, None, **kw).hist) == list(r.hist)


@pytest.mark.parametrize("precision", ["fp64", "bf16x3"])
@pytest.mark.parametrize("n", [200, 700])
@pytest.mark.parametrize("max_sweeps", [3, 4, 30])
def test_reported_residual_is_the_results(zf, n, precision, max_sweeps):
    """The reported RMS is that of the Z returned, capped (above the rounding floor) or
    stopped, with the last iterate or the one before: within the evaluation's own error,
    2 n u64 sqrt(n) for FP64 and, above it for the pairs, (3 n u32 + 6 2^-16) sqrt(n)
    (|Z^T S Z| is close to I)."""
    S = inputs.overlap_gaussian(n, 1.0, 5)
    r = zf.refine(torch.from_numpy(S).cuda(), None, precision=precision, refine="off",
                  max_sweeps=max_sweeps)
    Z = r.Z.cpu().numpy()
    err = np.linalg.norm(Z.T @ S @ Z - np.eye(n)) / np.sqrt(n)
    u = 2 * n * 2.0 ** -53 if precision == "fp64" else 3 * n * 2.0 ** -24 + 6 * 2.0 ** -16
    scale = np.linalg.norm(np.abs(Z).T @ np.abs(S) @ np.abs(Z)) / np.sqrt(n)
    assert abs(r.final_rms - err) <= u * scale
