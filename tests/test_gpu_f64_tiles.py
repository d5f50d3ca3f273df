"""Tile edges of the FP64 matrix-core GEMM (GPU; through the C ABI).

The products of an output element run in ascending K on either tile edge, so the 32- and
the 64-wide tile must agree bit for bit, and both must meet the dot-product bound
|C - C_ref| <= 2 K u (|A||B|^T) + 2 u |C_ref|, u = 2^-53, against the plain product.
"""
import numpy as np
import pytest
import torch

from oracle import zf_oracle as O
from paper_2404_19163_amd import inputs

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def zf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_19163_amd import zf as _zf
    _zf.lib()
    return _zf


@pytest.mark.parametrize("sym", [False, True])
@pytest.mark.parametrize("m,nn,k", [(1, 1, 1), (31, 33, 65), (257, 255, 511), (640, 640, 100)])
def test_edges_agree(zf, monkeypatch, m, nn, k, sym):
    rng = np.random.default_rng(m + 3 * nn + k)
    A = rng.standard_normal((m, k))
    B = A if sym else rng.standard_normal((nn, k))
    ref = A @ B.T
    bound = 2 * k * U64 * (np.abs(A) @ np.abs(B).T) + 2 * U64 * np.abs(ref)
    Ad, Bd = (torch.from_numpy(x).cuda() for x in (A, B))
    out = {}
    for tile in ("32", "64"):
        monkeypatch.setenv("ZF_F64_TILE", tile)
        monkeypatch.setenv("ZF_F64_SYM_TILE", tile)
        out[tile], s = zf.t_gemm("fp64", Ad, Bd, sym=sym)
        assert np.all(np.abs(out[tile].cpu().numpy() - ref) <= bound)
        assert s == pytest.approx(np.sum(ref * ref), rel=1e-12)
    assert torch.equal(out["32"], out["64"])


@pytest.mark.parametrize("m,nn,sym", [(1200, 1200, False), (1500, 1500, True), (1030, 1290, False),
                                      (2500, 2500, True), (1100, 1100, True)])
def test_quartered_rest_agrees(zf, monkeypatch, m, nn, sym):
    """Grids with a rest beyond full rounds over the CUs (quartered or, beyond 192 tiles, not):
    the same elements, bit for bit, as 64-wide tiles alone, and a norm of each once."""
    rng = np.random.default_rng(m + nn)
    A = torch.from_numpy(rng.standard_normal((m, 70))).cuda()
    B = A if sym else torch.from_numpy(rng.standard_normal((nn, 70))).cuda()
    C, s = zf.t_gemm("fp64", A, B, sym=sym)
    monkeypatch.setenv("ZF_F64_TILE", "64")
    monkeypatch.setenv("ZF_F64_SYM_TILE", "64")
    C64, s64 = zf.t_gemm("fp64", A, B, sym=sym)
    assert torch.equal(C, C64)
    assert s == pytest.approx(s64, rel=1e-12)


@pytest.mark.parametrize("n", [1, 63, 64, 65])
def test_shortest_contraction(zf, n):
    """One and two 64-wide tiles in the batched path: the shortest K the ring runs."""
    S = inputs.overlap_gaussian(n, 1.0, n)
    r = zf.refine_batched([torch.from_numpy(S).cuda()]).results[0]
    assert O.residual_rms(S, r.Z.cpu().numpy()) < 1e-8
