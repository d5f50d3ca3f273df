"""Tile edges and ring depths of the 16-bit-pair GEMM (GPU; through the C ABI).

Per output element every tile runs the same products in the same order (16-wide K steps;
(h)(h), (h)(l), (l)(h) in each), so all tile edges must agree bit for bit.  The 64-wide
tile takes a two-stage ring from 513 to 1024 blocks and a four-stage ring otherwise; the
orders below cover both, in full and symmetric mode, and the shortest contraction
(np = 256) of each ring.  The norms are FP64 sums over different block partials.
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


@pytest.mark.parametrize("prec", ["bf16x3", "bf16", "fp16x3", "fp16"])
@pytest.mark.parametrize("n,sym", [(200, False), (200, True), (1500, False), (2048, True)])
def test_edges_agree_bitwise(zf, monkeypatch, prec, n, sym):
    rng = np.random.default_rng(n)
    A = torch.from_numpy(rng.standard_normal((n, 70))).cuda()
    B = A if sym else torch.from_numpy(rng.standard_normal((n, 70))).cuda()
    out = {}
    for tile in ("64", "128", "256"):
        monkeypatch.setenv("ZF_X3_TILE", tile)
        monkeypatch.setenv("ZF_X3_SYM_TILE", tile)
        out[tile] = zf.t_gemm(prec, A, B, sym=sym, kblocked=True)
    for tile in ("128", "256"):
        assert torch.equal(out[tile][0], out["64"][0])
        assert out[tile][1] == pytest.approx(out["64"][1], rel=1e-12)


@pytest.mark.parametrize("tile", ["64", "128", "256"])
@pytest.mark.parametrize("n", [1, 31, 33, 65, 260])
def test_symmetric_epilogue(zf, monkeypatch, tile, n):
    """alpha D + beta A A^T + gamma I around the diagonal blocks: exactly symmetric, within
    the split product's bound 3 K u32 (|A_h| + |A_l|)(|A_h| + |A_l|)^T plus its 3 u^2 |A||A|^T
    (u = 2^-8), and a norm that counts every element once."""
    monkeypatch.setenv("ZF_X3_SYM_TILE", tile)
    rng = np.random.default_rng(n)
    k = 48
    A = rng.standard_normal((n, k))
    D = rng.standard_normal((n, n))
    D = D + D.T
    al, be, ga = 0.75, -1.25, 2.0
    C, s = zf.t_gemm("bf16x3", torch.from_numpy(A).cuda(), torch.from_numpy(A).cuda(), sym=True,
                     alpha=al, D=torch.from_numpy(D).cuda(), beta=be, gamma=ga, kblocked=True)
    C = C.cpu().numpy()
    assert np.array_equal(C, C.T)
    ref = al * D + be * (A @ A.T) + ga * np.eye(n)
    absx = np.abs(A) @ np.abs(A).T
    bound = abs(be) * (3 * 2.0 ** -16 + 3 * k * 2.0 ** -24 * 1.02) * absx * 1.01 + 1e-14
    assert np.all(np.abs(C - ref) <= bound)
    assert s == pytest.approx(np.sum(C * C), rel=1e-12)


@pytest.mark.parametrize("prec", ["bf16x3", "bf16", "fp16x3"])
@pytest.mark.parametrize("n,k,sym", [(190, 40, True), (200, 128, False), (200, 40, True),
                                     (330, 180, True), (580, 250, False), (580, 70, True),
                                     (1100, 40, False), (2048, 390, True)])
def test_192_wide_edge_agrees_bitwise(zf, monkeypatch, prec, n, k, sym):
    """The 192-wide tile need not divide the padded order: its last row and column of tiles
    move back inside the matrix and leave the other tiles' blocks alone.  Remainders of 0, 64
    and 128, contractions from the shortest (64), with D, both layouts and the norm, each
    element counted once."""
    rng = np.random.default_rng(n)
    A = torch.from_numpy(rng.standard_normal((n, k))).cuda()
    B = A if sym else torch.from_numpy(rng.standard_normal((n, k))).cuda()
    D = rng.standard_normal((n, n))
    D = torch.from_numpy(D + D.T).cuda()
    out = {}
    for tile in ("64", "192"):
        monkeypatch.setenv("ZF_X3_TILE", tile)
        monkeypatch.setenv("ZF_X3_SYM_TILE", tile)
        out[tile] = zf.t_gemm(prec, A, B, sym=sym, alpha=0.5, D=D, beta=-1.5, gamma=0.25,
                              kblocked=True)
    assert torch.equal(out["192"][0], out["64"][0])
    assert out["192"][1] == pytest.approx(out["64"][1], rel=1e-12)


@pytest.mark.parametrize("n,sym", [(200, False), (200, True), (1500, True), (2048, False)])
def test_fp32_edges_agree_bitwise(zf, monkeypatch, n, sym):
    """The FP32 products of an element run in one order on every tile edge, the chosen one
    included."""
    rng = np.random.default_rng(n)
    A = torch.from_numpy(rng.standard_normal((n, 70))).cuda()
    B = A if sym else torch.from_numpy(rng.standard_normal((n, 70))).cuda()
    out = [zf.t_gemm("fp32", A, B, sym=sym)]
    for tile in ("64", "128", "256"):
        monkeypatch.setenv("ZF_X3_TILE", tile)
        monkeypatch.setenv("ZF_X3_SYM_TILE", tile)
        out.append(zf.t_gemm("fp32", A, B, sym=sym))
    for C, s in out[1:]:
        assert torch.equal(C, out[0][0])
        assert s == pytest.approx(out[0][1], rel=1e-12)
