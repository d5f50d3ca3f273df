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
