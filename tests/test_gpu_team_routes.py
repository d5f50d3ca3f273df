"""Where the one-kernel path of small orders ends (GPU; through the C ABI): the last order
that it takes and the first that goes by launches, in each arithmetic, give the Z of both
routes bit for bit, so the line may lie wherever the measured times put it."""
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


@pytest.mark.parametrize("last,kw", [(192, dict(precision="fp64", refine="off")),
                                     (256, dict()), (320, dict(refine="off"))])
def test_the_line(zf, monkeypatch, last, kw):
    for n in (last, last + 1):
        S = torch.from_numpy(inputs.overlap_gaussian(n, 1.1, n)).cuda()
        monkeypatch.delenv("ZF_TEAM_MAX", raising=False)
        r = zf.refine(S, **kw)
        for limit in ("0", "512"):
            monkeypatch.setenv("ZF_TEAM_MAX", limit)
            q = zf.refine(S, **kw)
            assert torch.equal(q.Z, r.Z) and q.iters == r.iters and len(q.hist) == len(r.hist)
