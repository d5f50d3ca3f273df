"""One-kernel refinement of small orders (GPU; through the C ABI).

A team of workgroups runs the whole solve with the arithmetic of the separate launches, so
Z must be the same bit for bit, with the same sweep counts; residual norms are sums of the
same squares in another order (relative difference below 2^-53 times a few hundred terms,
held to 1e-12 above the FP64 floor).
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


def _same(a, b):
    assert torch.equal(a.Z, b.Z)
    assert (a.iters, a.low_evals, a.high_evals, a.flags, a.z0_used) == \
        (b.iters, b.low_evals, b.high_evals, b.flags, b.z0_used)
    assert len(a.hist) == len(b.hist)
    for x, y in zip(a.hist, b.hist):
        assert x == pytest.approx(y, rel=1e-12, abs=1e-24)


@pytest.mark.parametrize("n", [1, 31, 64, 65, 129, 192, 256, 257, 320])
@pytest.mark.parametrize("prec,ref,order,stop", [
    ("bf16x3", "f64_delta", 2, "ratio"), ("bf16x3", "off", 1, "ratio"),
    ("bf16x3", "f64_delta", 5, "monotone"), ("fp64", "off", 3, "ratio"), ("fp64", "off", 1, "ratio")])
def test_equals_separate_launches(zf, monkeypatch, n, prec, ref, order, stop):
    S = torch.from_numpy(inputs.overlap_gaussian(n, 1.1, n)).cuda()
    kw = dict(precision=prec, refine=ref, order=order, stop=stop, max_sweeps=30)
    Z0 = None
    if order == 2:  # a given, unsymmetric start
        rng = np.random.default_rng(n)
        g = S.abs().sum(1).max().item()
        Z0 = torch.eye(n, dtype=torch.float64, device="cuda") / g ** 0.5
        Z0 += 1e-4 * torch.from_numpy(rng.standard_normal((n, n))).cuda()
    monkeypatch.setenv("ZF_TEAM_MAX", "0")
    a = zf.refine(S, Z0, **kw)
    monkeypatch.setenv("ZF_TEAM_MAX", "320")
    _same(a, zf.refine(S, Z0, **kw))


def test_sweep_caps(zf, monkeypatch):
    S = torch.from_numpy(inputs.overlap_gaussian(100, 1.1, 0)).cuda()
    kw = dict(max_sweeps=5, max_refine=1, stop="monotone")
    monkeypatch.setenv("ZF_TEAM_MAX", "0")
    a = zf.refine(S, **kw)
    monkeypatch.setenv("ZF_TEAM_MAX", "320")
    _same(a, zf.refine(S, **kw))


def test_gives_up_waiting(zf, monkeypatch):
    """With no time to wait the team leaves and the solve runs by launches; Z may alias Z0."""
    S = torch.from_numpy(inputs.overlap_gaussian(200, 1.1, 3)).cuda()
    Z0 = torch.eye(200, dtype=torch.float64, device="cuda") / S.abs().sum(1).max().sqrt()
    monkeypatch.setenv("ZF_TEAM_MAX", "0")
    a = zf.refine(S, Z0)
    monkeypatch.setenv("ZF_TEAM_MAX", "320")
    for spin in ("0", "100", "20000000"):
        monkeypatch.setenv("ZF_TEAM_SPIN", spin)
        out = Z0.clone()
        _same(a, zf.refine(S, out, out=out))


def test_not_finite(zf):
    S = torch.from_numpy(inputs.overlap_gaussian(90, 1.1, 3)).cuda()
    S[4, 7] = S[7, 4] = float("nan")
    with pytest.raises(zf.ZFError) as e:
        zf.refine(S)
    assert e.value.code == zf.ERR_NONFINITE
