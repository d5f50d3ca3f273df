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


ORDERS = [1, 40, 64, 65, 100, 129, 192, 200, 256, 300, 385, 512]


def _batch(seed, orders=ORDERS):
    return [torch.from_numpy(inputs.overlap_gaussian(n, 1.0 + 0.02 * i, seed + i)).cuda()
            for i, n in enumerate(orders)]


def _same_batch(a, b):
    assert a.rc == b.rc
    for x, y in zip(a.results, b.results):
        assert (x.status, x.flags) == (y.status, y.flags)
        _same(x, y)


@pytest.mark.parametrize("guess,ref,stop", [("identity", "f64_delta", "ratio"),
                                            ("learned", "f64_delta", "ratio"),
                                            ("identity", "off", "monotone")])
def test_batch_equals_macro_sweeps(zf, monkeypatch, guess, ref, stop):
    """Teams and lockstep macro-sweeps; matrix 3 starts from a given guess."""
    if guess == "learned":
        zf.mlp_set_params([0.0] * zf.N_PARAMS)
        zf.mlp_set_norm([0.0] * 8, [1.0] * 8, [2.2, -2.0, 0.9], [1.0] * 3)
    S = _batch(1)
    Z0 = [None] * len(S)
    Z0[3] = torch.eye(65, dtype=torch.float64, device="cuda") / S[3].abs().sum(1).max().sqrt()
    Z0[3][0, 1] += 1e-3
    kw = dict(guess=guess, refine=ref, stop=stop, max_sweeps=20)
    monkeypatch.setenv("ZF_TEAM_BATCH_MAX", "0")
    a = zf.refine_batched(S, Z0, **kw)
    monkeypatch.setenv("ZF_TEAM_BATCH_MAX", "512")
    _same_batch(a, zf.refine_batched(S, Z0, **kw))
    assert zf.batched_last_stats()[1] == 0  # no graph was launched


@pytest.mark.parametrize("guess", ["identity", "learned"])
def test_batch_gives_up_waiting(zf, monkeypatch, guess):
    """Teams without time to wait: their matrices, aliased guesses included, run by
    macro-sweeps, the one-member teams' do not."""
    zf.mlp_set_params([0.0] * zf.N_PARAMS)
    zf.mlp_set_norm([0.0] * 8, [1.0] * 8, [2.2, -2.0, 0.9], [1.0] * 3)
    S = _batch(7)
    Z0 = [torch.eye(s.shape[0], dtype=torch.float64, device="cuda") / s.abs().sum(1).max().sqrt()
          if i % 2 else None for i, s in enumerate(S)]
    monkeypatch.setenv("ZF_TEAM_BATCH_MAX", "0")
    a = zf.refine_batched(S, Z0, guess=guess)
    monkeypatch.setenv("ZF_TEAM_BATCH_MAX", "512")
    for spin in ("0", "300", "20000000"):
        monkeypatch.setenv("ZF_TEAM_SPIN", spin)
        out = [torch.empty_like(s) if z is None else z.clone() for s, z in zip(S, Z0)]
        z0 = [None if z is None else o for z, o in zip(Z0, out)]
        _same_batch(a, zf.refine_batched(S, z0, guess=guess, out=out))


def test_batch_error_isolated(zf):
    S = _batch(11, [100, 90, 300])
    S[1][2, 3] = S[1][3, 2] = float("nan")
    out = zf.refine_batched(S, raise_on_error=False)
    assert out.rc == zf.ERR_NONFINITE
    assert [r.status for r in out.results] == [0, zf.ERR_NONFINITE, 0]
