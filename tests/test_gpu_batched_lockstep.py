"""Small orders on both routes of the batched path, by teams and in lockstep macro-sweeps
(GPU; through the C ABI).  By default small batches go by teams, so what is to run in
lockstep is sent there (ZF_TEAM_BATCH_MAX=0), and each test says which route ran.

Bars as in test_gpu_batched: oracle-measured RMS residual at most 1e-6 with the FP64
refinement phase, ||Z - Z_oracle|| / ||Z_oracle|| at most 1e-4.
"""
import numpy as np
import pytest
import torch

from oracle import zf_oracle as O
from paper_2404_19163_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [64, 70, 100, 128, 129, 257]


@pytest.fixture(scope="module")
def zf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_19163_amd import zf as _zf
    _zf.lib()
    return _zf


@pytest.fixture(params=["teams", "lockstep"])
def route(request, zf, monkeypatch):
    monkeypatch.setenv("ZF_TEAM_BATCH_MAX", "512" if request.param == "teams" else "0")

    def ran():
        assert (zf.batched_last_stats()[1] == 0) == (request.param == "teams")
    return ran


@pytest.fixture(scope="module")
def mats():
    rng = np.random.default_rng(5)
    out = []
    for n in SIZES:
        pos = inputs.rsa_positions(n, 0.1, 0.0, rng)
        K = inputs.gaussian_kernel_overlap(pos, 1.0)
        out.append(inputs.shift_to_condition(K, float(10 ** rng.uniform(1, 4))))
    return out


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def test_tile_edges(zf, route, mats):
    saved = zf.batched_get_tiles()
    try:
        for edge in (64, 128):
            zf.batched_set_tiles([1 << 20], [edge])
            out = zf.refine_batched([_cuda(S) for S in mats])
            route()
            for S, r in zip(mats, out.results):
                assert O.residual_rms(S, r.Z.cpu().numpy()) <= 1e-6
    finally:
        zf.batched_set_tiles(*saved)


@pytest.mark.parametrize("bad", [0, 2, 5])
def test_error_isolated(zf, route, mats, bad):
    """A NaN in one matrix, at the front, inside and at the end of the batch, fails that
    matrix and changes no bit of the others."""
    S = [_cuda(x) for x in mats]
    good = zf.refine_batched(S)
    S[bad] = S[bad].clone()
    S[bad][2, 3] = S[bad][3, 2] = float("nan")
    out = zf.refine_batched(S, raise_on_error=False)
    route()
    assert out.rc == zf.ERR_NONFINITE
    for i, (a, b) in enumerate(zip(good.results, out.results)):
        if i == bad:
            assert b.status == zf.ERR_NONFINITE
        else:
            assert b.status == 0 and torch.equal(a.Z, b.Z) and a.iters == b.iters


def test_given_guesses(zf, route, mats):
    z0 = [None if i % 2 else _cuda(O.lowdin(S) + 1e-3 * inputs.uniform_noise(S.shape[0], i))
          for i, S in enumerate(mats)]
    out = zf.refine_batched([_cuda(S) for S in mats], z0)
    route()
    for S, z, r in zip(mats, z0, out.results):
        Z = r.Z.cpu().numpy()
        assert O.residual_rms(S, Z) <= 1e-6
        if z is not None:
            assert _rel(Z, O.limit_for_guess(S, z.cpu().numpy())) <= 1e-4


def test_refine_off(zf, route, mats):
    out = zf.refine_batched([_cuda(S) for S in mats], refine="off")
    route()
    for S, r in zip(mats, out.results):
        assert O.residual_rms(S, r.Z.cpu().numpy()) < 1e-3 and r.high_evals == 0


def test_deterministic(zf, route, mats):
    S = [_cuda(x) for x in mats]
    a = zf.refine_batched(S)
    b = zf.refine_batched(S)
    route()
    for x, y in zip(a.results, b.results):
        assert torch.equal(x.Z, y.Z) and x.hist == y.hist


@pytest.mark.parametrize("n", [1, 63, 64, 65])
def test_shortest_contraction(zf, route, n):
    """Padded orders of 64 and 128: the shortest K of the teams' rings and, in lockstep, of the
    two-stage rings of the 64-wide tiles."""
    S = inputs.overlap_gaussian(n, 1.0, n)
    r = zf.refine_batched([_cuda(S)]).results[0]
    route()
    assert O.residual_rms(S, r.Z.cpu().numpy()) < 1e-8
