"""Which route a batch takes, by teams or in lockstep, and what must not depend on it (GPU;
through the C ABI).  Z is the same bit for bit on both; a call by teams launches no graph."""
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


def _by_teams(zf):
    return zf.batched_last_stats()[1] == 0


def _overlap(n, seed, sigma=1.1):
    return torch.from_numpy(inputs.overlap_gaussian(n, sigma, seed)).cuda()


@pytest.mark.parametrize("guess", ["identity", "learned"])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_results_over_guesses(zf, guess, shift):
    """The results replace the guesses, each its own or in another order: a batch whose results
    are other matrices' guesses gives what it gives with results of their own."""
    zf.mlp_set_params([0.0] * zf.N_PARAMS)
    zf.mlp_set_norm([0.0] * 8, [1.0] * 8, [2.2, -2.0, 0.9], [1.0] * 3)
    count, n = 12, 150
    S = [_overlap(n, i) for i in range(count)]
    Z0 = [torch.eye(n, dtype=torch.float64, device="cuda") / s.abs().sum(1).max().sqrt()
          for s in S]
    for i, z in enumerate(Z0):
        z[0, 1] += 1e-3 * (i + 1)
    given = [None if guess == "learned" and i % 4 == 2 else z for i, z in enumerate(Z0)]
    want = [r.Z.clone() for r in zf.refine_batched(S, given, guess=guess).results]
    assert _by_teams(zf)
    out = [Z0[(i + shift) % count] for i in range(count)]
    zf.refine_batched(S, given, guess=guess, out=out)
    assert _by_teams(zf) == (shift == 0)
    for a, b in zip(want, out):
        assert torch.equal(a, b)


def test_results_over_inputs(zf):
    """A result written over another matrix's S, or over a part of it, and one over its own."""
    S = [_overlap(n, n) for n in (65, 128, 200, 256)]
    want = [r.Z.clone() for r in zf.refine_batched(S).results]
    s = [x.clone() for x in S]
    out = [s[1].view(-1)[100:100 + 65 * 65].view(65, 65), torch.empty_like(s[1]), s[2],
           torch.empty_like(s[3])]
    zf.refine_batched(s, out=out)
    assert not _by_teams(zf)
    for a, b in zip(want, out):
        assert torch.equal(a, b)
    s = [x.clone() for x in S]
    zf.refine_batched(s, out=s)
    assert _by_teams(zf)
    for a, b in zip(want, s):
        assert torch.equal(a, b)


def test_calls_after_a_late_team(zf, monkeypatch):
    """After a late team the next calls go by launches, then teams are tried again; the
    factors are the same throughout, in batches and in single solves."""
    S = [_overlap(n, n) for n in (129, 200, 256)]
    want = [r.Z.clone() for r in zf.refine_batched(S).results]
    assert _by_teams(zf)
    single = zf.refine(S[2])
    monkeypatch.setenv("ZF_TEAM_REST", "3")
    monkeypatch.setenv("ZF_TEAM_SPIN", "0")
    late = [zf.refine_batched(S), zf.refine(S[2])]
    monkeypatch.delenv("ZF_TEAM_SPIN")
    teams = []
    for _ in range(5):
        r = zf.refine_batched(S)
        teams.append(_by_teams(zf))
        late += [r, zf.refine(S[2])]
    assert teams == [False, False, False, True, True]
    for r in late:
        if isinstance(r, zf.Refined):
            assert torch.equal(r.Z, single.Z) and r.iters == single.iters
        else:
            assert all(torch.equal(a.Z, b) for a, b in zip(r.results, want))


@pytest.mark.parametrize("guess", ["identity", "learned"])
def test_tile_table_is_for_lockstep(zf, monkeypatch, guess):
    """Teams do not use the table: equal bits, norms included, whatever it says, also where
    the order is just past a multiple of 64.  In lockstep every edge runs, and agrees in Z."""
    zf.mlp_set_params([0.0] * zf.N_PARAMS)
    zf.mlp_set_norm([0.0] * 8, [1.0] * 8, [2.2, -2.0, 0.9], [1.0] * 3)
    S = [_overlap(n, n) for n in (1, 63, 65, 128, 129, 257, 300, 385, 512)]
    saved = zf.batched_get_tiles()
    runs = {}
    try:
        for limit in ("512", "0"):
            monkeypatch.setenv("ZF_TEAM_BATCH_MAX", limit)
            for edge in (64, 128):
                zf.batched_set_tiles([1 << 20], [edge])
                runs[limit, edge] = zf.refine_batched(S, guess=guess).results
                assert _by_teams(zf) == (limit == "512")
    finally:
        zf.batched_set_tiles(*saved)
    for a, b in zip(runs["512", 64], runs["512", 128]):
        assert a.hist == b.hist
    for r in runs.values():
        for a, b in zip(runs["512", 64], r):
            assert torch.equal(a.Z, b.Z) and a.iters == b.iters


@pytest.mark.parametrize("orders,teams", [([512] * 8, True), ([384] * 32, True), ([513] + [100] * 8, False),
                                          ([512] * 48, False), ([384] * 64, False),
                                          ([300] * 64, True), ([385] * 40 + [200] * 100, True)])
def test_route_by_work(zf, orders, teams):
    """Few orders above 320 go by teams, many in lockstep, where the wider tiles pay."""
    made = {n: _overlap(n, n) for n in set(orders)}
    out = zf.refine_batched([made[n] for n in orders], refine="off")
    assert _by_teams(zf) == teams
    for n, r in zip(orders, out.results):
        assert torch.equal(r.Z, out.results[orders.index(n)].Z)
