"""Calls on a stream of the caller's (GPU; through the C ABI).

A non-blocking stream is ordered behind nothing on the default stream.  Every entry point is
called with fresh buffers on one, while the default stream is busy, and must give what it
gives on the default stream, bit for bit.
"""
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


def _refined(r):
    return [r.Z, torch.tensor(r.hist + [r.iters, r.low_evals, r.high_evals, r.flags])]


def _batch(out):
    return [t for r in out.results for t in _refined(r)]


def _calls(zf, kind, S, stream):
    if kind == "team":
        return _refined(zf.refine(S[2], stream=stream))
    if kind == "team_fp64":
        return _refined(zf.refine(S[1], precision="fp64", refine="off", stream=stream))
    if kind == "launches":
        return _refined(zf.refine(S[4], stream=stream))
    if kind == "fp16x3":
        return _refined(zf.refine(S[3], precision="fp16x3", stream=stream))
    if kind == "batch_teams":
        return _batch(zf.refine_batched(S[:4], stream=stream))
    if kind == "batch_lockstep":
        return _batch(zf.refine_batched(S, stream=stream))
    if kind == "batch_learned":
        return _batch(zf.refine_batched(S[:4], guess="learned", stream=stream))
    Z = S[2] + torch.eye(S[2].shape[0], dtype=torch.float64, device="cuda")
    stream.synchronize() if stream is not None else None
    torch.cuda.default_stream().synchronize()
    if kind == "residual":
        return [torch.tensor(zf.residual(S[2], Z, stream=stream))]
    if kind == "residual_noalloc":
        out = torch.zeros(1, dtype=torch.float64, device="cuda")
        torch.cuda.default_stream().synchronize()
        zf.residual_noalloc(S[2], Z, out, stream=stream)
        return [out]
    return [zf.congruence(S[2], Z, stream=stream)]


@pytest.mark.parametrize("kind", ["team", "team_fp64", "launches", "fp16x3", "batch_teams",
                                  "batch_lockstep", "batch_learned", "residual",
                                  "residual_noalloc", "congruence"])
def test_side_stream(zf, kind):
    zf.mlp_set_params([0.0] * zf.N_PARAMS)
    zf.mlp_set_norm([0.0] * 8, [1.0] * 8, [2.2, -2.0, 0.9], [1.0] * 3)
    S = [torch.from_numpy(inputs.overlap_gaussian(n, 1.1, n)).cuda() for n in (40, 129, 256, 400, 600)]
    want = _calls(zf, kind, S, None)
    torch.cuda.synchronize()
    busy = torch.ones(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    zf.release()  # the next call allocates afresh
    torch.cuda.synchronize()
    for rep in range(3):
        for _ in range(20):
            busy = busy @ busy * 1e-4
        got = _calls(zf, kind, S, side)
        torch.cuda.synchronize()
        for a, b in zip(want, got):
            assert torch.equal(a, b), (kind, rep)


def test_first_congruence_in_a_graph(zf):
    """The transform is stream-ordered: its first call, which allocates, may be captured
    (capture mode relaxed), and every replay transforms what H holds then."""
    n = 200
    H = torch.from_numpy(inputs.overlap_gaussian(n, 1.1, 0)).cuda()
    Z = H + torch.eye(n, dtype=torch.float64, device="cuda")
    out = torch.empty_like(H)
    Hs = [H * k for k in (1.0, 2.0, 0.25)]
    want = [zf.congruence(h, Z).clone() for h in Hs]
    torch.cuda.synchronize()
    zf.release()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        zf.congruence(H, Z, out=out)
    for h, w in zip(Hs, want):
        H.copy_(h)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, w)
