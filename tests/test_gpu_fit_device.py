"""Codebook fit: the rounds on the running sums that the device forms against pq_fit_cluster, which forms them on the host from a
copy of the same counts, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2502_02617_amd import Context, PolarQuantError

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _vectors(kind, n, g):
    x = torch.randn((n, 2, 128), generator=g)
    if kind == "outliers":
        x[..., ::31] *= 30.0
    elif kind == "few":                       # most bins empty, the others large
        x = x[:1].expand(n, 2, 128).contiguous()
    elif kind == "zeros":
        x[n // 8:] = 0.0
    return x.bfloat16()


@pytest.mark.parametrize("kind,n", [("gauss", 3000), ("outliers", 700), ("few", 513), ("zeros", 1000), ("gauss", 1)])
@pytest.mark.parametrize("deep", [False, True])
def test_sums_formed_on_the_device_give_the_rounds_of_the_host(kind, n, deep):
    g = torch.Generator().manual_seed(n)
    ctx = Context(seed=2)
    if deep:
        ctx.set_recursion_depth(7, [2, 2, 3])
    x = _vectors(kind, n, g).to(DEV)
    ws = torch.empty(ctx.fit_workspace_bytes(), dtype=torch.uint8, device=DEV)
    rng = np.random.default_rng(n)
    spread = np.concatenate([np.sort(rng.uniform(lo, hi, k)) for lo, hi, k in
                             [(0.0, 6.28, 16), (-1.0, 2.0, 4), (0.7, 0.8, 4), (-3.0, -1.0, 4)]])  # cells outside the range, thin ones
    upper = np.sort(rng.uniform(0.0, 1.5, (3, 8)), axis=1)
    for init, init_t in ((None, None), (spread, upper)):
        for rounds in (0, 1, 2, 10, 300):
            if deep:
                got = ctx.fit_codebooks_deep(x, rounds, cb_init=init, cbt_init=init_t, workspace=ws)
            else:
                got = ctx.fit_codebooks(x, rounds, cb_init=init, workspace=ws), None
            want = ctx.fit_cluster(ws.cpu().numpy().view(np.uint32), rounds, cb_init=init, cbt_init=init_t)
            assert np.array_equal(got[0], want[0]), (rounds, np.abs(got[0] - want[0]).max())
            if deep:
                assert np.array_equal(got[1], want[1])


def test_fit_is_refused_on_a_capturing_stream():
    ctx, x = Context(seed=2), torch.randn((64, 1, 128), device=DEV)
    ws = torch.empty(ctx.fit_workspace_bytes(), dtype=torch.uint8, device=DEV)
    want = ctx.fit_codebooks(x, 3, workspace=ws)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin(capture_error_mode="relaxed")
        with pytest.raises(PolarQuantError):
            ctx.fit_codebooks(x, 3, workspace=ws)
        graph.capture_end()
    torch.cuda.synchronize()
    assert np.array_equal(ctx.fit_codebooks(x, 3, workspace=ws), want)


def test_a_refused_fit_leaves_nothing_in_the_graph():
    ctx, x = Context(seed=2), torch.randn((64, 1, 128), device=DEV)
    ws = torch.empty(ctx.fit_workspace_bytes(), dtype=torch.uint8, device=DEV)
    ctx.fit_codebooks(x, 3, workspace=ws)
    ws.fill_(0x5A)
    beside = torch.zeros(256, device=DEV)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin(capture_error_mode="relaxed")
        beside.add_(1.0)
        with pytest.raises(PolarQuantError):
            ctx.fit_codebooks(x, 3, workspace=ws)
        graph.capture_end()
    for r in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((beside == r + 1).all())
        assert bool((ws == 0x5A).all())
