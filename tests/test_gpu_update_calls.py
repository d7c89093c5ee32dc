"""Observation statistics around the rule that picks the chunked kernels, TD-lambda around its
batch of frames, and the soft update of a full list of tensors, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import paper_2204_07137_amd as P
from oracle import learn as OL

pytestmark = pytest.mark.gpu


def rel(x, y):
    x, y = x.double().cpu().reshape(-1), torch.as_tensor(y, dtype=torch.float64).reshape(-1)
    return float((x - y).norm() / y.norm().clamp_min(1e-300))


# FP32: the sums are FP64, only the results are rounded
@pytest.mark.parametrize("dt,tol", [(torch.float64, 1e-12), (torch.float32, 1e-6)])
@pytest.mark.parametrize("dim", [1, 5, 76, 257, 513])
def test_obs_stats_match_oracle(dim, dt, tol):
    for rows in (1, 1023, 1024, 1025, 9001):
        for count in (0.0, 12345.0):
            print(f"[update] stats rows={rows} dim={dim} count={count} {dt}", flush=True)
            rng = np.random.default_rng(rows + dim)
            x = torch.as_tensor((3.0 + rng.normal(size=(rows, dim))).astype(np.float32)).to("cuda", dt)
            mean = torch.as_tensor(rng.normal(size=dim).astype(np.float32)).to("cuda", dt)
            var = torch.as_tensor(rng.uniform(0.5, 2.0, dim).astype(np.float32)).to("cuda", dt)
            inv = torch.empty_like(mean)
            n, m, v, s = OL.obs_stats_update(x.cpu(), count, mean.cpu(), var.cpu(), 1e-5)
            assert P.obs_stats_update(x, count, mean, var, inv) == n
            assert rel(mean, m) < tol and rel(inv, s) < tol
            assert float((var.double().cpu() - v).abs().max()) < tol * (1.0 + float(v.max()))


# the wrapper's own line: wide FP32 batches take the single launch longer
@pytest.mark.parametrize("dim", [15, 16])
@pytest.mark.parametrize("rows", [2303, 2304])
def test_obs_stats_around_the_two_launches(rows, dim):
    rng = np.random.default_rng(rows + dim)
    x = torch.as_tensor(rng.normal(size=(rows, dim)).astype(np.float32)).cuda()
    mean, var, inv = (torch.as_tensor(rng.uniform(0.5, 2.0, dim).astype(np.float32)).cuda() for _ in range(3))
    n, m, v, s = OL.obs_stats_update(x.cpu(), 500.0, mean.cpu(), var.cpu(), 1e-5)
    assert P.obs_stats_update(x, 500.0, mean, var, inv) == n
    assert rel(mean, m) < 1e-6 and rel(var, v) < 1e-6 and rel(inv, s) < 1e-6


@pytest.mark.parametrize("h", [1, 7, 8, 9, 17])
def test_td_lambda_matches_oracle(h):
    rng = np.random.default_rng(h)
    for N in (1, 65):
        r, v = (torch.as_tensor(rng.normal(size=s)).cuda() for s in ((h, N), (h + 1, N)))
        for done in (None, torch.as_tensor(rng.uniform(size=(h, N)) < 0.3).to(torch.uint8).cuda()):
            got = P.td_lambda(r, v, 0.99, 0.95, done=done)
            ref = OL.td_lambda(r.cpu(), v.cpu(), 0.99, 0.95, None if done is None else done.cpu())
            assert rel(got, ref) < 1e-12


@pytest.mark.parametrize("n", [1, 6, 16])
def test_soft_update_lists(n):
    g = torch.Generator().manual_seed(n)
    t = [torch.randn(1 + 37 * i, generator=g, dtype=torch.float64).cuda() for i in range(n)]
    o = [torch.randn(x.shape, generator=g, dtype=torch.float64).cuda() for x in t]
    want = [0.995 * a.cpu() + (1.0 - 0.995) * b.cpu() for a, b in zip(t, o)]
    P.soft_update(t, o, 0.995)
    for a, b in zip(t, want):
        assert rel(a, b) < 1e-15


def test_soft_update_takes_a_list_in_its_order():
    """A list may hand a network on (b follows a, then c follows b) or name a tensor twice."""
    g = torch.Generator().manual_seed(3)
    a, b, c = (torch.randn(300001, generator=g, dtype=torch.float64).cuda() for _ in range(3))
    mix = lambda x, y: 0.25 * x + 0.75 * y
    b1 = mix(b.cpu(), a.cpu())
    c1 = mix(c.cpu(), b1)
    c2 = mix(c1, a.cpu())
    tail = mix(c2[1000:], b1[1000:])
    P.soft_update([b, c, c, c[1000:]], [a, b, a, b[1000:]], 0.25)
    assert rel(b, b1) < 1e-15
    assert rel(c, torch.cat([c2[:1000], tail])) < 1e-15


def test_obs_stats_under_capture():
    """A captured call holds no memory of torch's allocator, and every replay merges the batch as an
    eager call does, with eager work and allocations in between."""
    rng = np.random.default_rng(8)
    x = torch.as_tensor(rng.normal(size=(4096, 37)).astype(np.float32)).cuda()
    mean, var, inv = (torch.as_tensor(rng.uniform(0.5, 2.0, 37).astype(np.float32)).cuda() for _ in range(3))
    P.obs_stats_update(x, 1000.0, mean.clone(), var.clone(), inv.clone())   # the library is loaded
    state, graph = (mean.clone(), var.clone(), inv.clone()), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        P.obs_stats_update(x, 1000.0, *state)
        after = torch.cuda.memory_stats()["allocation.all.allocated"]
    assert after == before
    want = (mean.clone(), var.clone(), inv.clone())
    for i in range(3):
        x.copy_(torch.as_tensor(rng.normal(size=(4096, 37)).astype(np.float32)))
        graph.replay()
        scribble = [torch.full((4096, 37), float("nan"), device="cuda") for _ in range(4)]
        P.obs_stats_update(x, 1000.0, *want)
        torch.cuda.synchronize()
        for a, b in zip(state, want):
            assert rel(a, b.cpu()) < 1e-6, i
        del scribble
