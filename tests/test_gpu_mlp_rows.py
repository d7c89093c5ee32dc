"""The row-tile MLP kernels (critic values and fit, dL/dtheta) at the edges of their tiles and
dispatch rules, against the FP64 oracle's networks: rows around a tile of 16 / 32 / 48, networks
without hidden layers, widths that are no multiple of 4 or 16, networks too wide for the fused
fit or for 64 KB of LDS, and layer normalisation on all of them."""
import numpy as np
import pytest
import torch

import paper_2204_07137_amd as P
import workloads as wl
from oracle import learn as OL
from oracle.window import mlp_forward

pytestmark = pytest.mark.gpu

# (hidden widths of the Ant critic, 37 inputs)
NETS = [[], [5], [64, 64], [70, 33], [512, 300]]
F64 = torch.float64


def rel(x, y):
    x, y = x.double().cpu().reshape(-1), torch.as_tensor(y, dtype=F64).reshape(-1)
    return float((x - y).norm() / y.norm().clamp_min(1e-300))


def _critic(hidden, layer_norm, precision, seed=3):
    md = wl.model_by_name("ant")
    dims = [37] + hidden + [1]
    sim = P.Sim(md, 4, 1, None, dims, ckpt_interval=16, precision=precision, layer_norm=layer_norm)
    net = wl.mlp_params(dims, seed)
    rng = np.random.default_rng(seed)
    ln = [(1.0 + 0.1 * rng.normal(size=w), 0.1 * rng.normal(size=w)) for w in hidden] if layer_norm else None
    return sim, net, ln


def _inputs(rows, seed=4):
    rng = np.random.default_rng(seed)
    return rng.normal(size=(rows, 37)).astype(np.float32), rng.normal(size=rows).astype(np.float32)


def _put(layers, dt):
    return [tuple(torch.as_tensor(x, dtype=dt, device="cuda").contiguous() for x in pair) for pair in layers]


# FP32: values of order one from 512-term products at 6e-8 each; FP64 as the other critic tests
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("layer_norm", [False, True])
@pytest.mark.parametrize("hidden", NETS)
def test_values(hidden, layer_norm, precision, tol):
    if layer_norm and not hidden:
        pytest.skip("layer normalisation needs a hidden layer")
    sim, net, ln = _critic(hidden, layer_norm, precision)
    # 33793 rows: one round of 48-row tiles; 8192: the first size with 32-row tiles
    for rows in (1, 15, 17, 8191, 8193, 33793):
        print(f"[mlp_rows] values {hidden} ln={layer_norm} {precision} rows={rows}", flush=True)
        x, _ = _inputs(rows)
        got = sim.critic_values(x, _put(net, sim.dtype), critic_ln=_put(ln, sim.dtype) if ln else None)
        assert rel(got, OL.critic_values(net, x, ln)) < tol
    # weights that start off a vector boundary take the scalar loads
    shifted = []
    for W, b in _put(net, sim.dtype):
        buf = torch.empty(W.numel() + 1, dtype=sim.dtype, device="cuda")
        shifted.append((buf[1:].view_as(W).copy_(W), b))
    assert shifted[0][0].data_ptr() % 16 != 0
    got2 = sim.critic_values(x, shifted, critic_ln=_put(ln, sim.dtype) if ln else None)
    assert torch.equal(got2, got)


# FP32 losses and weight changes as in the critic-fit test of the learning episode
@pytest.mark.parametrize("precision,tol_loss,tol", [("fp64", 1e-9, 1e-8), ("fp32", 1e-4, 2e-2)])
@pytest.mark.parametrize("layer_norm", [False, True])
@pytest.mark.parametrize("hidden", NETS)
def test_fit(hidden, layer_norm, precision, tol_loss, tol):
    if layer_norm and not hidden:
        pytest.skip("layer normalisation needs a hidden layer")
    # 3 minibatches of uneven size; 8200 rows in one: 32-row tiles with a ragged end
    for rows, n_mb in ((3, 3), (50, 3), (8200, 1)):
        sim, net, ln = _critic(hidden, layer_norm, precision)
        print(f"[mlp_rows] fit {hidden} ln={layer_norm} {precision} rows={rows}/{n_mb}", flush=True)
        x, y = _inputs(rows)
        perm = np.stack([np.random.default_rng(i).permutation(rows) for i in range(2)]).astype(np.int32)
        crit, cln = _put(net, sim.dtype), _put(ln, sim.dtype) if ln else None
        flat0 = [t.double().cpu() for t in OL._flat_params(net, ln)]
        rng = np.random.default_rng(8)
        m0 = [0.1 * rng.normal(size=t.shape) for t in flat0]
        v0 = [0.05 + 0.05 * rng.uniform(size=t.shape) for t in flat0]
        m, v = (torch.as_tensor(np.concatenate([t.ravel() for t in s]), dtype=sim.dtype, device="cuda") for s in (m0, v0))
        losses = sim.critic_fit(x, y, torch.as_tensor(perm), n_mb, crit, m, v, 20, 5e-4, critic_ln=cln)
        ref = OL.critic_fit(net, x, y, perm, n_mb, m0, v0, 20, 5e-4, 0.7, 0.95, 1e-8, ln=ln)
        want = OL._flat_params(ref[0], ref[1] if ln else None)
        got = []
        for i, pair in enumerate(crit):
            got += list(pair) + (list(cln[i]) if ln and i < len(cln) else [])
        assert rel(losses, ref[-1]) < tol_loss
        change = torch.cat([(a.double().cpu() - b).reshape(-1) for a, b in zip(got, flat0)])
        assert rel(change, torch.cat([(a - b).reshape(-1) for a, b in zip(want, flat0)])) < tol
        assert rel(m, torch.cat([t.reshape(-1) for t in ref[-3]])) < tol
        assert rel(v, torch.cat([t.reshape(-1) for t in ref[-2]])) < tol


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("fp32", 2e-5)])
@pytest.mark.parametrize("layer_norm", [False, True])
@pytest.mark.parametrize("hidden", NETS)
def test_policy_gradient(hidden, layer_norm, precision, tol):
    """dL/dtheta against the reverse mode of the actor on the window's own observations, from the
    window's own dL/da; the CartPole window is short, so its actions are far from saturation."""
    if layer_norm and not hidden:
        pytest.skip("layer normalisation needs a hidden layer")
    md = wl.model_by_name("cartpole")
    dims = [5] + hidden + [1]
    net, critic = wl.mlp_params(dims, 2), wl.mlp_params([5, 64, 1], 3)
    rng = np.random.default_rng(5)
    ln = [(1.0 + 0.1 * rng.normal(size=w), 0.1 * rng.normal(size=w)) for w in hidden] if layer_norm else None
    cln = [(np.ones(64), np.zeros(64))] if layer_norm else None
    for N, h in ((1, 1), (3, 5), (330, 4)):
        print(f"[mlp_rows] theta {hidden} ln={layer_norm} {precision} N={N} h={h}", flush=True)
        sim = P.Sim(md, N, h, dims, [5, 64, 1], policy_grad=True, precision=precision, layer_norm=layer_norm)
        fw = sim.forward(wl.initial_states(md, N, 1), net, critic, actor_ln=ln, critic_ln=cln)
        ad = sim.adjoint(fw, want_theta=True)
        layers = [(torch.as_tensor(W).requires_grad_(), torch.as_tensor(b).requires_grad_()) for W, b in net]
        lnt = [(torch.as_tensor(g).requires_grad_(), torch.as_tensor(b).requires_grad_()) for g, b in ln] if ln else None
        x = fw["obs"][:h].double().cpu().reshape(-1, 5)
        a = torch.tanh(mlp_forward(layers, x, lnt))
        params = []
        for i, (W, b) in enumerate(layers):
            params += [W, b] + (list(lnt[i]) if ln and i < len(lnt) else [])
        grads = torch.autograd.grad(a, params, ad["dL_da"].double().cpu().reshape(-1, 1))
        assert rel(ad["dL_dtheta_flat"], torch.cat([g.reshape(-1) for g in grads])) < tol
        sim.close()


# one hidden layer: the input of the output layer is the last of a tile's LDS
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("hidden", [[64], [128]])
@pytest.mark.parametrize("rows", [32769, 36864])
def test_values_of_48_row_tiles(rows, hidden, precision, tol):
    print(f"[mlp_rows] values {hidden} {precision} rows={rows}", flush=True)
    sim, net, _ = _critic(hidden, False, precision)
    x, _ = _inputs(rows)
    assert rel(sim.critic_values(x, _put(net, sim.dtype)), OL.critic_values(net, x, None)) < tol


# rows around the chunks of the weight gradient: one chunk, two, eight (whole XCDs), more than a
# chunk per 64 rows would make, and a ragged last chunk
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("fp32", 2e-5)])
@pytest.mark.parametrize("hidden", [[64, 64], [256, 128]])
def test_policy_gradient_chunks(hidden, precision, tol):
    md = wl.model_by_name("cartpole")
    dims = [5] + hidden + [1]
    net, critic = wl.mlp_params(dims, 2), wl.mlp_params([5, 64, 1], 3)
    for N, h in ((127, 1), (128, 1), (256, 2), (733, 5)):
        print(f"[mlp_rows] theta chunks {hidden} {precision} N={N} h={h}", flush=True)
        sim = P.Sim(md, N, h, dims, [5, 64, 1], policy_grad=True, precision=precision)
        fw = sim.forward(wl.initial_states(md, N, 1), net, critic)
        ad = sim.adjoint(fw, want_theta=True)
        layers = [(torch.as_tensor(W).requires_grad_(), torch.as_tensor(b).requires_grad_()) for W, b in net]
        a = torch.tanh(mlp_forward(layers, fw["obs"][:h].double().cpu().reshape(-1, 5), None))
        grads = torch.autograd.grad(a, [t for pair in layers for t in pair], ad["dL_da"].double().cpu().reshape(-1, 1))
        assert rel(ad["dL_dtheta_flat"], torch.cat([g.reshape(-1) for g in grads])) < tol
        sim.close()


# around the row counts at which a round of 48-row tiles begins to save a round of 32-row tiles, or no
# longer does (FP32: two against three rounds above 65536; FP64: one against two above 16384)
@pytest.mark.parametrize("precision,tol,rows", [("fp32", 1e-5, (36865, 65537, 73728, 73729)),
                                                ("fp64", 1e-12, (16385, 24576, 24577))])
@pytest.mark.parametrize("layer_norm", [False, True])
def test_values_around_the_rounds_of_tiles(layer_norm, precision, tol, rows):
    sim, net, ln = _critic([64, 64], layer_norm, precision)
    x, _ = _inputs(max(rows))
    want = OL.critic_values(net, x, ln)
    for n in rows:
        print(f"[mlp_rows] values of {n} rows ln={layer_norm} {precision}", flush=True)
        got = sim.critic_values(x[:n], _put(net, sim.dtype), critic_ln=_put(ln, sim.dtype) if ln else None)
        assert rel(got, want[:n]) < tol
