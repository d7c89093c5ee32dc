"""Critic values, critic fits and the policy gradient on both sides of the lines between row tiles and
layer by layer, against the FP64 oracle's networks, and fits whose minibatches take both in one call."""
import numpy as np
import pytest
import torch

import paper_2204_07137_amd as P
import workloads as wl
from oracle import learn as OL
from oracle.window import mlp_forward
from test_gpu_fit_routes import MODEL, check_fit, rel

pytestmark = pytest.mark.gpu


# FP32: values of order one from 512-term products at 6e-8 each; FP64 as the other critic tests
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("model,hidden,layer_norm,rows", [
    ("mtu", [400, 200], False, (1, 33, 2299, 2300, 4097, 6999, 7000)), ("ant", [512, 511], True, (1, 33, 2559, 2560)),
    ("humanoid", [400, 200], False, (15, 16, 4607, 4608)), ("humanoid", [400, 200], True, (15, 1299, 1300)),
    ("mtu", [512], False, (31, 2300)), ("ant", [256, 256], False, (15, 16))])
def test_values(model, hidden, layer_norm, rows, precision, tol):
    name, od = MODEL[model]
    dims = [od] + hidden + [1]
    sim = P.Sim(wl.model_by_name(name), 4, 1, None, dims, ckpt_interval=16, precision=precision, layer_norm=layer_norm)
    net, rng = wl.mlp_params(dims, 3), np.random.default_rng(4)
    ln = [(1.0 + 0.1 * rng.normal(size=w), 0.1 * rng.normal(size=w)) for w in hidden] if layer_norm else None
    put = lambda layers: [tuple(torch.as_tensor(x, dtype=sim.dtype, device="cuda").contiguous() for x in p) for p in layers]
    norm = rng.normal(size=od), rng.uniform(0.5, 2.0, od)
    x = rng.normal(size=(max(rows), od)).astype(np.float32)
    want = OL.critic_values(net, (x.astype(np.float64) - norm[0]) * norm[1], ln)
    for n in rows:
        print(f"[layers] values {model} {hidden} ln={layer_norm} {precision} rows={n}", flush=True)
        got = sim.critic_values(x[:n], put(net), critic_ln=put(ln) if ln else None,
                                obs_norm=tuple(torch.as_tensor(t, dtype=sim.dtype, device="cuda") for t in norm))
        assert rel(got, want[:n]) < tol


# minibatches of 383 and 384 rows (FP32) and 511 and 512 (FP64) on the two sides of a line; 2048 and
# 2049 rows of a normalised network, whose gains and biases are summed apart in one form and among
# the other gradients in the other
@pytest.mark.parametrize("model,hidden,layer_norm,precision,rows,n_mb", [
    ("mtu", [400, 200], False, "fp32", 767, 2), ("mtu", [400, 200], False, "fp32", 5, 2),
    ("ant", [256, 256], False, "fp64", 1023, 2), ("humanoid", [400, 200], False, "fp64", 70, 2),
    ("ant", [512, 512], True, "fp32", 4097, 2), ("mtu", [400, 200], True, "fp64", 4097, 2),
    ("ant", [300, 511], True, "fp64", 37, 2), ("mtu", [512], False, "fp32", 101, 3)])
def test_fit(model, hidden, layer_norm, precision, rows, n_mb):
    check_fit(model, hidden, layer_norm, precision, rows, n_mb, 2)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("fp32", 2e-5)])
@pytest.mark.parametrize("hidden,layer_norm,shapes", [
    ([512, 509], False, ((1, 1), (3, 5), (330, 4))), ([512, 512], True, ((3, 5), (1125, 4)))])
def test_policy_gradient(hidden, layer_norm, shapes, precision, tol):
    """As the policy gradient's test at the edges of the row tiles; the stochastic policy's log-std
    gradient comes from the same call."""
    md = wl.model_by_name("cartpole")
    dims = [5] + hidden + [1]
    net, critic = wl.mlp_params(dims, 2), wl.mlp_params([5, 64, 1], 3)
    rng = np.random.default_rng(5)
    ln = [(1.0 + 0.1 * rng.normal(size=w), 0.1 * rng.normal(size=w)) for w in hidden] if layer_norm else None
    cln = [(np.ones(64), np.zeros(64))] if layer_norm else None
    norm = 0.1 * rng.normal(size=5), rng.uniform(0.5, 2.0, 5)
    for N, h in shapes:
        print(f"[layers] theta {hidden} ln={layer_norm} {precision} N={N} h={h}", flush=True)
        sim = P.Sim(md, N, h, dims, [5, 64, 1], policy_grad=True, precision=precision, layer_norm=layer_norm)
        eps, log_std = rng.normal(size=(h, N, 1)), np.full(1, -1.5)
        put = lambda t: torch.as_tensor(t, dtype=sim.dtype, device="cuda")
        fw = sim.forward(wl.initial_states(md, N, 1), net, critic, actor_ln=ln, critic_ln=cln, noise=put(eps),
                         log_std=put(log_std), obs_norm=(put(norm[0]), put(norm[1])))
        ad = sim.adjoint(fw, want_theta=True)
        layers = [(torch.as_tensor(W).requires_grad_(), torch.as_tensor(b).requires_grad_()) for W, b in net]
        lnt = [(torch.as_tensor(g).requires_grad_(), torch.as_tensor(b).requires_grad_()) for g, b in ln] if ln else None
        ls = torch.as_tensor(log_std).requires_grad_()
        x = (fw["obs"][:h].double().cpu().reshape(-1, 5) - torch.as_tensor(norm[0])) * torch.as_tensor(norm[1])
        a = torch.tanh(mlp_forward(layers, x, lnt) + torch.exp(ls) * torch.as_tensor(eps).reshape(-1, 1))
        params = []
        for i, (W, b) in enumerate(layers):
            params += [W, b] + (list(lnt[i]) if ln and i < len(lnt) else [])
        grads = torch.autograd.grad(a, params + [ls], ad["dL_da"].double().cpu().reshape(-1, 1))
        assert rel(ad["dL_dtheta_flat"], torch.cat([g.reshape(-1) for g in grads[:-1]])) < tol
        assert rel(ad["dL_dlog_std"], grads[-1]) < tol
        sim.close()


def test_allocation_free_values():
    """Layer by layer the allocation-free call keeps its hidden layers in the static scratch."""
    from test_zz_no_alloc import _values_both
    dims = [280, 400, 200, 1]
    sim = P.Sim(wl.model_by_name("mtu_humanoid"), 4, 1, None, dims, ckpt_interval=16)
    critic = sim.weights(wl.mlp_params(dims, 3))
    obs = torch.as_tensor(np.random.default_rng(6).normal(size=(2000, 280)).astype(np.float32)).cuda()
    for rows in (2000, 37):
        got, ref = _values_both(sim, obs[:rows].contiguous(), critic, None)
        assert np.isfinite(ref).all() and np.array_equal(got, ref)
