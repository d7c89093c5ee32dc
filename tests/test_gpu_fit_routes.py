"""Critic fits whose minibatches take different kernels in one call, against the FP64 oracle: a
call's minibatches differ by a row, and the size of the workspace may lie between them."""
import numpy as np
import pytest
import torch

import paper_2204_07137_amd as P
import workloads as wl
from oracle import learn as OL

pytestmark = pytest.mark.gpu


def rel(x, y):
    x, y = (torch.as_tensor(t, dtype=torch.float64).cpu().reshape(-1) for t in (x, y))
    return float((x - y).norm() / y.norm().clamp_min(1e-300))


@pytest.mark.parametrize("rows", [8385, 8545, 8737])
def test_layer_normalised_fit_of_uneven_minibatches(rows):
    """Two minibatches of 16 j and 16 j + 1 rows whose tiles' gradients fit the workspace and do
    not.  The tolerance of the weights' change and the moments is that of the other FP32 fits; the
    gains and biases, a small part of the parameters, are held to it by themselves."""
    print(f"[fit_routes] humanoid critic, layer normalisation, rows={rows}", flush=True)
    dims = [76, 128, 128, 1]
    sim = P.Sim(wl.model_by_name("humanoid"), 4, 1, None, dims, ckpt_interval=16, layer_norm=True)
    net = [tuple(x.astype(np.float32).astype(np.float64) for x in pair) for pair in wl.mlp_params(dims, 3)]
    rng = np.random.default_rng(rows)
    f32 = lambda x: x.astype(np.float32).astype(np.float64)
    ln = [(f32(1.0 + 0.1 * rng.normal(size=w)), f32(0.1 * rng.normal(size=w))) for w in dims[1:-1]]
    x, y = rng.normal(size=(rows, 76)).astype(np.float32), rng.normal(size=rows).astype(np.float32)
    perm = np.stack([rng.permutation(rows) for _ in range(3)]).astype(np.int32)
    put = lambda layers: [tuple(torch.as_tensor(t, dtype=torch.float32, device="cuda").contiguous() for t in pair)
                          for pair in layers]
    crit, cln = put(net), put(ln)
    flat0 = [torch.as_tensor(t) for t in OL._flat_params(net, ln)]
    m0 = [f32(0.1 * rng.normal(size=t.shape)) for t in flat0]
    v0 = [f32(0.05 + 0.05 * rng.uniform(size=t.shape)) for t in flat0]
    m, v = (torch.as_tensor(np.concatenate([t.ravel() for t in s]), dtype=torch.float32, device="cuda") for s in (m0, v0))
    losses = sim.critic_fit(x, y, torch.as_tensor(perm), 2, crit, m, v, 20, 5e-4, critic_ln=cln)
    ref = OL.critic_fit(net, x, y, perm, 2, m0, v0, 20, 5e-4, 0.7, 0.95, 1e-8, ln=ln)
    assert rel(losses, ref[-1]) < 1e-4
    got = [t for i, pair in enumerate(crit) for t in list(pair) + (list(cln[i]) if i < len(cln) else [])]
    want = OL._flat_params(ref[0], ref[1])
    ms, vs = (s.split([t.numel() for t in flat0]) for s in (m, v))
    flat = lambda tensors, part: torch.cat([torch.as_tensor(tensors[i], dtype=torch.float64).cpu().reshape(-1) for i in part])
    # parameters in the order W, b, gain, bias of two hidden layers, W, b
    for part in ([2], [3], [6], [7], range(len(got))):
        assert rel(flat(got, part) - flat(flat0, part), flat(want, part) - flat(flat0, part)) < 2e-2, part
        assert rel(flat(ms, part), flat(ref[-3], part)) < 2e-2, part
        assert rel(flat(vs, part), flat(ref[-2], part)) < 2e-2, part
