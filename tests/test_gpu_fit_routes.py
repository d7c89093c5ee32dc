"""Critic fits on both sides of the rules that pick their kernels, against the FP64 oracle, and fits
whose minibatches (which differ by a row) take different kernels in one call."""
import numpy as np
import pytest
import torch

import paper_2204_07137_amd as P
import workloads as wl
from oracle import learn as OL

pytestmark = pytest.mark.gpu

MODEL = {"cartpole": ("cartpole", 5), "ant": ("ant", 37), "humanoid": ("humanoid", 76), "mtu": ("mtu_humanoid", 280)}
# losses; changes of the parameters and moments: those of the other fits
TOL = {"fp32": (1e-4, 2e-2), "fp64": (1e-9, 1e-8)}


def rel(x, y):
    x, y = (torch.as_tensor(t, dtype=torch.float64).cpu().reshape(-1) for t in (x, y))
    return float((x - y).norm() / y.norm().clamp_min(1e-300))


def check_fit(model, hidden, layer_norm, precision, rows, n_mb, n_iter):
    """The gains and biases, a small part of the parameters, are held to the tolerance by themselves."""
    print(f"[fit_routes] {model} {hidden} ln={layer_norm} {precision} rows={rows}/{n_mb}", flush=True)
    name, od = MODEL[model]
    dims = [od] + hidden + [1]
    dt = torch.float32 if precision == "fp32" else torch.float64
    sim = P.Sim(wl.model_by_name(name), 4, 1, None, dims, ckpt_interval=1, precision=precision, layer_norm=layer_norm)
    rng = np.random.default_rng(rows)
    f32 = lambda x: np.asarray(x).astype(np.float32).astype(np.float64)
    net = [tuple(f32(x) for x in pair) for pair in wl.mlp_params(dims, 3)]
    ln = [(f32(1.0 + 0.1 * rng.normal(size=w)), f32(0.1 * rng.normal(size=w))) for w in hidden] if layer_norm else None
    x, y = rng.normal(size=(rows, od)).astype(np.float32), rng.normal(size=rows).astype(np.float32)
    perm = np.stack([rng.permutation(rows) for _ in range(n_iter)]).astype(np.int32)
    put = lambda layers: [tuple(torch.as_tensor(t, dtype=dt, device="cuda").contiguous() for t in pair) for pair in layers]
    crit, cln = put(net), put(ln) if ln else []
    flat0 = [torch.as_tensor(t) for t in OL._flat_params(net, ln)]
    m0 = [f32(0.1 * rng.normal(size=t.shape)) for t in flat0]
    v0 = [f32(0.05 + 0.05 * rng.uniform(size=t.shape)) for t in flat0]
    m, v = (torch.as_tensor(np.concatenate([t.ravel() for t in s]), dtype=dt, device="cuda") for s in (m0, v0))
    losses = sim.critic_fit(x, y, torch.as_tensor(perm), n_mb, crit, m, v, 20, 5e-4, critic_ln=cln or None)
    ref = OL.critic_fit(net, x, y, perm, n_mb, m0, v0, 20, 5e-4, 0.7, 0.95, 1e-8, ln=ln)
    tol_loss, tol = TOL[precision]
    assert rel(losses, ref[-1]) < tol_loss
    got = [t for i, pair in enumerate(crit) for t in list(pair) + (list(cln[i]) if i < len(cln) else [])]
    want = OL._flat_params(ref[0], ref[1] if ln else None)
    ms, vs = (s.split([t.numel() for t in flat0]) for s in (m, v))
    flat = lambda tensors, part: torch.cat([torch.as_tensor(tensors[i], dtype=torch.float64).cpu().reshape(-1) for i in part])
    # parameters in the order W, b, gain, bias of each hidden layer, W, b
    parts = [[4 * l + k] for l in range(len(cln)) for k in (2, 3)] + [range(len(got))]
    errs = [max(rel(flat(got, part) - flat(flat0, part), flat(want, part) - flat(flat0, part)),
                rel(flat(ms, part), flat(ref[-3], part)), rel(flat(vs, part), flat(ref[-2], part))) for part in parts]
    assert max(errs) < tol, errs
    sim.close()


@pytest.mark.parametrize("rows", [8385, 8545, 8737])
def test_layer_normalised_fit_of_uneven_minibatches(rows):
    """Two minibatches of 16 j and 16 j + 1 rows whose tiles' gradients fit the workspace and do not."""
    check_fit("humanoid", [128, 128], True, "fp32", rows, 2, 3)


# fused tiles of 32 rows two to a CU (280 inputs: 58 KB), and one to a CU (256-128: 63 to 126 KB); of
# 16 rows one to a CU (57 and 62 KB); 464-128 takes all but 128 bytes of a CU's LDS
@pytest.mark.parametrize("model,hidden,layer_norm,precision,rows,n_mb", [
    ("mtu", [64, 64], False, "fp32", 8193, 1), ("humanoid", [256, 128], False, "fp32", 8192, 1),
    ("humanoid", [256, 128], True, "fp32", 8207, 1), ("humanoid", [256, 128], False, "fp64", 8193, 1),
    ("mtu", [64, 64], False, "fp64", 100, 3), ("ant", [128, 64], True, "fp64", 100, 3),
    ("cartpole", [464, 128], True, "fp32", 8200, 1)])
def test_fused_forms(model, hidden, layer_norm, precision, rows, n_mb):
    check_fit(model, hidden, layer_norm, precision, rows, n_mb, 2)
