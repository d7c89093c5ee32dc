"""GPU parity, against the FP64 oracle through the C ABI, of the sums a substep is made of, at the
sizes where they take another route.

* The muscles' wrenches per body: along the host-made schedule up to its capacities (runs of a
  unit, slots of a pass, slots a pair of accumulators adds per pass), by atomics beyond them.
* The subtree sums, the triangular solves and the FREE root's rotation columns: trees of two to
  32 frames whose frames have one child, several or none, at every size class of the mass matrix.
* An environment whose state is not finite, or that recomputes a substep, leaves the others of its
  wavefront as they are.
"""
import numpy as np
import pytest
import torch

import paper_2204_07137_amd as P
import workloads as wl
from oracle import oracle_window_grads
from workloads.models import MTU_MAX_POINTS

pytestmark = pytest.mark.gpu


def relnorm(x, y):
    x, y = np.asarray(x, np.float64), np.asarray(y, np.float64)
    return float(np.linalg.norm(x - y) / max(np.linalg.norm(y), 1e-300))


def _np(d):
    return {k: v.double().cpu().numpy() for k, v in d.items() if torch.is_tensor(v)}


def _arms(n, runs):
    """The muscle arm with n units whose points alternate between cart and pole `runs` times; the
    last run has a second point where the unit has room for it."""
    md = wl.muscle_arm()
    rng = np.random.default_rng([n, runs])
    bodies, pos, npt = [], [], []
    for _ in range(n):
        b = [k % 2 for k in range(runs)]
        if runs < MTU_MAX_POINTS:
            b.append(b[-1])
        p = [np.array([rng.uniform(0.2, 0.4), 0.0, rng.uniform(-0.1, 0.1)]) if x == 0 else
             np.array([rng.uniform(-0.05, 0.05), 0.0, rng.uniform(0.4, 0.9)]) for x in b]
        npt.append(len(b))
        bodies.append(b + [0] * (MTU_MAX_POINTS - len(b)))
        pos.append(p + [np.zeros(3)] * (MTU_MAX_POINTS - len(b)))
    length = 0.7 * runs
    md.update(n_mtu=n, na=n, mtu_npt=np.array(npt, np.int32), mtu_body=np.array(bodies, np.int32),
              mtu_pos=np.array(pos, float), mtu_fmax=np.full(n, 50.0 / n), mtu_lopt=np.full(n, 0.7 * length),
              mtu_lslack=np.full(n, 0.3 * length))
    return md


# 36 units of 4 runs fill the adjoint's lists exactly, 37 do not fit; 64 units of 2 runs fill a
# pass, 65 and 160 take two and three; 64 units of 3 runs need more slots than a pass has; 5 runs
# are more than a unit may have.
@pytest.mark.parametrize("n,runs", [(1, 2), (36, 4), (37, 4), (64, 2), (65, 2), (160, 2), (64, 3), (8, 5)])
def test_muscle_sums(n, runs):
    """Tolerances: ten times those of one muscle over a full window, for sums of up to 160."""
    print(f"[sums] {n} units of {runs} runs", flush=True)
    md, h, N = _arms(n, runs), 2, 2
    rng = np.random.default_rng(5)
    s0 = np.concatenate([rng.normal(0, 0.1, (N, 1)), rng.uniform(-0.5, 0.5, (N, 1)), rng.normal(0, 0.3, (N, 2)),
                         rng.uniform(0.0, 1.0, (N, n))], 1)
    u = rng.uniform(0.05, 0.95, (h, N, n))
    critic = [(rng.normal(size=(1, 4 + n)), np.zeros(1))]
    sim = P.Sim(md, N, h, None, [4 + n, 1], ckpt_interval=2, precision="fp64")
    fw = sim.forward(s0, None, critic, actions_in=u)
    ad = _np(sim.adjoint(fw))
    torch.cuda.synchronize()
    ref = oracle_window_grads(md, s0, h, None, critic, actions=u, n_total=N)
    assert relnorm(_np(fw)["s_h"], ref["s_h"]) < 1e-11
    assert relnorm(ad["dL_da"], ref["dL_da"]) < 1e-9
    assert relnorm(ad["dL_ds0"], ref["dL_ds0"]) < 1e-9


# the forward's sums by atomics (at most 256 environments, one per CU) and along the schedule (more)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,runs", [(1, 2), (36, 4), (64, 2), (65, 2), (160, 2), (64, 3), (8, 5)])
def test_muscle_sums_of_few_and_many_environments(n, runs, precision):
    print(f"[sums] {n} units of {runs} runs, 256 and 257 environments, {precision}", flush=True)
    md, h = _arms(n, runs), 2
    rng = np.random.default_rng(6)
    s0 = np.concatenate([rng.normal(0, 0.1, (257, 1)), rng.uniform(-0.5, 0.5, (257, 1)), rng.normal(0, 0.3, (257, 2)),
                         rng.uniform(0.0, 1.0, (257, n))], 1)
    u = rng.uniform(0.05, 0.95, (h, 257, n))
    critic = [(rng.normal(size=(1, 4 + n)), np.zeros(1))]
    ends = []
    for N in (256, 257):
        sim = P.Sim(md, N, h, None, [4 + n, 1], ckpt_interval=2, precision=precision)
        ends.append(_np(sim.forward(s0[:N], None, critic, actions_in=np.ascontiguousarray(u[:, :N])))["s_h"])
        sim.close()
    ref = oracle_window_grads(md, s0[:2], h, None, critic, actions=u[:, :2], n_total=2)["s_h"]
    assert np.isfinite(ends[0]).all() and np.array_equal(ends[0], ends[1][:256])
    assert relnorm(ends[0][:2], ref) < (1e-11 if precision == "fp64" else 1e-5)


def _tree(n, free_root, N, h):
    md = wl.models.chain(n=n, free_root=free_root, substeps=4)
    rng = np.random.default_rng(n)
    nq, nv, na = int(md["nq"]), int(md["nv"]), int(md["na"])
    q = rng.uniform(-0.4, 0.4, (N, nq))
    if free_root:
        q[:, 3:7] = rng.normal(size=(N, 4))
        q[:, 3:7] /= np.linalg.norm(q[:, 3:7], axis=1, keepdims=True)
    s0 = np.concatenate([q, rng.normal(0, 0.3, (N, nv))], 1)
    critic = [(rng.normal(size=(1, nq + nv)), np.zeros(1))]
    return md, s0, rng.uniform(-0.5, 0.5, (h, N, na)), critic


@pytest.mark.parametrize("n,free_root", [(1, False), (1, True), (2, True), (8, True), (9, True), (13, False),
                                         (21, True), (26, True), (31, False)])
def test_trees(n, free_root):
    """Tolerances: those of the 152-muscle humanoid's short window."""
    print(f"[sums] tree of {n + 1} frames, free root {free_root}", flush=True)
    N, h = 3, 2
    md, s0, u, critic = _tree(n, free_root, N, h)
    ref = oracle_window_grads(md, s0, h, None, critic, actions=u, n_total=N)
    for kw in (dict(ckpt_interval=2), dict(path=P.PATH_TAPE), dict(ckpt_interval=2, factor_cache=True)):
        sim = P.Sim(md, N, h, None, [s0.shape[1], 1], precision="fp64", **kw)
        fw = sim.forward(s0, None, critic, actions_in=u)
        ad = _np(sim.adjoint(fw))
        torch.cuda.synchronize()
        assert relnorm(_np(fw)["s_h"], ref["s_h"]) < 1e-10, kw
        assert relnorm(ad["dL_da"], ref["dL_da"]) < 1e-8, kw
        assert relnorm(ad["dL_ds0"], ref["dL_ds0"]) < 1e-8, kw


@pytest.mark.parametrize("n,free_root", [(1, False), (8, True), (21, True)])
def test_a_state_that_is_not_finite(n, free_root):
    print(f"[sums] not finite, tree of {n + 1} frames", flush=True)
    N, h = 5, 2
    md, s0, u, critic = _tree(n, free_root, N, h)
    bad = s0.copy()
    bad[2, -1] = np.inf
    outs = []
    for s in (s0, bad):
        sim = P.Sim(md, N, h, None, [s0.shape[1], 1], ckpt_interval=2)
        fw = sim.forward(s, None, critic, actions_in=u)
        ad = sim.adjoint(fw)
        torch.cuda.synchronize()
        outs.append((_np(fw)["s_h"], _np(ad)["dL_ds0"]))
    others = [0, 1, 3, 4]
    for a, b in zip(*outs):
        assert np.isfinite(a).all()
        assert np.array_equal(a[others], b[others])
        assert not np.isfinite(b[2]).all()


@pytest.mark.parametrize("lanes", [32, 16])
@pytest.mark.parametrize("form", [dict(path=P.PATH_TAPE), dict(ckpt_interval=4, factor_cache=True)])
def test_environments_of_a_wavefront_that_recompute_apart(lanes, form):
    """Stored substeps that fell back to FP64 are recomputed by the adjoint, and only by the
    environments concerned: a threshold at which some of a wavefront's environments fall back and
    others do not must leave every result as one environment per wavefront gives it."""
    print(f"[sums] ant, {lanes} lanes, {form}", flush=True)
    N, h = 8, 2
    W = wl.workload("ant", N)
    od = W["obs_dim"]
    dims = [od] + [w.shape[0] for w, _ in W["actor"]], [od] + [w.shape[0] for w, _ in W["critic"]]

    def run(thr, lanes_per_env):
        sim = P.Sim(W["model"], N, h, *dims, lanes_per_env=lanes_per_env, chol_fp64_threshold=thr, **form)
        fw = sim.forward(W["s0"], W["actor"], W["critic"])
        ad = sim.adjoint(fw)
        torch.cuda.synchronize()
        return _np(fw), _np(ad)

    total = h * int(W["model"]["substeps"])
    # bisect for a threshold at which about half of all substeps fall back
    lo, hi = 1e-7, 1.0
    for _ in range(40):
        thr = float(np.sqrt(lo * hi))
        fw, ad = run(thr, 0)
        count = fw["fp64_refactor_count"]
        if (np.abs(np.diff(count)) > 0).sum() >= 4:
            break
        lo, hi = (thr, hi) if count.sum() < N * total / 2 else (lo, thr)
    assert (np.abs(np.diff(count)) > 0).sum() >= 4, "no threshold separates the environments"
    fc, ac = run(thr, lanes)
    for key in ("s_h", "rewards", "value", "fp64_refactor_count"):
        assert np.array_equal(fw[key], fc[key]), key
    for key in ("dL_da", "dL_ds0"):
        assert np.array_equal(ad[key], ac[key]), key
