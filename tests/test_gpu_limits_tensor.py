"""The per-env limits tensor on joints that the model leaves unlimited: more constraint rows than the model's own limits and
contacts make.  Every env against the oracle of its own limits."""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2108_10470_amd import ags, workloads as W
from tests import parity as PT
from tests.test_gpu_dense import caterpillar, swing

pytestmark = pytest.mark.gpu


def unlimited(env):
    for a in env.actors:
        for link in a.links:
            link.lower, link.upper = -np.inf, np.inf
    return env


@pytest.mark.parametrize("env", [unlimited(swing(8)), unlimited(caterpillar(5)), unlimited(caterpillar(12)), unlimited(caterpillar(22)),
                                 unlimited(caterpillar(27))], ids=lambda e: f"{e.name}{e.n_v}")
@pytest.mark.parametrize("fp64, lanes", [(True, 64), (True, 32), (False, 64), (False, 32)], ids=["fp64", "fp64x2", "fp32", "fp32x2"])
def test_limits_of_joints_without_model_limits(env, fp64, lanes):
    p = W.params_f32(W.SimParams())
    oe, root, dof, act = PT.oracle_states(env, p, n_envs=2, n_steps=6, every=2)
    env = W.as_f32(env)
    root, dof, act = (x.astype(np.float32) for x in (root, dof, act))
    E = root.shape[0]
    limits = np.stack([dof[:, :, 0] - np.float32(0.002), dof[:, :, 0] + np.float32(0.002)], axis=2).astype(np.float32)
    model = ags.Model(env)
    sim = ags.Sim([model], [0] * E, p, fp64=fp64, lanes_per_env=lanes)
    f32 = dict(dtype=torch.float32, device="cuda:0")
    for dst, src in ((sim.root_state, root), (sim.dof_state, dof), (sim.actuation, act)):
        dst.copy_(torch.tensor(src.reshape(dst.shape), **f32))
    sim.set_properties(limits=torch.tensor(limits.reshape(-1, 2), **f32).contiguous())
    sim.step()
    got = dict(root=sim.root_state, dof=sim.dof_state, contact_force=sim.contact_force)
    rows = 0
    for e in range(E):
        spec = copy.deepcopy(env)
        joints = [link for a in spec.actors for link in a.links if link.parent >= 0]
        for link, (lo, hi) in zip(joints, limits[e]):
            link.lower, link.upper = float(lo), float(hi)
        o = O.OracleEnv(spec).step(p, *(x[e:e + 1].astype(np.float64) for x in (root, dof, act)), r_cap=400)
        rows = max(rows, int(o["row_count"].max()))
        if (o["near"] & O.NEAR_VALUE).any():
            continue
        g = {k: v.double().cpu().numpy().reshape((E,) + o[k].shape[1:])[e] for k, v in got.items()}
        if fp64:
            cs = o["contact_scale"][0]
            bound = (PT.ATOL * cs[:, 0] / p.dt + PT.RTOL * cs[:, 1])[:, None]
            assert (np.abs(g["contact_force"] - o["contact_force"][0]) <= bound).all()
            for k in ("root", "dof"):
                assert PT.ratio(g[k], o[k][0]).max() <= 1.0, (e, k)
        else:  # FP32 compute: positions within ten times the FP64 bound
            assert PT.ratio(g["root"][:, :7], o["root"][0, :, :7]).max() <= 10.0 and PT.ratio(g["dof"][:, 0], o["dof"][0, :, 0]).max() <= 10.0
    assert rows > model.info.max_rows, (rows, model.info.max_rows)
