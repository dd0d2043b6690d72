"""Persistent launches of environment types with and without the dense form (FP64): the same bits as per-type launches."""
import pytest

torch = pytest.importorskip("torch")

import numpy as np

from paper_2108_10470_amd import ags, workloads as W
from tests.test_gpu_dense import caterpillar, swing

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("specs", [(W.env_ant(), caterpillar(27)), (swing(32), W.env_humanoid(), caterpillar(27), W.env_arm_box()),
                                   (caterpillar(27), swing(32))], ids=lambda s: "+".join(f"{e.name}{e.n_v}" for e in s))
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_persistent_launch_of_both_forms_equals_per_type_launches(specs, solver):
    E, T = 301, 6
    env_model = [(e * 7) % len(specs) for e in range(E)]
    p = W.SimParams(solver=solver)
    states = [W.initial_state(specs[m], 1, seed=e) for e, m in enumerate(env_model)]
    acts = [W.actuation(specs[m], 1, T, seed=e)[:, 0] for e, m in enumerate(env_model)]
    f32 = dict(dtype=torch.float32, device="cuda:0")
    a = torch.tensor(np.concatenate(acts, axis=1), **f32)
    outs = []
    for persistent in (False, True):
        sim = ags.Sim([ags.Model(s) for s in specs], env_model, p, fp64=True, persistent=persistent)
        sim.root_state.copy_(torch.tensor(np.concatenate([r.reshape(-1, 13) for r, _ in states]), **f32))
        sim.dof_state.copy_(torch.tensor(np.concatenate([d.reshape(-1, 2) for _, d in states]), **f32))
        out = []
        for t in range(T):
            sim.actuation.copy_(a[t])
            sim.step()
            out += [x.clone() for x in (sim.root_state, sim.dof_state, sim.contact_force, sim.dof_force)]
        outs.append(out)
    for x, y in zip(*outs):
        assert torch.isfinite(x).all() and torch.equal(x, y)
