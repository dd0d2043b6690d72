"""A non-finite actor of an environment with several: its state becomes non-finite and the environment is flagged, and the
environment's other actors (out of its reach here) step as they do beside a finite one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2108_10470_amd import ags, workloads as W
from tests import parity as PT
from tests.test_gpu_dense import boxes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make", [W.env_arm_box, lambda: boxes(3)], ids=["arm_box", "boxes"])
@pytest.mark.parametrize("value", [np.nan, np.inf], ids=["nan", "inf"])
def test_non_finite_actor_stays_alone(make, value):
    env = W.as_f32(make())
    p = W.params_f32(W.SimParams())
    _, root, dof, act = PT.oracle_states(env, p, n_envs=1, n_steps=2, every=1)
    E = 2 * env.n_actors + 1  # clean, then per actor a rate and a position of its first joint or of its free root
    root, dof, act = (np.repeat(x[-1:], E, axis=0).astype(np.float32) for x in (root, dof, act))
    joints, first = [], 0
    for a, actor in enumerate(env.actors):
        n = sum(link.joint in ("revolute", "prismatic") for link in actor.links)
        joints.append(range(first, first + n))
        if actor.links[0].joint == "free":
            root[1 + 2 * a, a, 8] = value
            root[2 + 2 * a, a, 1] = value
        else:
            dof[1 + 2 * a, first, 1] = value
            dof[2 + 2 * a, first, 0] = value
        first += n
    sim = ags.Sim([ags.Model(env)], [0] * E, p, fp64=True, rigid_body_state=True, status=True)
    sim.root_state.copy_(torch.tensor(root.reshape(-1, 13)))
    sim.dof_state.copy_(torch.tensor(dof.reshape(-1, 2)))
    sim.actuation.copy_(torch.tensor(act.reshape(-1)))
    sim.step()
    r = sim.root_state.double().cpu().numpy().reshape(E, env.n_actors, 13)
    d = sim.dof_state.double().cpu().numpy().reshape(E, -1, 2)
    f = sim.contact_force.double().cpu().numpy().reshape(E, -1)
    rb = sim.rb_state.double().cpu().numpy().reshape(E, -1, 13)
    status = sim.env_status.cpu().numpy().reshape(-1)
    links = np.concatenate([[a] * len(actor.links) for a, actor in enumerate(env.actors)])
    assert not status[0] & 1 and all(np.isfinite(x[0]).all() for x in (r, d, f, rb))
    for a, actor in enumerate(env.actors):
        for e in (1 + 2 * a, 2 + 2 * a):
            assert status[e] & 1
            assert not np.isfinite(r[e, a] if actor.links[0].joint == "free" else d[e, joints[a]]).any() or actor.fixed_base
            for b in set(range(env.n_actors)) - {a}:
                assert np.allclose(r[e, b], r[0, b], rtol=1e-6, atol=1e-6), (e, b)
                assert np.allclose(d[e, joints[b]], d[0, joints[b]], rtol=1e-6, atol=1e-6), (e, b)
                assert np.allclose(rb[e, links == b], rb[0, links == b], rtol=1e-6, atol=1e-6), (e, b)
            assert np.isfinite(f[e]).all()
