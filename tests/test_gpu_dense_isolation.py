"""Independent parts of an environment in the dense step (FP64, one environment per wavefront): a branch of a fixed base that
is not finite, or whose mass matrix is singular, leaves the other branches and actors as they are beside a sound one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2108_10470_amd import ags, workloads as W
from tests import parity as PT
from tests.test_gpu_dense import boxes

pytestmark = pytest.mark.gpu


def forked(*lengths) -> W.EnvSpec:
    """Fixed base and chains of the given numbers of joints on it, without contacts."""
    links = [W.Link("base", -1, "fixed")]
    for k, n in enumerate(lengths):
        for i in range(n):
            links.append(W.Link(f"b{k}_{i}", len(links) - 1 if i else 0, "revolute", anchor=(0.0, 0.0, -0.1) if i else (0.3 * k, 0.0, 0.0),
                                axis=(0.0, 1.0, 0.0) if i % 2 else (1.0, 0.0, 0.0), lower=-0.4, upper=0.4, kd=0.02, gear=0.3,
                                shapes=[W._capsule((0, 0, 0), (0, 0, -0.1), 0.02)]))
    return W.env_single(W.Actor("forked", links, root_pos=(0.0, 0.0, 10.0), init_q_halfwidth=0.45), ground=False)


def bare(env):
    """Without armature: a massless joint has a zero on the diagonal of the mass matrix."""
    for a in env.actors:
        for link in a.links:
            link.armature = 0.0
    return env


def branches(env):
    """Per link its independent part: the actor of a free root, the branch of a fixed base (-1: the base itself)."""
    parts, n = [], 0
    for a in env.actors:
        own = []
        for link in a.links:
            if link.parent < 0:
                own.append(n if link.joint == "free" else -1)
                n += link.joint == "free"
            elif own[link.parent] < 0:
                own.append(n)
                n += 1
            else:
                own.append(own[link.parent])
        parts += own
    return np.array(parts), n


def states(env, p, E):
    _, root, dof, act = PT.oracle_states(env, p, n_envs=1, n_steps=2, every=1)
    return [np.repeat(x[-1:], E, axis=0).astype(np.float32) for x in (root, dof, act)]


def make(env, p, root, dof, act, **kw):
    sim = ags.Sim([ags.Model(env)], [0] * root.shape[0], p, fp64=True, rigid_body_state=True, status=True, debug=True, **kw)
    for dst, src in ((sim.root_state, root), (sim.dof_state, dof), (sim.actuation, act)):
        dst.copy_(torch.tensor(np.asarray(src, np.float32).reshape(dst.shape)))
    return sim


def results(sim, env):
    E = sim.n_envs
    f = lambda x, *s: x.double().cpu().numpy().reshape(E, *s)  # noqa: E731
    return (f(sim.root_state, env.n_actors, 13), f(sim.dof_state, -1, 2), f(sim.rb_state, -1, 13),
            f(sim.contact_force, -1, 3), f(sim.dof_force, -1), sim.env_status.cpu().numpy().reshape(E))


def check_alone(env, out, part_of_env, parts, n_parts):
    """Environment 0 is clean, environment e >= 1 has its part part_of_env[e - 1] off: that part is non-finite, the others are
    as in environment 0."""
    root, dof, rb, cf, df, status = out
    assert not status[0] & 1 and all(np.isfinite(x[0]).all() for x in out[:5])
    dof_part = np.concatenate([[parts[k] for k, link in zip(range(o, o + len(a.links)), a.links) if link.parent >= 0]
                               for a, o in zip(env.actors, np.cumsum([0] + [len(a.links) for a in env.actors]))]).astype(int)
    roots = np.cumsum([0] + [len(a.links) for a in env.actors])[:-1]
    for e, k in enumerate(part_of_env, 1):
        assert status[e] & 1, e
        own = dof_part == k
        if own.any():
            assert not np.isfinite(dof[e, own, 1]).any(), e
        for a, r in enumerate(roots):
            if parts[r] == k:
                assert not np.isfinite(root[e, a, 7:]).any(), e
            elif env.actors[a].links[0].joint == "free":
                assert np.allclose(root[e, a], root[0, a], rtol=1e-6, atol=1e-6), (e, a)
        for j in set(range(n_parts)) - {k}:
            d, b = dof_part == j, parts == j
            assert np.allclose(dof[e, d], dof[0, d], rtol=1e-6, atol=1e-6), (e, j)
            assert np.allclose(df[e, d], df[0, d], rtol=1e-6, atol=1e-6), (e, j)
            assert np.allclose(rb[e, b], rb[0, b], rtol=1e-6, atol=1e-6), (e, j)
            assert np.allclose(cf[e, b], cf[0, b], rtol=1e-5, atol=1e-4), (e, j)


@pytest.mark.parametrize("lengths", [(2, 2), (1, 2, 2), (3, 5, 1, 4, 6), (15, 16)], ids=str)
@pytest.mark.parametrize("what", ["position", "rate", "actuation", "mass"])
@pytest.mark.parametrize("value", [np.nan, np.inf], ids=["nan", "inf"])
def test_non_finite_branch_of_a_fixed_base_stays_alone(lengths, what, value):
    env, p = W.as_f32(forked(*lengths)), W.params_f32(W.SimParams())
    parts, n = branches(env)
    root, dof, act = states(env, p, n + 1)
    mass = np.ones((n + 1, env.n_bodies), np.float32)
    for k in range(n):
        last = np.nonzero(parts == k)[0][-1]  # the tip; its joint is DOF last - 1
        if what == "mass":
            mass[k + 1, last] = value
        elif what == "actuation":
            act[k + 1, last - 1] = value
        else:
            dof[k + 1, last - 1, 0 if what == "position" else 1] = value
    sim = make(env, p, root, dof, act)
    sim.set_properties(mass_scale=torch.tensor(mass.reshape(-1), device="cuda:0"))
    for _ in range(2):
        sim.step()
        check_alone(env, results(sim, env), range(n), parts, n)


@pytest.mark.parametrize("env", [boxes(3), W.env_arm_box()], ids=lambda e: f"{e.name}{e.n_v}")
def test_actor_without_orientation_stays_alone(env):
    """A root quaternion of zeros (finite, but its unit quaternion is not)."""
    env, p = W.as_f32(env), W.params_f32(W.SimParams())
    parts, n = branches(env)
    first = np.cumsum([0] + [len(a.links) for a in env.actors])
    free = [a for a, actor in enumerate(env.actors) if actor.links[0].joint == "free"]
    root, dof, act = states(env, p, len(free) + 1)
    for e, a in enumerate(free, 1):
        root[e, a, 3:7] = 0.0
    sim = make(env, p, root, dof, act)
    sim.step()
    check_alone(env, results(sim, env), [parts[first[a]] for a in free], parts, n)


@pytest.mark.parametrize("env", [forked(2, 2), forked(1, 2, 3), bare(W.env_arm_box())], ids=lambda e: f"{e.name}{e.n_v}")
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_massless_branch_stays_alone(env, solver):
    """Mass factor 0 on every link of a branch of a fixed base: finite inputs, a singular mass matrix."""
    env, p = W.as_f32(env), W.params_f32(W.SimParams(solver=solver))
    parts, n = branches(env)
    chains = [k for k in range(n) if (parts == k).sum() > 1 or env.n_actors == 1]
    root, dof, act = states(env, p, len(chains) + 1)
    mass = np.ones((len(chains) + 1, env.n_bodies), np.float32)
    for e, k in enumerate(chains, 1):
        mass[e, parts == k] = 0.0
    zero = torch.zeros(mass.shape[0] * env.n_dof, device="cuda:0")
    sim = make(env, p, root, dof, act)
    sim.set_properties(mass_scale=torch.tensor(mass.reshape(-1), device="cuda:0"), damping=zero, stiffness=zero)
    sim.step()
    check_alone(env, results(sim, env), chains, parts, n)


@pytest.mark.parametrize("env", [boxes(1), boxes(3), W.env_arm_box(), bare(W.env_ant())], ids=lambda e: f"{e.name}{e.n_v}")
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_massless_free_body_as_in_the_articulated_form(env, solver):
    """Mass factor 0 on one free body (of the ant: its torso, the legs keep their mass): without force it keeps its velocity
    and follows its contacts.  Reference: the articulated form (two environments per wavefront, FP64), parity tolerance."""
    env, p = W.as_f32(env), W.params_f32(W.SimParams(solver=solver))
    first = np.cumsum([0] + [len(a.links) for a in env.actors])
    free = [k for k, a in zip(first, env.actors) if a.links[0].joint == "free"]
    root, dof, act = states(env, p, len(free) + 1)
    mass = np.ones((len(free) + 1, env.n_bodies), np.float32)
    for e, k in enumerate(free, 1):
        mass[e, k] = 0.0
        root[e, np.searchsorted(first, k, "right") - 1, 7:] += (0.3, -0.2, 0.1, 1.0, 2.0, -1.5)  # tumbling
    outs = []
    for lanes in (64, 32):
        sim = make(env, p, root, dof, act, lanes_per_env=lanes)
        sim.set_properties(mass_scale=torch.tensor(mass.reshape(-1), device="cuda:0"))
        sim.step()
        outs.append(results(sim, env))
    for x, y in zip(outs[0][:5], outs[1][:5]):
        assert np.isfinite(y).all() and (np.abs(x - y) <= PT.ATOL + PT.RTOL * np.abs(y)).all(), np.abs(x - y).max()
    assert (outs[0][5] == outs[1][5]).all()
