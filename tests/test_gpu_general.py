"""The general form of the FP64 step and adjoint (more than 31 generalized velocities) with contacts: up to 32 rows, 33-64 rows
of short chains (one row per lane, columns of the Delassus matrix streamed from scratch) and more, with limits and
sphere-box pairs.  The step against the FP64 oracle, the adjoint against its central finite differences, with the tolerances of the
dense form's tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2108_10470_amd import ags, workloads as W
from tests import adjoint as A, parity as PT
from tests.test_gpu_dense import boxes, caterpillar

pytestmark = pytest.mark.gpu


def field(n_boxes, n_balls, stacked=0):
    """Free boxes and balls on the ground (4 and 1 contacts), the first balls on top of the first boxes."""
    actors = [W.free_box(half=(0.05, 0.04, 0.03), pos=(0.3 * i, 0.1 * i, 0.0299)) for i in range(n_boxes)]
    for i in range(n_balls):
        pos = (0.3 * i, 0.1 * i, 0.0797 + 0.03) if i < stacked else (0.3 * i, 0.6, 0.0498)
        actors.append(W.Actor("ball", [W.Link("ball", -1, "free", shapes=[W.Shape("sphere", (0.0, 0.0, 0.0), radius=0.05)])], root_pos=pos))
    pairs = W._plane_pairs(actors) + [W.Pair(n_boxes + i, 0, 0, i, 0, 0) for i in range(stacked)]
    return W.EnvSpec("field", actors + [W.pendulum()], pairs)


def herd(n):
    """Ant-like robots in one environment: 14 n columns, chains of two joints with limits."""
    actors = [W.ant() for _ in range(n)]
    for i, a in enumerate(actors):
        a.root_pos = (3.0 * i, 0.0, a.root_pos[2])
    return W.EnvSpec("herd", actors, W._plane_pairs(actors))


# environment, rolled-out steps, range of the most rows of an environment
CASES = [(field(0, 6), 9, 18, 32), (field(2, 4), 9, 33, 64), (field(3, 4), 9, 33, 64), (field(3, 3, 3), 9, 33, 64), (herd(3), 60, 33, 64),
         (herd(4), 60, 33, 128), (boxes(6), 9, 65, 200)]
ID = lambda x: f"{x.name}{x.n_v}" if isinstance(x, W.EnvSpec) else str(x)  # noqa: E731


@pytest.mark.parametrize("env, steps, lo, hi", CASES, ids=ID)
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_general_step_matches_oracle(env, steps, lo, hi, solver):
    p = W.SimParams(solver=solver)
    oe, root, dof, act = PT.oracle_states(env, p, n_envs=6, n_steps=steps, every=max(2, steps // 5))
    g, o = PT.run(env, p, root, dof, act, oe=oe, fp64=True)
    s = PT.summarize(PT.compare(env, p, g, o))
    print(env.name, env.n_v, "rows", int(o["row_count"].min()), int(o["row_count"].max()), s)
    assert env.n_v > 31 and lo <= o["row_count"].max() <= hi
    assert np.isfinite(g["root"]).all() and np.isfinite(g["dof"]).all()
    assert s["rows_mismatch_not_near"] == 0 and s["near_switch"] < s["envs"]
    for k in PT.GATED:
        assert s[k + "_pass_rate"] == 1.0, (k, s)


@pytest.mark.parametrize("iters", [0, 1, 2, 7])
def test_general_step_few_sweeps_match_oracle(iters):
    env, p = field(3, 3), W.SimParams(pgs_iters=iters)
    oe, root, dof, act = PT.oracle_states(env, p, n_envs=6, n_steps=9, every=2)
    g, o = PT.run(env, p, root, dof, act, oe=oe, fp64=True)
    s = PT.summarize(PT.compare(env, p, g, o))
    assert ((o["row_count"] > 32) & (o["row_count"] <= 64)).any() and s["rows_mismatch_not_near"] == 0
    for k in PT.GATED:
        assert s[k + "_pass_rate"] == 1.0, (k, s)


@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_general_persistent_launch_is_bitwise_equal_to_per_type_launches(solver):
    specs = [field(0, 6), field(3, 3), herd(3)]
    E, T = 150, 4
    env_model = [e % 3 for e in range(E)]
    p = W.SimParams(solver=solver)
    states = [PT.oracle_states(s, p, n_envs=2, n_steps=9, every=2)[1:3] for s in specs]
    f32 = dict(dtype=torch.float32, device="cuda:0")
    pick = lambda k, w: np.concatenate([states[m][k][(e // 3) % len(states[m][k])].reshape(-1, w) for e, m in enumerate(env_model)])  # noqa: E731
    outs, rows = [], 0
    for persistent in (False, True):
        sim = ags.Sim([ags.Model(s) for s in specs], env_model, p, fp64=True, persistent=persistent, debug=True)
        sim.root_state.copy_(torch.tensor(pick(0, 13), **f32))
        sim.dof_state.copy_(torch.tensor(pick(1, 2), **f32))
        for _ in range(T):
            sim.step()
            rows = max(rows, int(sim.dbg_rc.max()))
        outs.append([x.clone() for x in (sim.root_state, sim.dof_state, sim.contact_force, sim.dof_force)])
    assert 32 < rows <= 64
    for x, y in zip(*outs):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("env, lo, hi", [(field(0, 6), 18, 32), (field(2, 4), 33, 64), (field(3, 3, 3), 33, 64), (herd(3), 0, 64),
                                         (caterpillar(27), 65, 200)], ids=ID)
@pytest.mark.parametrize("substeps, iters", [(1, 1), (2, 8)])
def test_general_adjoint_matches_finite_differences(env, lo, hi, substeps, iters):
    p = W.SimParams(substeps=substeps, pgs_iters=iters)
    env, params, oe, root, dof, act, wr, wd = A.f32_inputs(env, p, 4, 40 if env.name == "herd" else 6)
    rc = oe.step(params, root, dof, act)["row_count"].reshape(4, -1).max(axis=1)
    assert lo <= rc.max() <= hi, rc
    g, status = A.gpu_grads(env, params, root, dof, act, wr, wd, True)
    over = rc > 64
    assert (status == over).all() and (g[over] == 0).all(), (status, rc)
    if over.all():
        return
    fd, _ = A.fd_grads(oe, params, root, dof, act, wr, wd)
    worst, ok = A.compare(g, fd, 1e-6)
    print(env.name, env.n_v, "rows", rc, "entries", int(ok.sum()), "of", ok.size, "worst", worst)
    assert np.isfinite(g).all() and ok[~over].any()
    assert (worst[~over] <= 1.0).all(), worst
