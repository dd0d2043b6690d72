"""The dense step (FP64, at most 31 generalized velocities and 32 links per environment) at the edges of its lanes,
tiles and row paths, against the FP64 oracle with the parity tolerance; one column or link more runs the general form."""
import numpy as np
import pytest

from paper_2108_10470_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu


def caterpillar(n_links: int) -> W.EnvSpec:
    """Free root and a chain of links with alternating joint axes, one sphere each, on the ground: 5 + n_links
    columns, up to 3 n_links contact rows and n_links - 1 limit rows."""
    ball = lambda: [W.Shape("sphere", (0.0, 0.0, 0.0), radius=0.05)]  # noqa: E731
    links = [W.Link("head", -1, "free", shapes=ball())]
    for i in range(1, n_links):
        ax = ((0.0, 0.0, 1.0), (0.0, 1.0, 0.0), (1.0, 0.0, 0.0))[i % 3]
        links.append(W.Link(f"l{i}", i - 1, "prismatic" if i % 7 == 6 else "revolute", anchor=(0.11, 0.0, 0.0), axis=ax,
                            lower=-0.3, upper=0.3, kd=0.05, armature=0.01, gear=0.2, shapes=ball()))
    return W.env_single(W.Actor("caterpillar", links, root_pos=(0.0, 0.0, 0.0515), init_q_halfwidth=0.02))


def boxes(n: int) -> W.EnvSpec:
    """n free boxes on the ground and a pendulum in one environment: 6 n + 1 columns, 24 n contact rows."""
    actors = [W.free_box(half=(0.05, 0.04, 0.03), pos=(0.3 * i, 0.1 * i, 0.0299)) for i in range(n)]
    return W.EnvSpec("boxes", actors + [W.pendulum()], W._plane_pairs(actors))


def swing(n: int) -> W.EnvSpec:
    """Fixed base and n joints in a chain without contacts."""
    links = [W.Link("base", -1, "fixed")]
    for i in range(n):
        links.append(W.Link(f"r{i}", i, "revolute", anchor=(0.0, 0.0, -0.1), axis=(0.0, 1.0, 0.0) if i % 2 else (1.0, 0.0, 0.0),
                            lower=-0.4, upper=0.4, kd=0.02, armature=0.01, gear=0.3,
                            shapes=[W._capsule((0, 0, 0), (0, 0, -0.1), 0.02)]))
    return W.env_single(W.Actor("swing", links, root_pos=(0.0, 0.0, 10.0), init_q_halfwidth=0.45), ground=False)


@pytest.mark.parametrize("env, rows", [
    (caterpillar(5), 15),     # 10 columns: one tile
    (caterpillar(11), 33),    # 16 columns, 33 rows: one more than fit in LDS
    (caterpillar(12), 36),    # 17 columns
    (caterpillar(20), 60),    # 25 columns
    (caterpillar(22), 66),    # 27 columns, 66 rows: more than lanes
    (caterpillar(26), 78),    # 31 columns: the last the dense form takes
    (caterpillar(27), 81),    # 32 columns: the general form
    (boxes(1), 12), (boxes(4), 48), (boxes(5), 60),
    (swing(1), 0), (swing(15), 0), (swing(16), 0), (swing(31), 0),  # 32 links
    (swing(32), 0),           # 33 links: the general form
], ids=lambda x: f"{x.name}{x.n_v}" if isinstance(x, W.EnvSpec) else str(x))
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_dense_step_edges_match_oracle(env, rows, solver):
    check(env, rows, solver, 1)


@pytest.mark.parametrize("env, rows", [(caterpillar(5), 15), (caterpillar(11), 33), (caterpillar(20), 60), (caterpillar(22), 66),
                                       (caterpillar(26), 78), (boxes(5), 60)],
                         ids=lambda x: f"{x.name}{x.n_v}" if isinstance(x, W.EnvSpec) else str(x))
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_dense_step_large_batch_matches_oracle(env, rows, solver):
    """More than four environments per CU: up to 32 rows in LDS, more streamed from scratch."""
    check(env, rows, solver, 40)


@pytest.mark.parametrize("iters", [0, 1, 2])
@pytest.mark.parametrize("env, rows", [(caterpillar(10), 30), (boxes(1), 12), (swing(8), 0)],
                         ids=lambda x: f"{x.name}{x.n_v}" if isinstance(x, W.EnvSpec) else str(x))
def test_dense_step_few_sweeps_match_oracle(env, rows, iters):
    """No sweep, only the one that keeps the rows' values, and one before it."""
    check(env, rows, 0, 1, iters)


def check(env, rows, solver, copies, iters=5):
    p = W.SimParams(solver=solver, pgs_iters=iters)
    oe, root, dof, act = PT.oracle_states(env, p, n_envs=6, n_steps=9, every=2)
    root, dof, act = (np.tile(x, (copies,) + (1,) * (x.ndim - 1)) for x in (root, dof, act))
    g, o = PT.run(env, p, root, dof, act, oe=oe, fp64=True)
    for k in ("root", "dof", "contact_force"):  # copies of an environment give the same bits
        assert (g[k].reshape(copies, -1) == g[k].reshape(copies, -1)[0]).all(), k
    s = PT.summarize(PT.compare(env, p, g, o))
    print(env.name, env.n_v, "max rows", int(o["row_count"].max()), s)
    assert o["row_count"].max() >= rows
    assert np.isfinite(g["root"]).all() and np.isfinite(g["dof"]).all()
    assert s["rows_mismatch_not_near"] == 0
    for k in PT.GATED:
        assert s[k + "_pass_rate"] == 1.0, (k, s)
