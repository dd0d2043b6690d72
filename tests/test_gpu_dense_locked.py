"""Joints locked by an infinite armature in the dense step and its adjoint: they keep their rate, and the rest moves as in the
FP64 oracle."""
import copy

import numpy as np
import pytest

from paper_2108_10470_amd import workloads as W
from tests import adjoint as A, parity as PT
from tests.test_gpu_dense import caterpillar, swing

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env", [swing(4), caterpillar(5), caterpillar(12)], ids=lambda e: f"{e.name}{e.n_v}")
@pytest.mark.parametrize("locked", [(2,), (1, 2), (3,)], ids=str)
def test_infinite_armature_locks_a_joint(env, locked):
    env = copy.deepcopy(env)
    for j in locked:
        env.actors[0].links[j].armature = np.inf
    p = W.SimParams()
    oe, root, dof, act = PT.oracle_states(env, p, n_envs=3, n_steps=5, every=2)
    g, o = PT.run(env, p, root, dof, act, oe=oe, fp64=True)
    s = PT.summarize(PT.compare(env, p, g, o))
    assert np.isfinite(o["root"]).all() and s["rows_mismatch_not_near"] == 0
    for k in PT.GATED:
        assert s[k + "_pass_rate"] == 1.0, (k, s)
    for j in locked:
        assert (g["dof"][:, j - 1, 1] == dof[:, j - 1, 1].astype(np.float32)).all()
    env, params, oe, root, dof, act, wr, wd = A.f32_inputs(env, p, 4, 6)
    grad, status = A.gpu_grads(env, params, root, dof, act, wr, wd, True)
    fd, _ = A.fd_grads(oe, params, root, dof, act, wr, wd)
    worst, ok = A.compare(grad, fd, 1e-6)
    assert (status == 0).all() and np.isfinite(grad).all() and ok.any() and (worst <= 1.0).all(), worst
