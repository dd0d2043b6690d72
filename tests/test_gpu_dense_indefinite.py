"""Drive damping so negative that a joint's inertia with it is below zero: the mass matrix is indefinite, and the dense step
gives what the articulated form gives (two environments per wavefront, FP64; parity tolerance with the largest entry of an
environment as its scale)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2108_10470_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_dense import caterpillar, swing
from tests.test_gpu_dense_isolation import forked, make, results

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env", [swing(1), swing(8), forked(2, 3), caterpillar(5), caterpillar(12), caterpillar(22)],
                         ids=lambda e: f"{e.name}{e.n_v}")
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
def test_indefinite_mass_matrix_as_in_the_articulated_form(env, solver):
    """One joint per environment; the first environment has none."""
    env, p = W.as_f32(env), W.params_f32(W.SimParams(solver=solver))
    E = env.n_dof + 1
    _, root, dof, act = PT.oracle_states(env, p, n_envs=1, n_steps=4, every=3)
    root, dof, act = (np.repeat(x[-1:], E, axis=0).astype(np.float32) for x in (root, dof, act))
    kd = np.tile(np.array([link.kd for a in env.actors for link in a.links if link.parent >= 0], np.float32), (E, 1))
    for j in range(E - 1):
        kd[j + 1, j] = -200.0
    outs = []
    for lanes in (64, 32):
        sim = make(env, p, root, dof, act, lanes_per_env=lanes)
        sim.set_properties(damping=torch.tensor(kd.reshape(-1), device="cuda:0"))
        sim.step()
        outs.append(results(sim, env) + (sim.dbg_rc.cpu().numpy(),))
    for x, y in zip(outs[0][:5], outs[1][:5]):
        assert np.isfinite(y).all() and np.isfinite(x).all()
        scale = np.abs(y).reshape(E, -1).max(axis=1).reshape((E,) + (1,) * (y.ndim - 1))
        assert (np.abs(x - y) <= PT.ATOL + PT.RTOL * np.maximum(np.abs(y), scale)).all(), np.abs(x - y).max()
    assert (outs[0][5] & 1 == 0).all() and (outs[0][6] == outs[1][6]).all()
