"""The dense Jacobian and mass-matrix kernel (at most 31 generalized velocities and 32 links) at the edges of its tiles
against the FP64 oracle, with the tolerance of the other tests of these tensors; one column or link more runs the general
form.  Inertias scaled per environment scale M by the same factor."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2108_10470_amd import ags, workloads as W
from tests import test_gpu_jacmass as JM
from tests.test_gpu_dense import boxes, caterpillar, swing

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env", [caterpillar(5), caterpillar(11), caterpillar(12), caterpillar(26), caterpillar(27), boxes(1),
                                 boxes(5), swing(1), swing(15), swing(16), swing(31), swing(32)],
                         ids=lambda e: f"{e.name}{e.n_v}")
def test_dense_jacobian_and_mass_edges_match_oracle(env):
    env = W.as_f32(env)
    oe = O.OracleEnv(env)
    root, dof = JM._poses(env, 3, 5)
    sim = ags.Sim([ags.Model(env)], [0] * 3, W.params_f32(W.SimParams()))
    J, M = JM._gpu(sim, 0, root, dof)
    JM._check(f"jacmass_edges_{env.name}{env.n_v}", env, oe, root, dof, J, M, range(3))
    assert (M == M.transpose(0, 2, 1)).all()
    sim.bind(ags.BODY_MASS_SCALE, torch.full(sim.shapes[ags.BODY_MASS_SCALE], 2.0, dtype=torch.float32, device=sim.device))
    J2, M2 = JM._gpu(sim, 0, root, dof)
    assert (J2 == J).all() and (M2 == 2 * M).all()


def test_non_finite_links_spoil_only_their_own_entries():
    """A joint angle that is not finite: the Jacobian rows and mass-matrix entries that do not depend on it are unchanged."""
    env = W.as_f32(W.env_arm_box())
    root, dof = JM._poses(env, 2, 3)
    dof[1, 2, 0] = np.nan  # the third joint of the arm
    sim = ags.Sim([ags.Model(env)], [0] * 2, W.params_f32(W.SimParams()))
    root[1], dof[1, [0, 1]], dof[1, 3:] = root[0], dof[0, [0, 1]], dof[0, 3:]
    J, M = JM._gpu(sim, 0, root, dof)
    box = slice(env.n_v - 6, env.n_v)
    assert np.isfinite(J[0]).all() and np.isfinite(M[0]).all()
    assert (M[1][box, box] == M[0][box, box]).all() and (J[1][-1] == J[0][-1]).all()
    assert (M[1][box, :env.n_v - 6] == 0).all() and np.isnan(M[1][2, 2])
