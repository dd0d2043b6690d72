"""An environment's bits do not depend on how its batch is launched: a small batch of the dense step (up to 64 rows of the
Delassus matrix in LDS), a large one (32; rows past them streamed from scratch) and the persistent launch, here with
environments between 33 and 64 rows."""
import pytest

torch = pytest.importorskip("torch")

from paper_2108_10470_amd import ags, workloads as W
from tests import parity as PT
from tests.test_gpu_dense import boxes, caterpillar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env", [caterpillar(11), caterpillar(12), caterpillar(20), boxes(4)], ids=lambda e: f"{e.name}{e.n_v}")
@pytest.mark.parametrize("solver", [0, 1], ids=["pgs", "tgs"])
@pytest.mark.parametrize("iters", [1, 4, 5])
def test_rows_past_32_have_the_same_bits_in_every_launch_form(env, solver, iters):
    p = W.params_f32(W.SimParams(solver=solver, pgs_iters=iters))
    env = W.as_f32(env)
    _, root, dof, act = PT.oracle_states(env, p, n_envs=6, n_steps=9, every=2)
    n = root.shape[0]
    large = 4 * torch.cuda.get_device_properties(0).multi_processor_count // n + 1  # more than four environments per CU
    outs = []
    for copies, persistent in ((1, False), (large, False), (1, True)):
        sim = ags.Sim([ags.Model(env)], [0] * (n * copies), p, fp64=True, persistent=persistent, debug=True)
        for dst, src in ((sim.root_state, root), (sim.dof_state, dof), (sim.actuation, act)):
            dst.copy_(torch.tensor(src.reshape(-1), dtype=torch.float32).repeat(copies).reshape(dst.shape))
        rows = 0
        for _ in range(2):
            sim.step()
            rows = max(rows, int(sim.dbg_rc.max()))
        assert 32 < rows <= 64
        out = [x.reshape(copies, -1) for x in (sim.root_state, sim.dof_state, sim.contact_force, sim.dof_force, sim.dbg_lam)]
        assert all(torch.isfinite(x).all() for x in out)
        assert all((x == x[0]).all() for x in out)
        outs.append([x[0].clone() for x in out])
    for other in outs[1:]:
        for x, y in zip(outs[0], other):
            assert torch.equal(x, y), float((x - y).abs().max())
