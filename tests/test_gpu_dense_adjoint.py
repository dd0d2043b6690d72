"""The dense FP64 adjoint (at most 31 generalized velocities and 32 links per environment) at the edges of its tiles, row
forms and sweep padding, against central finite differences of the FP64 oracle; one column or link more runs the general
form.  Tolerance of the FP64 adjoint tests: 1e-3 relative with a floor of 1e-6 of the env's largest entry."""
import numpy as np
import pytest

from paper_2108_10470_amd import workloads as W
from tests import adjoint as A
from tests.test_gpu_dense import boxes, caterpillar, swing

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env, rows", [
    (caterpillar(5), 15),     # 10 columns: one tile
    (caterpillar(11), 33),    # 16 columns, 33 rows: one more than the first form holds
    (caterpillar(12), 36), (caterpillar(20), 60),
    (caterpillar(22), 66),    # more rows than the adjoint takes: zero gradients, status 1
    (boxes(1), 12), (boxes(4), 48), (boxes(5), 60),
    (swing(1), 0), (swing(15), 0), (swing(16), 0), (swing(31), 0),
    (swing(32), 0),           # 33 links: the general form
], ids=lambda x: f"{x.name}{x.n_v}" if isinstance(x, W.EnvSpec) else str(x))
@pytest.mark.parametrize("substeps, iters", [(1, 1), (2, 8), (3, 5)])
def test_dense_adjoint_edges_match_finite_differences(env, rows, substeps, iters):
    p = W.SimParams(substeps=substeps, pgs_iters=iters)
    env, params, oe, root, dof, act, wr, wd = A.f32_inputs(env, p, 4, 6)
    rc = oe.step(params, root, dof, act)["row_count"].reshape(4, -1).max(axis=1)
    assert rc.max() >= rows
    g, status = A.gpu_grads(env, params, root, dof, act, wr, wd, True)
    over = rc > 64
    assert (status == over).all(), (status, rc)
    assert (g[over] == 0).all()
    if over.all():
        return
    fd, _ = A.fd_grads(oe, params, root, dof, act, wr, wd)
    worst, ok = A.compare(g, fd, 1e-6)
    print(env.name, env.n_v, "rows", rc, "entries", int(ok.sum()), "of", ok.size, "worst", worst)
    assert np.isfinite(g).all() and ok[~over].any()
    assert (worst[~over] <= 1.0).all(), worst
