"""Host-side checks of the dense kernels' LDS layouts (CPU only): tests/dense_lds_check.cpp replays DenseLds and DenseAdjLds (the
header that the runtime and the kernels use) with every array's words and the phases in which it is alive, built with
AddressSanitizer and UBSan, for the workload models and for the smallest and largest models of every size class."""
import json
import os
import subprocess

import pytest

from paper_2108_10470_amd import ags, workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_10470_amd", "csrc")

# links, velocities, DOFs, actors, rows
SIZES = [(2, 1, 1, 1, 2), (16, 15, 15, 1, 62), (10, 15, 9, 2, 200), (16, 16, 15, 1, 62), (17, 15, 15, 1, 62), (28, 27, 27, 1, 200),
         (22, 27, 21, 1, 200), (32, 31, 31, 1, 62), (29, 27, 21, 1, 200), (26, 31, 25, 1, 400), (32, 31, 7, 24, 400)]
MODELS = {"humanoid": W.env_humanoid, "ant": W.env_ant, "arm_box": W.env_arm_box, "hand_cube": W.env_hand_cube,
          "pendulum": lambda: W.EnvSpec("pend", [W.pendulum()], [])}


def info(model):
    i = ags.Model(MODELS[model]()).info
    return i.n_links, i.n_v, i.n_dof, i.n_actors, i.max_rows


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("denselds") / "dense_lds_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                           "-I", os.path.join(ROOT, "include"), "-o", exe, os.path.join(ROOT, "tests", "dense_lds_check.cpp")])

    def run(*args):
        r = subprocess.run([exe, *[str(x) for x in args]], capture_output=True, text=True)
        assert r.returncode == 0, (args, r.stderr)
        return json.loads(r.stdout)
    return run


@pytest.mark.parametrize("size", SIZES + sorted(MODELS), ids=str)
def test_dense_step_layout(check, size):
    links, v, dofs, actors, _ = size if isinstance(size, tuple) else info(size)
    for tendon_joints in (0, dofs, 64):
        d = check("step", links, v, dofs, actors, tendon_joints)
        assert d["bytes_64_rows"] <= 64 * 1024, d  # launched without a raised limit
    print(size, d)


@pytest.mark.parametrize("size", SIZES + sorted(MODELS), ids=str)
def test_dense_adjoint_layout(check, size):
    links, v, dofs, actors, rows = size if isinstance(size, tuple) else info(size)
    for substeps in (1, 2, 3, 8):
        for iters in (0, 1, 3, 4, 8, 12, 31, 32):
            for cap in (5, 32, 64):
                d = check("adjoint", links, v, dofs, actors, rows, substeps, iters, cap)
    print(size, d)


def test_six_workgroups_of_the_humanoid_fit_a_cu(check):
    """Two substeps, eight sweeps, 32 rows; LDS is allocated in steps of 1280 B, and the kernel has 104 B of its own."""
    links, v, dofs, actors, rows = info("humanoid")
    d = check("adjoint", links, v, dofs, actors, rows, 2, 8, 64)
    assert 6 * -(-(d["bytes_32_rows"] + 104) // 1280) * 1280 <= 160 * 1024, d
