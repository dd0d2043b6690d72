"""The gfx950 assembly of the dense kernels (CPU only: compiled here, not run).

The wait states that gfx950 asks for between a lane read and the write of its source, and between a vector instruction and the
lane read that wrote its scalar operand, are inserted by the compiler, and only for instructions that it knows: the kernels'
inline assembly may order and hide values but must not hold instructions.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_10470_amd", "csrc")
SOURCES = {"ags_dense": 24, "ags_dense_adjoint": 6, "ags_dense_jacmass": 3}  # kernels of each


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out, jobs = tmp_path_factory.mktemp("asm"), []
    for src in SOURCES:  # compiled side by side, with the library's flags
        jobs.append(subprocess.Popen(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--cuda-device-only", "-S", "-O3", "-std=c++17",
                                      "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                                      os.path.join(CSRC, src + ".hip"), "-o", str(out / (src + ".s"))], stderr=subprocess.DEVNULL))
    assert [job.wait() for job in jobs] == [0] * len(jobs)
    return {src: (out / (src + ".s")).read_text() for src in SOURCES}


def kernels(text):
    """Name and body of every kernel."""
    names = re.findall(r"^\t\.amdhsa_kernel (\S+)", text, flags=re.M)
    return {n: text.split(f"\n{n}:", 1)[1].split(".amdhsa_kernel", 1)[0] for n in names}


@pytest.mark.parametrize("src", sorted(SOURCES))
def test_inline_assembly_holds_no_instructions(assembly, src):
    bodies = kernels(assembly[src])
    assert len(bodies) == SOURCES[src]
    for name, body in bodies.items():
        for block in re.findall(r";+#?ASMSTART\n(.*?);+#?ASMEND", body, flags=re.S):
            code = [line.split(";")[0].strip() for line in block.splitlines()]
            assert not any(code), (name, block)
