"""The gfx950 assembly of the dense kernels (CPU only: compiled here, not run).

1. The wait states that gfx950 asks for between a lane read and the write of its source, and between a vector instruction and the
lane read that wrote its scalar operand, are inserted by the compiler, and only for instructions that it knows: the kernels'
inline assembly may order and hide values but must not hold instructions.
2. LDS is reached through DS instructions only: no FLAT memory instruction and no call (the 64-row layouts lie partly beyond
64 KiB of LDS; an earlier instrumented adjoint that reached such words through FLAT instructions faulted).
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


@pytest.mark.parametrize("src", sorted(SOURCES))
def test_lds_is_reached_through_ds_instructions_only(assembly, src):
    for name, body in kernels(assembly[src]).items():
        assert not re.search(r"\bflat_(load|store|atomic)", body), name
        assert "s_swappc" not in body and "s_call" not in body, name
        lines = body.splitlines()
        for n, line in enumerate(lines):  # an s_setpc may only end a long branch to a label of the kernel
            if "s_setpc_b64" in line:
                window = "\n".join(lines[max(0, n - 4):n])
                assert "s_getpc_b64" in window and re.search(r"\(\.LBB\w+-\.Lpost_getpc\w*\)", window), (name, n)
        assert re.search(r"\bds_(read|write)", body), name
