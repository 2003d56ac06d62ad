"""The built library's own gfx950 code, read back on the CPU: properties of a kernel's instruction order that its
speed rests on and that the compiler can lose without any result changing."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2609_35263_amd as wp

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")

pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs ROCm's llvm-objdump")


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """Kernel symbol -> its instructions, in program order."""
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(wp.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=d)
    kernels, name = {}, None
    for obj in sorted(d.glob("*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", str(obj)], check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                name = m[1]
                kernels[name] = []
            elif name and line.startswith("\t"):
                kernels[name].append(line.split("//")[0].strip())
    return kernels


def _find(code, *parts):
    names = [n for n in code if all(p in n for p in parts) and not n.endswith(".kd")]
    assert len(names) == 1, names
    return code[names[0]]


@pytest.mark.parametrize("dv", [64, 128, 512])
def test_merge_has_every_partial_in_flight(code, dv):
    """A thread of the merge of up to 16 splits issues its 16 partial loads without a wait for memory in between."""
    ins = _find(code, "12merge_kernel", f"ILi{dv}E")
    flight = most = 0
    for x in ins:
        if x.startswith("s_waitcnt") and "vmcnt" in x:
            flight = 0
        flight += x.startswith("global_load_dwordx4")
        most = max(most, flight)
    assert most == 16


@pytest.mark.parametrize("dims", [(64, 64), (128, 128), (576, 0)])
@pytest.mark.parametrize("early", [False, True])
def test_append_of_eight_tokens(code, dims, early):
    """The append of eight tokens a workgroup stores each token's row before it loads the next in waves that fill the
    chip (with all rows loaded first, the workgroups read together and then write together and keep half of the
    memory's directions idle), and loads all eight first in smaller ones, which wait for round trips."""
    ins = _find(code, "append_kernel", "ILi%dELi%dELi8ELb%dE" % (*dims, early))
    moves = [x.split("_")[1] for x in ins if re.match(r"global_(load|store)_dwordx4", x)]
    if early:
        assert moves.index("store") >= 8, moves
    else:
        assert moves.count("load") >= 8 and ("load", "load") not in zip(moves, moves[1:]), moves
