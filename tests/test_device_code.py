"""Properties of the built device code that no numerical test can show reliably.

The disassembly is that of the library built here (gfx950)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2010_09701_amd", "liboefe.so")
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")

pytestmark = pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(OBJDUMP)),
                                reason="liboefe.so not built, or no llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel symbol -> its instructions, in order."""
    d = tmp_path_factory.mktemp("device_code")
    shutil.copy(LIB, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    res = {}
    for f in sorted(d.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", f.name], cwd=d, check=True,
                              capture_output=True, text=True).stdout
        for m in re.finditer(r"^<(_Z\S+)>:\n((?:[ \t]+\S.*\n)+)", text, flags=re.M):
            res[m.group(1)] = [ln.split("//")[0].strip() for ln in m.group(2).splitlines()]
    return res


def test_part_kernel_waits_for_its_copies(kernels):
    """fe_part_kernel copies a tile's coupling block to LDS and reads it after a barrier.  Every wave has to
    wait for its own share of the copies before that barrier, also one whose rows all lie past the mesh and
    whose loads of X the compiler may have branched around: so the wait stands right before the barrier."""
    names = [k for k in kernels if "fe_part_kernel" in k]
    assert len(names) >= 5, names
    for k in names:
        code = kernels[k]
        copies = [i for i, c in enumerate(code) if c.startswith("global_load_lds")]
        assert copies, k
        bar = next(i for i in range(copies[-1], len(code)) if code[i].startswith("s_barrier"))
        assert code[bar - 1].startswith("s_waitcnt") and "vmcnt(0)" in code[bar - 1], (k, code[bar - 3:bar + 1])
