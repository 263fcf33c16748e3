"""What the device code of the built library has to look like (no GPU needed):
properties of hand-written assembly that no compiler checks."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_05693_amd import batchmax as bmx
from paper_2412_05693_amd.build import hipcc

LLVM_OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc()))), "llvm", "bin",
                            "llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: its instructions' texts} of the library's gfx950 code."""
    objdump = LLVM_OBJDUMP if os.path.exists(LLVM_OBJDUMP) else shutil.which("llvm-objdump")
    assert objdump, "llvm-objdump of the ROCm toolchain not found"
    d = tmp_path_factory.mktemp("code")
    shutil.copy(bmx.LIB_PATH, d / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([objdump, "-d", f], cwd=d, check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                name = m.group(1)
                out[name] = []
            elif name and line.startswith("\t"):
                out[name].append(line.split("//")[0].strip())
    return out


def test_copies_into_lds_wait_for_their_scalar_registers(kernels):
    """A load may read a scalar register (its resource) five wait states after a
    vector instruction wrote it, and M0 one after a scalar one did.  The compiler
    counts such states outside inline assembly only, so the copy blocks bring all
    five: s_mov m0 and an s_nop of four.  And nothing but those blocks uses M0, which
    their clobber lists name although the compiler does not save it."""
    prefill = {n: c for n, c in kernels.items() if "prefill_attn_kernel" in n}
    assert len(prefill) == 48        # 2 types x 2 head sizes x 3 groups x padded x split
    blocks = 0
    for name, code in kernels.items():
        for i, ins in enumerate(code):
            if ins.endswith(" lds"):
                assert name in prefill and re.match(r"buffer_load_dword", ins), (name, ins)
                # back over the block's earlier copies to its start
                j = i - 1
                while code[j].endswith(" lds"):
                    j -= 1
                m = re.fullmatch(r"s_nop (\d+)", code[j])
                assert m and code[j - 1].startswith("s_mov_b32 m0,"), (name, code[j - 1:i + 1])
                assert 1 + int(m.group(1)) + 1 >= 5, (name, code[j - 1:i + 1])
                blocks += 1
            if re.search(r"\bm0\b", ins):
                assert ins.startswith("s_mov_b32 m0,") and code[i + 2].endswith(" lds"), (name, ins)
    assert blocks > 1000


def test_no_kernel_uses_scratch_memory(kernels):
    """Registers and LDS hold every value: no kernel spills to (or indexes) scratch."""
    used = {n for n, code in kernels.items() for ins in code if ins.startswith("scratch_")}
    assert not used, sorted(used)
