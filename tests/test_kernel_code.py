"""What the compiler made of the kernels that depend on its scheduling, read
from the disassembly of the library built here (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1801_01072_amd as ent

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(ent.LIB_PATH),
                                reason="needs llvm-objdump and the built library")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled name -> instructions (address, mnemonic, operands) of every
    kernel of the dense and BF16x3 code objects."""
    d = tmp_path_factory.mktemp("code")
    lib = str(d / "lib.so")
    shutil.copy(ent.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(d.glob("lib.so.*gfx950*")):
        syms = subprocess.run([OBJDUMP, "-t", str(f)], capture_output=True, text=True, check=True).stdout
        if "batch_dense_" not in syms and "batch_bf16x3_" not in syms:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True,
                              check=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
            if m:
                name = m.group(1)
                out[name] = []
                continue
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):?", line)
            if m and name:
                out[name].append((int(m.group(3), 16), m.group(1), m.group(2)))
    return out


def test_dense_k_loops_wait_only_where_they_say(kernels):
    """The K loop of a dense tile keeps two chunks of direct loads to LDS in
    flight: its own waits for them stand ahead of a barrier.  A wait for loads
    straight ahead of an LDS read is the compiler's, and drains them all."""
    names = [n for n in kernels if re.search(r"(batch_dense_step|batch_dense_persistent|dense_step|dense_step_split)_kernel", n)
             and any(op.startswith("global_load_lds") for _, op, _ in kernels[n])]
    assert len(names) >= 16
    for n in names:
        ins = kernels[n]
        bad = [hex(a) for i, (a, op, args) in enumerate(ins) if op == "s_waitcnt" and "vmcnt(0)" in args
               and any(o.startswith("ds_read") for _, o, _ in ins[i + 1:i + 3])]
        assert not bad, (n, bad)
