"""The hand-over of greedy_small_kernel in the built code: the block that counts
itself done last reads what the others wrote, so each wave's stores and atomics
have to be complete (vmcnt) before its block's barrier, not only those of the
wave that counts."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_waves_wait_for_their_writes_before_the_block_counts(tmp_path):
    import paper_2411_15419_amd as L
    lib = tmp_path / "lib.so"
    shutil.copy(os.path.join(os.path.dirname(L.__file__), "libluffy.so"), lib)
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=tmp_path, check=True, capture_output=True)
    bodies = {}
    for f in sorted(tmp_path.glob("*gfx950")):
        syms = subprocess.run([OBJDUMP, "-t", f.name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for name in re.findall(r"\.text\s+[0-9a-f]+ (?:\.\w+ )?(\S*greedy_small_kernel\S*)$", syms, re.M):
            bodies[name] = subprocess.run([OBJDUMP, "-d", f"--disassemble-symbols={name}", f.name], cwd=tmp_path,
                                          check=True, capture_output=True, text=True).stdout
    assert len(bodies) == 2, "greedy_small_kernel, alone and shared, in libluffy.so"
    for name, code in bodies.items():
        ops = [ln.split("//")[0].strip() for ln in code.splitlines() if "//" in ln]
        # the completion counter's add (the kernel's only global add), and the barrier before it
        add = [i for i, op in enumerate(ops) if op.startswith("global_atomic_add ")]
        assert len(add) == 1, [ops[i] for i in add]
        barrier = max(i for i in range(add[0]) if ops[i] == "s_barrier")
        wrote = max(i for i in range(barrier) if re.match(r"(global|flat|buffer)_(store|atomic)", ops[i]))
        waits = [op for op in ops[wrote + 1:barrier] if op.startswith("s_waitcnt") and "vmcnt(0)" in op]
        assert waits, (name, ops[wrote:barrier + 1])
