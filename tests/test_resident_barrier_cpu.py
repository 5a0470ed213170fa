"""The barrier of resident workgroups in the library as built: behind every
write back of the L2 the code waits for it before anything else goes to
memory, the count that lets the other workgroups read among it."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2601_19505_amd as fq

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MEMORY = re.compile(r"\b(global|flat|buffer|scratch)_\w+")


def unwaited(lines):
    """The write backs with a memory access, or the end of the code, before
    the wait for them."""
    bad, kernel, pending = [], "", None
    for line in lines:
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m:
            if pending:
                bad.append(pending)
            kernel, pending = m.group(1), None
            continue
        text = line.split("//")[0]
        if "buffer_wbl2" in text:
            if pending:
                bad.append(pending)
            pending = (kernel, line.strip())
        elif pending and re.search(r"s_waitcnt .*vmcnt\(0\)", text):
            pending = None
        elif pending and MEMORY.search(text):
            bad.append(pending)
            pending = None
    if pending:
        bad.append(pending)
    return bad


def test_the_reader_finds_a_missing_wait():
    good = ["00 <k>:", "buffer_wbl2 sc1", "s_or_b64 exec, exec, s[2:3]", "s_waitcnt vmcnt(0)", "global_atomic_add v1, v2"]
    assert unwaited(good) == []
    assert len(unwaited(good[:3] + good[4:])) == 1
    assert len(unwaited(good[:2])) == 1
    assert len(unwaited(good[:3] + ["s_waitcnt lgkmcnt(0)"] + good[4:])) == 1


def test_every_write_back_is_waited_for(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(fq.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    seen = 0
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        # the resident kernels are in every object but the host runtime's
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", os.path.join(tmp_path, name)], check=True,
                              capture_output=True, text=True).stdout.splitlines()
        seen += sum("buffer_wbl2" in line for line in text)
        assert unwaited(text) == [], name
    assert seen >= 8
