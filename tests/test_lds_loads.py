"""Every load into LDS of the built library finds in M0 what was set for it.

The destination is written to M0 a few instructions ahead of the load, in assembly.  In the machine code of the library's kernels there
must be, between the two, at least one instruction (the hardware asks for it), no other write of M0 and no way in or out."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2602_11543_amd as S

OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin:/opt/rocm/lib/llvm/bin:" + os.environ.get("PATH", ""))


def check(lines):
    """Number of loads into LDS in a disassembly, and those that break the rule."""
    loads, bad, since = 0, [], None         # since: instructions after the write of M0, None where there is none to use
    for n, line in enumerate(lines):
        text = line.split("//")[0].strip()
        if text.startswith("<") or text.endswith(">:"):
            since = None                    # a label
            continue
        op = text.split(" ")[0]
        if re.match(r"[a-z]\w+$", op) is None:
            continue
        if re.match(r"(s_\w+|v_read\w+) m0\b", text):
            since = 0
        elif op.startswith(("s_cbranch", "s_branch", "s_setpc", "s_swappc", "s_endpgm")):
            since = None
        elif op.startswith("buffer_load") and text.endswith(" lds"):
            loads += 1
            if not since:
                bad.append((n, text))
            since = None                    # one write for one load
        elif since is not None:
            since += 1
    return loads, bad


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_destination_of_every_load(tmp_path):
    shutil.copy(S.library_path(), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    total = 0
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" in name:
            text = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
            loads, bad = check(text.splitlines())
            assert not bad, (name, len(bad), bad[:3])
            total += loads
    assert total > 1000          # those of the GEMM loops


def test_the_rule_itself():
    ok = ["\ts_mov_b32 m0, s3   // 0: x", "\tv_add_u32_e32 v0, v1, v2", "\tbuffer_load_dwordx4 v1, s[4:7], 0 offen lds"]
    assert check(ok) == (1, [])
    for lines in (ok[:1] + ok[2:], ok[1:], ok[:2] + ["<L1>:"] + ok[2:], ok[:2] + ["\ts_cbranch_scc0 <L1>"] + ok[2:], ok[:2] + ["\ts_mov_b32 m0, s9"] + ok[2:]):
        assert len(check(lines)[1]) == 1
    assert len(check(ok + ok[1:])[1]) == 1
