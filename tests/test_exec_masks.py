"""The device code as built: no vector instruction between the end of a divergent
condition nested in another and the place where the lanes of both are active
again.

Where two nested conditions end at one place, the compiler drops the inner one's
restore of the execution mask (the outer one's covers it).  The block between the
two ends then runs with the inner condition's lanes, and copies that register
allocation puts there reach those lanes only: values that the other lanes still
need are lost.  The scan finds such blocks: the target of the branch after an
"s_and_b64 exec, exec, x" (a narrowing without a save), up to the instruction that
sets the mask again."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1407_2052_amd import amrvac as A

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LINE = re.compile(r"^\t(\S.*?)\s*// ([0-9A-F]{12}):.*?(?:<(\S+?)\+0x([0-9a-f]+)>)?$")


def kernels(text):
    """(name, [(address, instruction, branch target or None)]) of a disassembly."""
    name, base, body = None, 0, []
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]{16}) <(\S+)>:", line)
        if m:
            if name:
                yield name, body
            base, name, body = int(m.group(1), 16), m.group(2), []
            continue
        m = LINE.match(line)
        if m and name:
            body.append((int(m.group(2), 16), m.group(1), base + int(m.group(4), 16) if m.group(4) else None))
    if name:
        yield name, body


def partial_blocks(body):
    """Vector instructions that run with the lanes of an unsaved narrowing after
    its end, or after a loop with the lanes (none) that are still in it:
    (address of the narrowing, instruction)."""
    at = {a: i for i, (a, _, _) in enumerate(body)}
    found = []
    for i, (addr, ins, _) in enumerate(body):
        if not re.match(r"s_(and|andn2)_b64 exec, ", ins):
            continue
        k, branch = next(((k, b) for k, b in enumerate(body[i + 1:i + 4], i + 1)
                          if re.match(r"s_cbranch_exec(n?z)", b[1])), (0, None))
        if branch is None:
            continue
        if branch[1].startswith("s_cbranch_execz"):
            if branch[2] not in at:
                continue
            start = at[branch[2]]
        else:
            start = k + 1
        for _, u, _ in body[start:]:
            if re.match(r"s_\w+_b64 exec\b|s_\w+_saveexec_b64|s_c?branch|s_endpgm|s_barrier|s_setpc", u):
                break
            # v_readlane and v_writelane ignore the mask
            if re.match(r"(v|ds|global|scratch|buffer|flat)_(?!(read|write)lane)", u):
                found.append((hex(addr), u))
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs llvm-objdump")
def test_no_vector_instruction_runs_with_lanes_missing(tmp_path):
    A.lib()   # raises if it is not built
    shutil.copy(A.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    objects = [f for f in sorted(os.listdir(tmp_path)) if "amdgcn" in f]
    seen, bad = 0, {}
    for f in objects:
        text = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for name, body in kernels(text):
            seen += 1
            hits = partial_blocks(body)
            if hits:
                bad[name] = hits
    assert seen > 100, objects
    assert not bad, bad


def test_the_scan_finds_a_lost_copy():
    text = "\n".join(["0000000000001000 <k>:",
                      "\ts_and_saveexec_b64 s[10:11], vcc    // 000000001000: 00000000",
                      "\ts_cbranch_execz 8                   // 000000001004: 00000000 <k+0x24>",
                      "\tv_mov_b32_e32 v1, v2                // 000000001008: 00000000",
                      "\ts_and_b64 exec, exec, vcc           // 00000000100C: 00000000",
                      "\ts_cbranch_execz 2                   // 000000001010: 00000000 <k+0x1c>",
                      "\tv_mov_b32_e32 v3, v4                // 000000001018: 00000000",
                      "\tv_mov_b32_e32 v2, v1                // 00000000101C: 00000000",
                      "\tv_mov_b32_e32 v5, v1                // 000000001020: 00000000",
                      "\ts_or_b64 exec, exec, s[10:11]       // 000000001024: 00000000"])
    (name, body), = kernels(text)
    assert name == "k" and len(body) == 9
    assert partial_blocks(body) == [("0x100c", "v_mov_b32_e32 v2, v1"), ("0x100c", "v_mov_b32_e32 v5, v1")]
