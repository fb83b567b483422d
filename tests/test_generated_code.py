"""Properties of the kernels that only their generated code shows: the device code is compiled as the library's is, on
the CPU, and its assembly looked through."""
import os
import re
import subprocess

import pytest

from paper_2509_21354_amd import build as kvev_build

pytestmark = pytest.mark.skipif(not os.path.exists(kvev_build.HIPCC), reason="needs hipcc")


def assembly(name, tmp_path):
    src, out = os.path.join(kvev_build.CSRC, name), str(tmp_path / (name + ".s"))
    r = subprocess.run([kvev_build.HIPCC, *kvev_build.FLAGS, "-S", "--cuda-device-only", src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(out) as f:
        return f.read()


def kernels(asm):
    """name -> lines of each function of an assembly listing"""
    out, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif name:
            out[name].append(line.split(";")[0].strip())
    return out


def waits_before_ticket(lines):
    """Whether the last barrier before the ticket is drawn follows a wait for all vector stores, with no store and no
    entry from elsewhere in between.  None: the function draws no ticket."""
    at = [i for i, s in enumerate(lines) if s.startswith("global_atomic_add")]
    if not at:
        return None
    assert len(at) == 1
    i = at[0]
    while not lines[i].startswith("s_barrier"):
        i -= 1
    while i > 0:
        i -= 1
        s = lines[i]
        if s.startswith("s_waitcnt") and "vmcnt(0)" in s:
            return True
        if s.startswith(("global_store", "buffer_store", "flat_store", "s_branch", "s_cbranch")) or s.endswith(":"):
            return False
    return False


def test_partials_are_in_memory_before_the_ticket(tmp_path):
    """The split merge of decode attention (Eq. 1): the workgroup that draws the last ticket reads partials which the
    other workgroups wrote, so every storing wave has to wait for its stores before the barrier behind which the ticket
    is drawn.  (Without the wait results are right nearly always.)"""
    found = {n: waits_before_ticket(lines) for n, lines in kernels(assembly("attention_decode.hip", tmp_path)).items()}
    draws = {n: ok for n, ok in found.items() if ok is not None}
    assert len([n for n in draws if "attn_decode_kernel" in n]) == len([n for n in found if "attn_decode_kernel" in n]) > 0
    assert all(draws.values()), [n for n, ok in draws.items() if not ok]


def test_retention_leaves_room_for_eight_waves(tmp_path):
    """The merge of new chunks into the store moves memory: at more than 64 registers a SIMD holds fewer than 8 waves and
    a launch of thousands of sequences gets slower (8192 x 248 chunks: 136 us with 124 registers, 119 us with 60)."""
    asm = assembly("retain.hip", tmp_path)
    used = [int(v) for v in re.findall(r"\.vgpr_count:\s+(\d+)", asm)]
    spilt = [int(v) for v in re.findall(r"\.vgpr_spill_count:\s+(\d+)", asm)]
    assert len(used) == len(spilt) == 5 and max(used) <= 64 and max(spilt) == 0, (used, spilt)
