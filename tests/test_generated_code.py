"""Properties of the kernels that only their generated code shows: the device code is compiled as the library's is, on
the CPU, and its assembly looked through."""
import concurrent.futures
import glob
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


M0_PROBE = """
#include "%s/common.hpp"
extern "C" __global__ void probe(const uint32_t *src, uint32_t *out, int at)
{
    __shared__ uint32_t s[4096];
    auto *l = (__attribute__((address_space(3))) uint32_t *)s;
    auto *g = (const __attribute__((address_space(1))) uint32_t *)src;
    __builtin_amdgcn_global_load_lds(g + threadIdx.x, l + at, 4, 0, 0);
    kvev::copy_to_lds<false>(src + 4 * threadIdx.x, 8192);
    __builtin_amdgcn_global_load_lds(g + 64 + threadIdx.x, l + at, 4, 0, 0);
    kvev::wait_vmem<0>();
    out[threadIdx.x] = s[threadIdx.x];
}
"""


def test_copies_to_lds_own_up_to_m0(tmp_path):
    """The copies that are written as assembly take their LDS address from m0, as the compiler's own do: between two of the
    compiler's to one address it has to set the register again."""
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(M0_PROBE % kvev_build.CSRC)
    r = subprocess.run([kvev_build.HIPCC, *kvev_build.FLAGS, "-S", "--cuda-device-only", str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    seen = [w[0] for line in out.read_text().splitlines() if (w := re.findall(r"^\s(global_load_lds_\w+|s_\w+\s+m0,)", line))]
    assert [w.split("_")[0] for w in seen] == ["s", "global"] * 3, seen


def registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"([va])(\d+)$", operand)
    return {(m.group(1), int(m.group(2)))} if m else set()


def written(instruction):
    """the vector registers that a vector instruction writes at once (a matrix instruction takes longer than what is
    looked for here)"""
    op, _, rest = instruction.partition(" ")
    if not op.startswith("v_") or op.startswith(("v_mfma", "v_cmp", "v_readfirstlane", "v_readlane")):
        return set()
    ops = [o.strip() for o in rest.split(",")]
    return registers(ops[0]) | (registers(ops[1]) if "swap" in op else set())


def early_overwrites(lines):
    """(store, instruction) for every store of more than 8 bytes whose data registers a following instruction may
    overwrite before the hardware has read them: 1 instruction further on at the least for a buffer store with its offset
    in a scalar register, 2 otherwise (s_nop n counts n + 1), along every path."""
    label = {s[:-1]: i for i, s in enumerate(lines) if s.endswith(":")}
    found = []
    for i, store in enumerate(lines):
        m = re.match(r"(buffer|global|flat|scratch)_store_dwordx[34]\s+(.*)", store)
        if not m:
            continue
        ops = [o.strip() for o in m.group(2).split(",")]
        data = registers(ops[0] if m.group(1) == "buffer" else ops[1])
        assert data, store
        need = 1 if m.group(1) == "buffer" and re.match(r"s\d+", ops[3]) else 2
        todo, seen = [(i + 1, 0)], set()
        while todo:
            k, distance = todo.pop()
            if distance >= need or k >= len(lines) or (k, distance) in seen:
                continue
            seen.add((k, distance))
            s = lines[k]
            if not s or s.startswith(".") or s.endswith(":"):
                todo.append((k + 1, distance))
            elif written(s) & data:
                found.append((store, s))
            elif not s.startswith("s_endpgm"):
                nop = re.match(r"s_nop (\d+)", s)
                distance += int(nop.group(1)) + 1 if nop else 1
                branch = re.match(r"s_c?branch\w*\s+(\S+)", s)
                if branch:
                    todo.append((label[branch.group(1)], distance))
                if not s.startswith("s_branch"):
                    todo.append((k + 1, distance))
    return found


def test_early_overwrites_are_recognised():
    store, nt = "buffer_store_dwordx4 v[4:7], v1, s[0:3], s9 offen sc1", "global_store_dwordx4 v[2:3], v[4:7], off"
    assert early_overwrites([store, ".LBB0_1:", "v_mov_b32_e32 v7, v9"])
    assert not early_overwrites([store, "s_nop 0", "v_mov_b32_e32 v7, v9"])
    assert early_overwrites([nt, "s_nop 0", "v_mov_b32_e32 v4, v9"])
    assert not early_overwrites([nt, "s_nop 1", "v_mov_b32_e32 v4, v9"])
    assert early_overwrites([nt, "s_cbranch_vccnz .LBB0_2", "s_endpgm", ".LBB0_2:", "v_permlane16_swap_b32_e32 v9, v4"])
    assert not early_overwrites([nt, "s_branch .LBB0_2", "v_mov_b32_e32 v4, v9", ".LBB0_2:", "v_add_f32_e32 v9, v4, v5", "v_mov_b32_e32 v4, v9"])


def test_store_data_is_read_before_it_is_overwritten(tmp_path):
    """Every kernel: see hold_store_data in common.hpp."""
    names = sorted(os.path.basename(p) for p in glob.glob(os.path.join(kvev_build.CSRC, "*.hip")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(names))) as ex:
        found = {n: f for asm in ex.map(lambda n: assembly(n, tmp_path), names) for n, lines in kernels(asm).items() if (f := early_overwrites(lines))}
    assert not found, found


def test_the_small_gate_asks_early_and_again(tmp_path):
    """lstm_rec_few_kernel at 256 units: a look at the partners' slots that is thrown away, a pause, the look that is taken, in both
    copies of the step (the compiler may drop a request that it finds no use for; without it a step takes 7 % longer)."""
    lines = next(ls for n, ls in kernels(assembly("lstm_oct.hip", tmp_path)).items() if "lstm_rec_few_kernelILi256" in n)
    look = re.compile(r"buffer_load_dwordx4 (v\[\d+:\d+\]),.* sc1")
    at = [i for i, s in enumerate(lines) if s.startswith("s_sleep 8")]
    assert len(at) == 2
    for i in at:
        before, after = (next(m.group(1) for s in part if (m := look.match(s))) for part in (lines[i - 1:i - 16:-1], lines[i + 1:i + 16]))
        assert before != after
