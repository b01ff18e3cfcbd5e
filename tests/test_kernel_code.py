"""The built gfx950 kernels themselves: what the compiler made of them, read from the library's own code objects (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_12639_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects inside the library, one per translation unit."""
    if not os.path.exists(build.LIB) or not shutil.which(f"{LLVM}/llvm-readelf"):
        pytest.skip("library not built, or no LLVM tools")
    data, out, at = open(build.LIB, "rb").read(), [], 0
    where = tmp_path_factory.mktemp("code")
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        u64 = lambda o: int.from_bytes(data[o:o + 8], "little")
        p = at + 32
        for _ in range(min(u64(at + 24), 16)):
            offset, size, n = u64(p), u64(p + 8), u64(p + 16)
            name = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in name and size:
                out.append(where / f"{len(out)}.co")
                out[-1].write_bytes(data[at + offset:at + offset + size])
        at += 24
    assert len(out) == len(build.UNITS)
    return out


def test_kernels_that_are_meant_to_fit_the_registers_use_no_scratch(code_objects):
    scratch = {}
    for co in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(co)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            scratch[name] = int(size)
    meant = {n: b for n, b in scratch.items() if re.match(r"_ZL?(11k_gemm_ring|6k_attnI|13k_gemm_paired|18k_gemm_paired_long|13k_gemm_direct|13k_gemm_commit|12k_gemm_small|18k_gemm_small_split|10k_gemm_fix|12k_lstm_chain|13k_lstm_levels)", n)}
    assert len(meant) > 60
    assert not {n: b for n, b in meant.items() if b}


def test_the_resident_acceptance_does_no_more_exponentials_than_its_groups_hold_tokens(code_objects):
    """A group is 2048 tokens for 512 threads: four exponentials a thread, one scaling by a power of two each.  A vocabulary takes the fewest groups
    that hold it, so that a small one does not pay for 32768 tokens; and the working distribution is in registers, which the largest instances fill (one
    value of theirs, eight bytes, is kept in scratch)."""
    found = {}
    for co in code_objects:
        asm = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(co)], capture_output=True, text=True, check=True).stdout
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(co)], capture_output=True, text=True, check=True).stdout
        scratch = dict(re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S))
        for name, q, groups, body in re.findall(r"^[0-9a-f]+ <(_ZL18k_sampled_residentILb([01])ELi(\d+)E\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", asm, re.S | re.M):
            assert body.count("v_ldexp_f64") == 4 * int(groups), name
            assert int(scratch[name]) <= (8 if groups == "16" else 0), name
            found[q, int(groups)] = name
    assert sorted(found) == [(q, g) for q in "01" for g in (2, 4, 8, 16)]


def test_the_ring_reads_a_steps_weights_past_the_caches_or_plainly(code_objects):
    """By the matrix's size, which the kernel sees at run time: of every stage's weights (two loads a wavefront) both forms are there, of its activations (one load for
    64 rows) and of a prompt's tiles only the plain one."""
    found = 0
    for co in code_objects:
        asm = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(co)], capture_output=True, text=True, check=True).stdout
        for name, tb, wide, body in re.findall(r"^[0-9a-f]+ <(_Z11k_gemm_ringILi(\d)ELi\d+ELi\dELb([01])E\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", asm, re.S | re.M):
            loads = [l for l in body.splitlines() if "buffer_load_dwordx4" in l and " lds" in l]
            past = sum(" nt" in l for l in loads)
            if wide == "1":
                assert loads and not past, name
            else:
                assert past and 2 * (len(loads) - past) == past * (2 + int(tb) // 2), (name, len(loads), past)
            found += 1
    assert found == 2 * (4 * 2 + 3)     # four epilogues at 128 and at 256 rows, three for prompts, two head sizes


def _registers(text):
    """Vector registers an operand list names."""
    out = set()
    for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        out |= set(range(int(lo), int(hi) + 1))
    return out | {int(r) for r in re.findall(r"\bv(\d+)\b", text)}


def smfmac_faults(lines):
    """What in a list of instructions the chain kernel's hand-written matrix instructions do not allow: one without wait states in front of
    it, their sums touched before the wait behind the last, a lane mask written by a vector instruction."""
    faults, sums, count = [], set(), 0
    for before, line in zip([""] + lines, lines):
        op, _, args = line.partition(" ")
        if op.startswith("v_smfmac"):
            count += 1
            if not re.match(r"s_nop [1-9]", before):
                faults.append(line)
            sums |= _registers(args.split(",")[0])
        elif line.startswith("s_nop 15"):
            sums = set()
        elif op.startswith("v_cmpx") or sums & _registers(args):
            faults.append(line)
    return count, faults


def test_the_chain_kernels_matrix_instructions_are_apart_from_what_they_depend_on(code_objects):
    """They are inline assembly, which the compiler schedules without knowing their hazards."""
    counts = []
    for co in code_objects:
        asm = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(co)], capture_output=True, text=True, check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(_ZL?12k_lstm_chain\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", asm, re.S | re.M):
            lines = [" ".join(l.split("//")[0].split()) for l in body.splitlines() if l.strip()]
            count, faults = smfmac_faults(lines)
            assert not faults, (name, faults[:5])
            counts.append(count)
    assert sorted(counts) == [4, 8, 16, 32, 64]      # four gates, one instruction for every 64 columns of a wavefront's quarter


def test_the_look_finds_what_it_is_for():
    ok = ["ds_read_b128 v[20:23], v9", "s_nop 1", "v_smfmac_f32_16x16x64_bf16 v[0:3], v[20:23], a[0:7], v8", "v_mov_b32_e32 v30, v31", "s_nop 1",
          "v_smfmac_f32_16x16x64_bf16 v[0:3], v[20:23], v[40:47], v8", "s_nop 15", "s_nop 3", "v_add_f32_e32 v0, v0, v1"]
    assert smfmac_faults(ok) == (2, [])
    assert len(smfmac_faults([l for l in ok if l != "s_nop 1"])[1]) == 2
    assert len(smfmac_faults(ok[:3] + ["v_mov_b32_e32 v30, v2"] + ok[3:])[1]) == 1
    assert len(smfmac_faults(ok[:6] + ok[8:])[1]) == 1


def test_no_fill_runs_on_the_null_stream():
    """The library's work is ordered by the caller's stream, which need not wait for the null stream: a hipMemset there can fall before or behind it."""
    for name in sorted(os.listdir(build.CSRC)):
        text = re.sub(r"//.*", "", open(os.path.join(build.CSRC, name)).read())
        assert not re.search(r"\bhipMemset\s*\(", text), name
