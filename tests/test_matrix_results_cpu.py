"""Results of matrix instructions and the instructions that read them, in the library as it is built.

A vector or LDS instruction that reads (or writes) registers of a matrix instruction that is still under way gets (or leaves) an old value: nothing in the
hardware holds it back.  The compiler keeps instructions of its own far enough away, but not those of inline assembly, which it does not look into.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_29727_amd", "libbastion_tv.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

# Wait states (an instruction is one, s_nop k is k + 1) that the compiler leaves between the instruction and an ordinary reader of its result.
STATES = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x16_bf16": 12}


def registers(text):
    out = set()
    for kind, lo, hi, one_kind, one in re.findall(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        out |= {(kind, i) for i in range(int(lo), int(hi) + 1)} if kind else {(one_kind, int(one))}
    return out


def instructions(listing):
    """(address, mnemonic, operands, address of the branch's target) of a disassembly."""
    start, out = {}, []
    for line in listing.splitlines():
        m = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if m:
            start[m.group(2)] = int(m.group(1), 16)
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<(.+?)(?:\+0x([0-9a-f]+))?>)?$", line)
        if m:
            out.append((int(m.group(3), 16), m.group(1), m.group(2), (m.group(4), int(m.group(5) or "0", 16)) if m.group(4) else None))
    return [(at, op, args, start[to[0]] + to[1] if to and to[0] in start else None) for at, op, args, to in out]


def too_near(code):
    at = {x[0]: i for i, x in enumerate(code)}
    found = []
    for i, (_, op, args, _) in enumerate(code):
        if op not in STATES:
            assert not op.startswith("v_mfma") or not args.startswith("v"), f"{op}: how many states?"
            continue
        result, need = registers(args.split(",")[0]), STATES[op]
        todo, seen = [(i + 1, 0)], set()
        while todo:
            k, states = todo.pop()
            while k < len(code) and states < need and (k, states) not in seen:
                seen.add((k, states))
                _, o, a, to = code[k]
                if o in ("s_endpgm", "s_setpc_b64"):
                    break
                if o[:2] in ("v_", "ds") or o.startswith(("global", "buffer")):
                    if not o.startswith("v_mfma") and registers(a) & result:
                        found.append((op, args, o, a, states))
                        break
                states += int(a, 0) + 1 if o == "s_nop" else 1
                if o.startswith("s_cbranch"):
                    todo.append((at[to], states))
                k = at[to] if o == "s_branch" else k + 1
    return found


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not os.path.exists(LIB):
        from paper_2605_29727_amd import build
        build.build()
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "lib.so")
    subprocess.check_call([OBJDUMP, "--offloading", "lib.so"], cwd=d, stdout=subprocess.DEVNULL)
    return [subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], text=True) for f in sorted(d.glob("*gfx950"))]


def test_the_check_sees_a_reader_that_comes_too_early():
    listing = """0000000000000100 <k>:
	v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]  // 000000000100: D3E70000
	s_nop 5                                                     // 000000000108: BF800005
	s_cbranch_scc1 1                                            // 00000000010C: BF850001 <k+0x14>
	s_nop 7                                                     // 000000000110: BF800007
	ds_write_b128 v20, v[0:3]                                   // 000000000114: D9BE0000
	s_endpgm                                                    // 00000000011C: BF810000
"""
    assert [x[4] for x in too_near(instructions(listing))] == [7]
    assert too_near(instructions(listing.replace("s_nop 5", "s_nop 6"))) == []


def test_no_instruction_reads_a_matrix_result_too_early(listings):
    seen = 0
    for listing in listings:
        code = instructions(listing)
        seen += sum(op in STATES for _, op, _, _ in code)
        assert too_near(code) == []
    assert seen > 1000
