"""The gfx950 code of the built library, read as assembly: the wait states that transfers from global memory into LDS need.
The hardware does not wait there by itself and the compiler only sees to it for instructions that it places itself, not
inside inline assembly:
  - M0, which holds the LDS address, written by a scalar instruction: one wait state before the transfer;
  - a scalar register of the transfer's address written by a vector instruction: five.
Needs no GPU."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2311_12023_amd", "liblq_hip.so")
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
TRANSFER = re.compile(r"(global|buffer|scratch)_load_(lds_\w+|\w+ .*\blds\b)")


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", blob, entry)
            if b"gfx950" in blob[entry + 24:entry + 24 + length]:
                yield blob[at + offset:at + offset + size]
            entry += 24 + length
        at = blob.find(MAGIC, at + len(MAGIC))


def _registers(operand):
    """Numbers of the scalar registers that an operand names."""
    one, many = re.fullmatch(r"s(\d+)", operand), re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if one:
        return {int(one[1])}
    return set(range(int(many[1]), int(many[2]) + 1)) if many else set()


def _violations(lines):
    """-> (transfers seen, [(kernel, transfer, what)]) of a disassembly; straight-line order, as the code lies in memory."""
    kernel, seen, bad = "", 0, []
    since_m0, since_valu = 99, {}              # wait states since the write; per scalar register
    for line in lines:
        label = re.match(r"[0-9a-f]* ?<(.+)>:", line)
        if label:
            kernel, since_m0, since_valu = label[1], 99, {}
            continue
        text = line.split("//")[0].strip()
        if not re.match(r"[a-z]+_", text):
            continue
        op, _, rest = text.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        if TRANSFER.match(text):
            seen += 1
            if since_m0 < 1:
                bad.append((kernel, text, "M0 written by the instruction before"))
            for o in operands:
                for r in _registers(o.split(" ")[0]):
                    if since_valu.get(r, 99) < 5:
                        bad.append((kernel, text, f"s{r} written by a vector instruction {since_valu[r]} wait states before"))
        states = int(rest, 0) + 1 if op == "s_nop" else 1
        since_m0 += states
        since_valu = {r: n + states for r, n in since_valu.items() if n < 5}
        if op.startswith("s_") and operands[0] == "m0":
            since_m0 = 0
        if op.startswith("v_"):
            for r in _registers(operands[0]) | (_registers(operands[1]) if "_co_" in op or "div_scale" in op else set()):
                since_valu[r] = 0
    return seen, bad


def test_wait_states_are_recognised():
    code = ["<k>:", "s_mov_b32 m0, s1", "global_load_lds_dwordx4 v1, s[2:3]", "s_mov_b32 m0, s1", "s_nop 0",
            "global_load_lds_dwordx4 v1, s[2:3]", "v_readfirstlane_b32 s3, v0", "s_mov_b32 m0, s1", "s_nop 2",
            "global_load_lds_dwordx4 v1, s[2:3]", "v_readlane_b32 s2, v0, 1", "s_nop 4", "global_load_lds_dwordx4 v1, s[2:3]"]
    seen, bad = _violations(code)
    assert seen == 4 and [b[2][:2] for b in bad] == ["M0", "s3"]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_transfers_into_lds_keep_their_wait_states(tmp_path):
    if not os.path.exists(LIB):
        from paper_2311_12023_amd import build
        build.build()
    with open(LIB, "rb") as f:
        blob = f.read()
    total = 0
    for i, code in enumerate(_code_objects(blob)):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(code)
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        seen, bad = _violations(out.splitlines())
        total += seen
        assert not bad, (len(bad), bad[:4])
    assert total > 0
