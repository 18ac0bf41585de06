"""Wait states in the built library.  A vector ALU write of a register must be two wait states away from a DPP read or a row swap
(v_permlane16_swap, v_permlane32_swap) of it.  The compiler sees to that between its own instructions; it does not look inside inline
assembly, where the rollout kernels' multiply-add runs are, so the distance is checked in the code as it was built."""
import re
import struct
import subprocess
from collections import deque
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

import pytest

LIB = Path(__file__).resolve().parent.parent / "paper_2501_15129_amd" / "libes_hip.so"
OBJDUMP = Path("/opt/rocm/llvm/bin/llvm-objdump")
NEEDED = 2
REG = re.compile(r"v(\d+)$|v\[(\d+):(\d+)\]$")


def registers(operand):
    m = REG.match(operand.strip(" ,|-"))
    if not m:
        return ()
    return range(int(m[1]), int(m[1]) + 1) if m[1] else range(int(m[2]), int(m[3]) + 1)


def vgprs_written(name, ops):
    if not name.startswith("v_") or name.startswith(("v_cmp", "v_mfma", "v_accvgpr_write", "v_readlane", "v_readfirstlane", "v_nop")):
        return set()
    return {r for op in (ops[:2] if "swap" in name else ops[:1]) for r in registers(op)}


def violations(lines):
    """(function, writer, reader) of every read that is too early; lines of a disassembly in order."""
    found, seen, reads = [], deque(maxlen=NEEDED), 0
    function = "?"
    for line in lines:
        if line[:1] not in "\t ":
            if line.endswith(">:"):
                function = line.split("<", 1)[1][:-2]
                seen.clear()
            continue
        text = line.split("//", 1)[0].strip()
        if not text:
            continue
        name, _, rest = text.partition(" ")
        if "_dpp" in name or ("permlane" in name and "swap" in name):
            reads += 1
            ops = rest.split(",")
            used = {r for op in (ops[:2] if "swap" in name else [ops[1].split()[0] if ops[1].split() else ""]) for r in registers(op)}
            distance = 0
            for before, operands, states in reversed(seen):
                if distance >= NEEDED:
                    break
                if used & vgprs_written(before, operands.split(",")):
                    found.append((function, f"{before} {operands}", text))
                    break
                distance += states
        seen.append((name, rest, 1 + int(rest, 0) if name == "s_nop" else 1))
    return found, reads


def test_the_check_sees_what_it_looks_for():
    code = ["0000 <k>:", "\tv_fmac_f32_dpp v3, v1, v2 row_newbcast:1 row_mask:0xf bank_mask:0xf", "\ts_mov_b32 s0, s1", "\tv_permlane16_swap_b32_e32 v4, v3"]
    assert len(violations(code)[0]) == 1
    assert not violations(code[:3] + ["\ts_nop 0"] + code[3:])[0]
    assert not violations(code[:2] + ["\ts_nop 1"] + code[3:])[0]
    assert len(violations(["0000 <k>:", "\tv_mul_f32_e32 v1, v5, v6", "\tv_fmac_f32_dpp v3, v1, v2 row_ror:1"])[0]) == 1
    assert not violations(["0000 <k>:", "\tv_mul_f32_e32 v2, v5, v6", "\tv_fmac_f32_dpp v3, v1, v2 row_ror:1"])[0]      # (only the first source moves between lanes)
    assert len(violations(["0000 <k>:", "\tv_permlane32_swap_b32_e32 v1, v2", "\ts_nop 0", "\tv_permlane16_swap_b32_e32 v2, v9"])[0]) == 1


def device_code(image):
    """The gfx950 code objects of a library: entries of its offload bundles (magic, count, then offset, size and target of each)."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := image.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", image, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", image, pos)
            target = image[pos + 24:pos + 24 + length]
            pos += 24 + length
            if size and target.endswith(b"gfx950"):
                yield image[at + offset:at + offset + size]
        at += len(magic)


@pytest.mark.skipif(not OBJDUMP.exists(), reason="no disassembler")
def test_two_wait_states_before_every_row_swap_and_dpp_read(tmp_path):
    parts = list(device_code(LIB.read_bytes()))
    assert len(parts) > 10

    def check(k):
        f = tmp_path / f"{k}.co"
        f.write_bytes(parts[k])
        p = subprocess.Popen([str(OBJDUMP), "-d", "--no-show-raw-insn", "--no-leading-addr", str(f)], stdout=subprocess.PIPE, text=True)
        result = violations(line.rstrip("\n") for line in p.stdout)
        assert p.wait() == 0
        return result

    with ThreadPoolExecutor(4) as ex:
        results = list(ex.map(check, range(len(parts))))
    assert sum(n for _, n in results) > 10000, "no such instructions found: has the disassembler's output changed?"
    bad = [v for found, _ in results for v in found]
    assert not bad, f"{len(bad)} reads too early, in {len({v[0] for v in bad})} kernels, e.g. {bad[:5]}"
