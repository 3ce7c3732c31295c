"""Wait states in the built gfx950 code. The compiler keeps them between its own instructions but does not look
into inline assembly, so the library's listing is read: a mask or scalar that one vector instruction writes is read by
another only after two wait states, a register that a DPP, lane-swap or matrix instruction reads is two old, and a
transcendental result one. (The distances are those the compiler itself keeps for gfx950.) Blocks are taken in the
order of the listing. No GPU."""
import os
import re
import struct
import subprocess

import pytest

import paper_2603_26110_amd as tq

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
pytestmark = pytest.mark.skipif(not os.path.exists(tq.lib_path) or not os.path.exists(OBJDUMP),
                                reason="libturboesm.so or llvm-objdump is missing")
# instructions from a write to a read of each kind, at least
LEAST = {"mask": 3, "dpp": 3, "swap": 3, "matrix": 3, "transcendental": 2}


def _code_objects(path):
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + length]:
                yield data[at + off:at + off + size]
            pos += 24 + length
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _registers(operand):
    operand = operand.split(" ")[0].strip("-|")
    if operand.startswith("vcc"):
        return ["vcc"]
    m = re.fullmatch(r"([vs])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return []
    lo, hi = (m[2], m[2]) if m[2] else (m[3], m[4])
    return [m[1] + str(i) for i in range(int(lo), int(hi) + 1)]


def too_early(listing):
    """[(kind, writer, reader)] of the reads in a listing that come too early."""
    found, now, written = [], 0, {}
    for line in listing.splitlines():
        if not line.startswith("\t"):
            if line.endswith(">:"):
                written = {}
            continue
        text = line.split("//")[0].strip()
        op, _, rest = text.partition(" ")
        now += int(rest) + 1 if op == "s_nop" else 1
        if not op.startswith("v_"):
            if op in ("s_branch", "s_endpgm"):
                written = {}
            elif rest and op != "s_nop":
                for r in _registers(rest.split(",")[0]):
                    written.pop(r, None)
            continue
        operands = [o.strip() for o in rest.split(",")]
        swap = op.startswith("v_permlane")
        outs = 2 if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", op) else 1
        reads = operands if swap or op.startswith("v_fmac") else operands[outs:]
        dpp = re.search(r"row_|quad_perm", rest) is not None
        for i, o in enumerate(reads):
            for r in _registers(o):
                if r not in written:
                    continue
                when, by = written[r]
                trans = re.match(r"v_(exp|log|rcp|rsq|sqrt|sin|cos)_", by)
                if not r.startswith("v") or r == "vcc":
                    kind = "mask"
                elif "mfma" in by:
                    continue                                     # (the compiler's own: none is read in assembly)
                elif dpp and (i == 0 or (op.startswith("v_fmac") and i == 1)):
                    kind = "dpp"
                elif swap or "mfma" in op:
                    kind = "swap" if swap else "matrix"
                elif trans and not re.match(r"v_(exp|log|rcp|rsq|sqrt|sin|cos)_", op):
                    kind = "transcendental"
                else:
                    continue
                if now - when < LEAST[kind]:
                    found.append((kind, by, text))
        for o in operands if swap else operands[:outs]:
            for r in _registers(o):
                written[r] = (now, text)
    return found


def test_the_reader_sees_each_kind():
    code = lambda *lines: "0000 <f>:\n" + "".join(f"\t{ln}   // 0:\n" for ln in lines)
    assert [k for k, _, _ in too_early(code("v_cmp_lt_f32_e32 vcc, v1, v2", "v_addc_co_u32_e32 v3, vcc, v3, v3, vcc"))] == ["mask"]
    assert [k for k, _, _ in too_early(code("v_cmp_lt_f32_e64 s[4:5], v1, v2", "s_nop 0", "v_cndmask_b32_e64 v3, 0, 1, s[4:5]"))] == ["mask", "mask"]
    assert not too_early(code("v_cmp_lt_f32_e32 vcc, v1, v2", "s_nop 1", "v_cndmask_b32_e32 v3, v1, v2, vcc"))
    assert [k for k, _, _ in too_early(code("v_mov_b32_e32 v4, v1", "v_nop", "v_fmac_f32_dpp v5, v4, v6 row_newbcast:3 row_mask:0xf bank_mask:0xf"))] == ["dpp"]
    assert [k for k, _, _ in too_early(code("v_mov_b32_e32 v4, v1", "v_permlane32_swap_b32_e32 v7, v4"))] == ["swap"]
    assert [k for k, _, _ in too_early(code("v_fma_mixhi_f16 v9, v1, v2, 0", "v_mfma_f32_32x32x16_f16 a[0:15], v[2:5], v[6:9], a[0:15]"))] == ["matrix"]
    assert [k for k, _, _ in too_early(code("v_rcp_f32_e32 v1, v2", "v_mul_f32_e32 v3, v1, v2"))] == ["transcendental"]


def test_no_register_is_read_too_early(tmp_path):
    instructions = 0
    for i, obj in enumerate(_code_objects(tq.lib_path)):
        path = tmp_path / f"{i}.o"
        path.write_bytes(obj)
        listing = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", str(path)], capture_output=True,
                                 text=True, check=True).stdout
        instructions += listing.count("\n\tv_")
        found = too_early(listing)
        assert not found, (len(found), found[:5])
    assert instructions > 10000
