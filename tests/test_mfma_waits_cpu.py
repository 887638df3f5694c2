"""A matrix instruction writes its sums some wait states after it is issued, and nothing but the instructions in between keeps a later read of them
waiting.  hipcc counts those, but of several ways from the product to the read it may follow one: a branch that passes by other work is then a
shorter way nobody counted.  So the built library is followed here: from every matrix instruction along every way to what takes its result."""
import os
import re
import struct
import subprocess

import pytest

from paper_2604_25422_amd import _build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
# wait states from the instruction to a read of its result, and passes, for which it holds up the next one of its kind (four cycles each)
STATES = {"v_mfma_f32_16x16x4_f32": (10, 8), "v_mfma_f32_16x16x16_bf16": (8, 4), "v_mfma_f32_16x16x32_bf16": (8, 4), "v_mfma_f32_32x32x16_bf16": (12, 8)}
REGISTERS = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(text):
    out = set()
    for kind, a, b, one in REGISTERS.findall(text):
        base = 0 if kind == "v" else 1024
        out.update(range(base + int(a or one), base + int(b or one) + 1))
    return out


def functions(lines):
    """(name, instructions, label -> index) of every function of a disassembly."""
    name, ins, labels = None, [], {}
    for line in lines:
        m = re.match(r"^[0-9a-f]+ <(\w+)>:", line)
        if m and re.fullmatch(r"L\d+", m[1]):
            labels[m[1]] = len(ins)
        elif m:
            if ins:
                yield name, ins, labels
            name, ins, labels = m[1], [], {}
        elif line[:1].isspace():
            text = line.split("//")[0].split()
            if text:
                ins.append((text[0], " ".join(text[1:])))
    if ins:
        yield name, ins, labels


def reads(op, args):
    """Vector registers an instruction takes (of one that writes a register, the operands behind the first)."""
    if not op.startswith(("v_", "ds_", "buffer_", "global_", "flat_")):
        return set()
    whole = "write" in op or "store" in op or args.endswith(" lds") or op.startswith(("v_cmp", "v_read", "v_fmac", "v_mac", "v_swap"))
    return registers(args if whole else args.partition(",")[2])


def short_ways(ins, labels):
    """(instruction, reader, wait states) of results that are taken before they are there."""
    found = []
    for at, (op, args) in enumerate(ins):
        if not op.startswith("v_mfma"):
            continue
        need, passes = STATES[op]
        result = registers(args.partition(", ")[0])
        ways, best = [(at + 1, 0)], {}
        while ways:
            i, states = ways.pop()
            if states >= need or i >= len(ins) or best.get(i, need) <= states:
                continue
            best[i] = states
            o, a = ins[i]
            if o == "s_nop":
                ways.append((i + 1, states + 1 + int(a, 0)))
            elif o.startswith("s_cbranch"):
                ways += [(labels[a], states + 1), (i + 1, states + 1)]
            elif o == "s_branch":
                ways.append((labels[a], states + 1))
            elif o in ("s_endpgm", "s_setpc_b64"):
                continue
            elif o.startswith("v_mfma"):
                d, rest = a.split(", ", 1)
                c = rest.split(", ")[2]
                if (registers(", ".join(rest.split(", ")[:2])) & result) or (o != op and registers(c) & result):
                    found.append((at, i, states))
                elif not registers(d) & result:                          # (sums handed to the next product wait in the matrix pipe)
                    ways.append((i + 1, states + passes))
            elif reads(o, a) & result:
                found.append((at, i, states))
            else:
                ways.append((i + 1, states + 1))
    return found


def code_objects(path):
    """The gfx950 code objects of a library."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(magic))[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if triple.endswith(b"gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 1)


def test_a_short_way_is_found():
    lines = ["0000000000000100 <kernel>:", "\tv_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], v[4:7]", "\ts_cbranch_scc1 L0",
             "\tv_mfma_f32_16x16x32_bf16 v[16:19], v[8:11], v[12:15], v[16:19]", "\ts_nop 7", "0000000000000120 <L0>:", "\tv_fma_f32 v1, v4, v2, v3", "\ts_endpgm"]
    (name, ins, labels), = functions(lines)
    assert name == "kernel" and short_ways(ins, labels) == [(0, 4, 1)]
    ins[0:1] = [ins[0], ("s_nop", "6")]
    assert short_ways(ins, {"L0": labels["L0"] + 1}) == []


def test_no_result_is_taken_before_it_is_there(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(_build.LIB_PATH):
        _build.build()
    products, wrong = 0, []
    for n, code in enumerate(code_objects(_build.LIB_PATH)):
        path = tmp_path / f"{n}.co"
        path.write_bytes(code)
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(path)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        for name, ins, labels in functions(r.stdout.splitlines()):
            products += sum(op.startswith("v_mfma") for op, _ in ins)
            wrong += [f"{name}: {ins[at]} is {states} wait states in front of {ins[i]}" for at, i, states in short_ways(ins, labels)]
    assert products > 10000
    assert not wrong, f"{len(wrong)}, among them " + "; ".join(wrong[:4])
