"""The kernels read fragments from LDS in inline asm and wait for them by hand (``lds_read4_async`` and its
neighbours in ``csrc/common.h``): to the compiler such a register is written at once, so nothing but its own choice of
registers and places keeps it from copying or reusing one that is still on its way.  The built code is checked instead: on no
path through a kernel does an instruction touch a register that an LDS read has not filled yet."""
import os
import re
import struct
import subprocess

import pytest

from paper_2512_04939_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
REG = re.compile(r"\bv(?:(\d+)\b|\[(\d+):(\d+)\])")
WAIT = re.compile(r"lgkmcnt\((\d+)\)")
OLDEST = 16          # the counter's range: older reads need no finer age


def _vgprs(text):
    out = set()
    for one, lo, hi in REG.findall(text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def early_uses(code):
    """``code``: [(address, mnemonic, operands, branch target or None)] of one kernel.  Addresses of instructions that touch a
    register whose LDS read may still be under way."""
    at = {c[0]: i for i, c in enumerate(code)}
    # per instruction, on entry: register -> LDS operations issued since its read (they complete in order)
    entry, todo, bad = {0: {}}, [0], set()
    while todo:
        i = todo.pop()
        state = dict(entry[i])
        while True:
            addr, op, args, target = code[i]
            if op == "s_waitcnt":
                n = WAIT.search(args)
                if n:
                    state = {r: a for r, a in state.items() if a < int(n[1])}
            elif not op.startswith("s_"):
                regs = _vgprs(args)
                if not regs.isdisjoint(state):
                    bad.add(addr)
                if op.startswith("ds_"):
                    state = {r: min(a + 1, OLDEST) for r, a in state.items()}
                    if "read" in op or "permute" in op or "swizzle" in op or "_rtn" in op:
                        state.update(dict.fromkeys(_vgprs(args.split(",")[0]), 0))
            follow = [] if op in ("s_endpgm", "s_branch") else [i + 1]
            if target is not None:
                follow.append(at[target])
            if follow == [i + 1] and i + 1 not in entry:
                i += 1
                continue
            for j in follow:
                old = entry.get(j)
                new = dict(state) if old is None else {r: min(old.get(r, OLDEST), state.get(r, OLDEST)) for r in {**old, **state}}
                if new != old:
                    entry[j] = new
                    todo.append(j)
            break
    return sorted(bad)


def _kernels(text):
    """{name: code} of a disassembly."""
    out, code = {}, None
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if head:
            base, code = int(head[1], 16), out.setdefault(head[2], [])
            continue
        ins = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<.*\+0x([0-9a-f]+)>|<.*>)?$", line)
        if ins and code is not None:
            op, args, addr, off = ins.groups()
            branch = op.startswith("s_cbranch") or op == "s_branch"
            code.append((int(addr, 16), op, args, (base + int(off or "0", 16)) if branch else None))
    return out


def _disassembly(tmp_path):
    """Text of every gfx950 code object in the built library."""
    fat = str(tmp_path / "fat")
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), "--dump-section=.hip_fatbin=" + fat, build.LIB, str(tmp_path / "rest")])
    data = open(fat, "rb").read()
    start = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while start >= 0:
        count, p = struct.unpack_from("<Q", data, start + 24)[0], start + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                obj = tmp_path / f"{start + off}.o"
                obj.write_bytes(data[start + off:start + off + size])
                yield subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", str(obj)], capture_output=True, text=True, check=True).stdout
            p += 24 + n
        start = data.find(b"__CLANG_OFFLOAD_BUNDLE__", start + 24)


def test_no_register_is_touched_before_its_lds_read_has_ended(tmp_path):
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no disassembler")
    kernels, reads = 0, 0
    for text in _disassembly(tmp_path):
        for name, code in _kernels(text).items():
            kernels += 1
            reads += sum(op.startswith("ds_read") for _, op, _, _ in code)
            assert early_uses(code) == [], name
    assert kernels > 80 and reads > 2000


def _code(*lines):
    return [(i, *(line.split(None, 1) + [""])[:2], None) for i, line in enumerate(lines)]


READ2 = ("ds_read_b128 v[0:3], v8", "ds_read_b128 v[4:7], v8 offset:1024")


@pytest.mark.parametrize("lines,bad", [
    (READ2 + ("s_waitcnt lgkmcnt(0)", "v_add_u32_e32 v9, v3, v7", "s_endpgm"), []),
    (READ2 + ("s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v9, v3", "s_endpgm"), []),
    (READ2 + ("s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v9, v4", "s_endpgm"), [3]),           # the newer one is under way
    (READ2 + ("s_waitcnt vmcnt(0)", "v_mov_b32_e32 v9, v0", "s_endpgm"), [3]),
    (READ2 + ("v_mfma_f32_32x32x16_bf16 v[16:31], v[2:5], v[10:13], v[16:31]", "s_endpgm"), [2]),
    (READ2 + ("v_mov_b32_e32 v5, v9", "s_waitcnt lgkmcnt(0)", "s_endpgm"), [2]),           # written while the read is
    (READ2 + ("ds_write_b32 v9, v10", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v9, v4", "s_endpgm"), []),
    (("ds_bpermute_b32 v1, v2, v3", "v_mov_b32_e32 v9, v1", "s_endpgm"), [1]),
])
def test_early_uses_on_straight_code(lines, bad):
    assert early_uses(_code(*lines)) == bad


def test_early_uses_follows_branches():
    code = _code("v_mov_b32_e32 v9, v0", "ds_read_b128 v[0:3], v8", "s_cbranch_scc1 x", "s_waitcnt lgkmcnt(0)", "s_endpgm")
    code[2] = (*code[2][:3], 0)                                   # back to the start without a wait
    assert early_uses(code) == [0, 1]
    code[2] = (*code[2][:3], 3)
    assert early_uses(code) == []
