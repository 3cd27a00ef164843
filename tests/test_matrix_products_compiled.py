"""Waits around the matrix products that are written as instructions of their own (csrc/gemm.hip, `mfma_add`): the compiler does
not know them as products, so it puts no wait states between them and a vector instruction that writes a source just
before one or touches a result too soon after.  What the sources arrange is checked on the built library, along every path through
the kernels that use them."""
import os
import re
import struct
import subprocess

import pytest

import paper_1806_00187_amd as A

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
STRIP_KERNELS = (r"gemm_persistent_kernelI", r"\d+gemm_kernelI", r"wgrad_group_kernelILi\d+ELi\d+ELi2E")
BEFORE = 2    # wait states between a vector instruction that writes a source and the product
BEHIND = 19   # and between a product and whatever else touches its result: the longest of any product


def code_objects(library):
    """The gfx950 code objects of a shared library built by hipcc."""
    data = open(library, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.end()
        (n,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name:
                yield data[m.start() + offset:m.start() + offset + size]


def registers(operand):
    """'v[4:7]' -> {v4, v5, v6, v7}; scalars, constants and modifiers -> {}."""
    m = re.search(r"\b([va])\[(\d+):(\d+)\]", operand)
    if m:
        return {m[1] + str(r) for r in range(int(m[2]), int(m[3]) + 1)}
    m = re.search(r"\b([va])(\d+)\b", operand)
    return {m[1] + m[2]} if m else set()


class Instruction:
    def __init__(self, text, address):
        self.text, self.address = text, address
        self.name, _, rest = text.partition(" ")
        operands = [registers(o) for o in rest.split(",")]
        self.product = "_mfma_" in self.name
        self.result = operands[0]
        self.sources = set().union(*operands[1:3]) if self.product else set()
        self.touched = set().union(*operands)
        written = 0 if self.name.startswith("v_cmp") or not self.name.startswith("v_") or self.product else 2 if "_swap_" in self.name else 1
        self.written = set().union(*operands[:written])
        self.states = int(rest) + 1 if self.name == "s_nop" else 1


def kernels(listing):
    """name -> (instructions, successors of each) from a disassembler's listing."""
    out, name, start, code, jumps = {}, None, 0, [], []

    def close():
        if name is None:
            return
        index = {c.address: i for i, c in enumerate(code)}
        nexts = []
        for i, (c, jump) in enumerate(zip(code, jumps)):
            n = [] if c.name in ("s_branch", "s_endpgm") else [i + 1]
            if jump is not None:
                n.append(index[jump])
            nexts.append([j for j in n if j < len(code)])
        out[name] = (code, nexts)

    for line in listing.splitlines():
        m = re.match(r"([0-9a-f]+) <(.+)>:", line)
        if m:
            close()
            name, start, code, jumps = m[2], int(m[1], 16), [], []
            continue
        m = re.match(r"\s+([a-z]\w+.*?)\s*// ([0-9A-F]+):(.*)", line)
        if not m:
            continue
        c = Instruction(m[1], int(m[2], 16))
        assert not re.match(r"s_(set|swap|get)pc|s_call", c.name), c.text
        jump = None
        if c.name.startswith(("s_branch", "s_cbranch")):
            to = re.search(r"<.+?(?:\+0x([0-9a-f]+))?>\s*$", m[3])
            jump = start + int(to[1] or "0", 16)
        code.append(c)
        jumps.append(jump)
    close()
    return out


def too_soon(code, nexts):
    """(first instruction, second, what the second does too soon) along every path."""
    found = []
    for i, c in enumerate(code):
        regs, limit = (c.result, BEHIND) if c.product else (c.written, BEFORE)
        if not regs:
            continue
        todo, best = [(j, 0) for j in nexts[i]], {}
        while todo:
            j, passed = todo.pop()
            if passed >= limit or best.get(j, limit) <= passed:
                continue
            best[j] = passed
            o = code[j]
            if c.product:
                again = o.product and o.result == c.result and not o.sources & regs  # (the next addend of the same sum)
                bad = o.touched & regs and not again
            else:
                bad = o.product and o.touched & regs
            if bad:
                found.append((c.text, o.text, f"{passed} wait states behind it"))
            elif c.product or not regs <= o.written:
                todo += [(k, passed + o.states) for k in nexts[j]]
    return found


def test_products_of_the_built_library_wait_for_their_operands_and_are_waited_for(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    seen = dict.fromkeys(STRIP_KERNELS, 0)
    for n, code in enumerate(code_objects(os.path.join(os.path.dirname(A.__file__), "libnmt.so"))):
        path = tmp_path / f"{n}.o"
        path.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], check=True, capture_output=True, text=True).stdout
        for name, (instructions, nexts) in kernels(listing).items():
            kind = next((k for k in STRIP_KERNELS if re.search(k, name)), None)
            if kind:
                seen[kind] += sum(c.product for c in instructions)
                assert not too_soon(instructions, nexts), name
    assert all(seen.values()), seen


LOOP = """0000000000000100 <k>:
	v_mov_b32_e32 v9, v8                                       // 000000000100: 00000000
	s_nop 1                                                    // 000000000104: 00000000
	v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[12:15], v[0:3]  // 000000000108: 00000000
	{0:<58} // 000000000110: 00000000
	s_cbranch_scc1 65533                                       // 000000000114: 00000000 <k+0x4>
	s_nop 14                                                   // 000000000118: 00000000
	s_nop {1}                                                    // 00000000011C: 00000000
	v_add_f32_e32 v4, v3, v3                                   // 000000000120: 00000000
	s_endpgm                                                   // 000000000124: 00000000
"""


@pytest.mark.parametrize("between,wait,faults", [
    ("s_nop 0", 1, 0),
    ("s_nop 0", 0, 1),                       # the result read 18 wait states behind the product
    ("v_mov_b32_e32 v2, v20", 1, 1),         # the result overwritten
    ("ds_write_b128 v20, v[2:5]", 1, 1),     # stored
    ("v_mov_b32_e32 v15, v20", 1, 0),        # a source written 3 wait states ahead of the next round's product
    ("v_mfma_f32_16x16x32_f16 v[24:27], v[0:3], v[12:15], v[24:27]", 1, 1)])   # the result as another product's operand
def test_the_check_finds_what_comes_too_soon(between, wait, faults):
    (code, nexts), = kernels(LOOP.format(between, wait)).values()
    assert len(too_soon(code, nexts)) == faults
    # without the wait ahead of the product
    (code, nexts), = kernels(LOOP.format("s_nop 0", 1).replace("s_nop 1 ", "s_nop 0 ", 1)).values()
    assert len(too_soon(code, nexts)) == 1
