"""Matrix-core results in the built library are not read too early on any path.

The hardware does not hold back a vector instruction that reads a matrix
product's registers before they are written: the compiler counts the wait
states.  It counts them along one path into a block only, so a short branch
between a product and its first read (a rescaling that most rows skip) can leave
the path around it without them, and such a read gives a register's old value.
This walks every path of every kernel from each product to the first use of its
registers.
"""

import os
import re
import shutil
import subprocess

import pytest

from paper_2608_09307_amd import linsimp as L

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# wait states from a product's issue to a read or write of its registers by
# anything but the next product of its chain (what the compiler keeps in
# straight code): by passes, 16 for the float32 product and 8 for the 16-bit ones
WAIT = {"v_mfma_f32_32x32x2_f32": 18, "v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_32x32x16_f16": 12}

REG = re.compile(r"\b([va])(\d+)\b|\b([va])\[(\d+):(\d+)\]")


def _regs(text):
    out = set()
    for m in REG.finditer(text):
        if m.group(1):
            out.add((m.group(1), int(m.group(2))))
        else:
            out.update((m.group(3), i) for i in range(int(m.group(4)), int(m.group(5)) + 1))
    return out


def _operands(text):
    return re.split(r",\s*(?![^\[]*\])", text) if text else []


def _kernels(listing):
    """(name, [(opcode, operands, address, branch target)]) of a disassembly."""
    base, name, ins = 0, None, []
    for line in listing.splitlines():
        m = re.match(r"^([0-9a-f]{16}) <(\S+)>:", line)
        if m:
            if ins:
                yield name, ins
            base, name, ins = int(m.group(1), 16), m.group(2), []
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):(.*)$", line)
        if m:
            to = re.search(r"<[^>+]+(?:\+0x([0-9a-f]+))?>", m.group(4))
            ins.append((m.group(1), m.group(2), int(m.group(3), 16),
                        base + int(to.group(1) or "0", 16) if to else None))
    if ins:
        yield name, ins


def early_reads(listing):
    bad, seen = [], set()
    for name, ins in _kernels(listing):
        at = {a: i for i, (_, _, a, _) in enumerate(ins)}
        for i, (op, text, _, _) in enumerate(ins):
            if not op.startswith("v_mfma"):
                continue
            seen.add(op)
            need, dst = WAIT[op], _regs(_operands(text)[0])
            best, stack = {}, [(i + 1, 0)]
            while stack:
                p, w = stack.pop()
                while p < len(ins) and w < need and best.get(p, need) > w:
                    best[p] = w
                    o, t, _, to = ins[p]
                    a = _operands(t)
                    if o.startswith("v_mfma"):
                        if (_regs(a[1]) | _regs(a[2])) & dst:
                            bad.append((name, w, op, text, o, t))
                            break
                        if (_regs(a[0]) | _regs(a[3])) & dst:
                            break                           # the chain's next product: the hardware waits
                    elif not o.startswith("s_") and a:
                        if _regs(t) & dst:                  # read, or written over
                            bad.append((name, w, op, text, o, t))
                            break
                    if o == "s_endpgm":
                        break
                    w += int(t, 0) + 1 if o == "s_nop" else 1
                    if o == "s_branch":
                        p = at[to]
                        continue
                    if o.startswith("s_cbranch"):
                        stack.append((at[to], w))
                    p += 1
    return bad, seen


def test_walk_finds_the_path_around_a_branch():
    head = "0000000000001000 <k>:\n"
    body = ["v_mfma_f32_32x32x2_f32 a[0:15], v2, v3, a[0:15]", "s_cbranch_vccnz 2", "v_mul_f32_e32 v8, s2, v8",
            "s_nop 15", "v_accvgpr_read_b32 v9, a15", "s_endpgm"]

    def listing(lines):
        out = head
        for k, x in enumerate(lines):
            to = " BF870002 <k+0x10>" if x.startswith("s_cbranch") else " 00000000"
            out += f"\t{x}   // {0x1000 + 4 * k:012X}:{to}\n"
        return out

    assert len(early_reads(listing(body))[0]) == 1                  # one instruction on the taken path
    assert not early_reads(listing(body[:1] + ["s_nop 15"] + body[1:]))[0]
    assert not early_reads(listing(body[:1] + body[2:3] * 2 + body[3:]))[0]         # straight: 18


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_product_is_read_early(tmp_path):
    lib = shutil.copy(L.lib_path(), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", os.path.basename(lib)], cwd=tmp_path, check=True, capture_output=True)
    seen = set()
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" in f:
            res = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True,
                                 capture_output=True, text=True)
            bad, ops = early_reads(res.stdout)
            assert not bad, bad[:4]
            seen |= ops
    assert seen == set(WAIT)
