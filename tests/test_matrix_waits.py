"""Wait states around the matrix instructions, in the AMD assembly of the library as built (host only).

Much of the matrix work is inline assembly, and the compiler puts no wait states around instructions it does not see.
This follows every path of every kernel that holds a matrix instruction and counts, as the compiler's own forms do: an
instruction is one wait state, s_nop n is n + 1.  The rules (CDNA3 ISA guide, tables of manually inserted wait states and of
required independent instructions; the compiler's own figures for gfx950):
  * a VGPR a vector instruction has written is read by a matrix instruction (any operand, scales included) no earlier
    than 2 wait states behind it;
  * the result of a matrix instruction of p passes is touched by anything but a matrix instruction that adds to exactly
    these registers no earlier than p + 4 wait states behind it (fp32 operands: p + 2);
  * an SGPR a vector instruction has written is read by a memory instruction no earlier than 5 wait states behind it.
"""
import functools
import os
import re
import struct
import subprocess

import pytest

from paper_2501_05460_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
PASSES = {"4x4x4": 2, "16x16x4": 8, "16x16x16": 4, "16x16x32": 4, "16x16x128": 8, "32x32x2": 16, "32x32x16": 8, "32x32x64": 16}
REG = re.compile(r"(?<![\w.])([vas])(?:(\d+)|\[(\d+):(\d+)\])(?!\w)|\b(vcc)\b")


def code_objects(path):
    """The gfx950 code objects of a shared library: bundles of (offset, size, triple) entries behind a magic word."""
    data, at, magic = open(path, "rb").read(), 0, b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + n]:
                yield data[at + off:at + off + size]
            entry += 24 + n
        at += 24


@functools.lru_cache(maxsize=None)
def regs(text):
    out = set()
    for kind, one, lo, hi, vcc in REG.findall(text):
        if vcc:
            out.add("vcc")
        else:
            out.update(f"{kind}{i}" for i in range(int(one or lo), int(one or hi) + 1))
    return frozenset(out)


def is_vector(name):
    return name.startswith("v_") and not name.startswith("v_mfma")


def is_memory(name):
    return name.startswith(("global_", "buffer_", "scratch_", "flat_"))


class Inst:
    """One instruction: its name, the registers it writes and reads, its wait states and the instructions behind it."""

    def __init__(self, name, operands):
        self.name, self.next = name, []
        ops = [regs(o) for o in operands.split(", ")] if operands else [frozenset()]
        first, rest = ops[0], frozenset().union(*ops[1:])
        self.writes, self.reads = first, rest
        self.states = int(operands.split()[0], 0) + 1 if name == "s_nop" else 1
        if name.startswith(("v_permlane16_swap", "v_permlane32_swap", "v_swap")):
            self.writes, self.reads = first | rest, first | rest
        elif name.startswith("v_"):
            if re.match(r"v_(add|sub|subrev|addc|subb)_co|v_mad_[iu]64|v_div_scale", name):   # carry or flag out
                self.writes = first | ops[1]
            if name.startswith(("v_fmac", "v_dot2c", "v_pk_fmac", "v_writelane")) or "dst_sel" in operands or "op_sel" in operands or "row_" in operands or "quad_perm" in operands:
                self.reads = first | rest   # reads the old destination
        elif "store" in name or "atomic" in name or "lds" in name or name.startswith("ds_write") or name.startswith("s_cmp"):
            self.writes, self.reads = frozenset(), first | rest
        self.mfma = name.startswith("v_mfma")
        if self.mfma:
            fp32 = name.endswith("_f32") and name.count("f32") == 2
            self.result_wait = PASSES[re.search(r"\d+x\d+x\d+", name).group()] + (2 if fp32 else 4)
            self.c, self.factors = ops[3], frozenset().union(ops[1], ops[2], *ops[4:])


def kernels(listing):
    """name -> instructions of every function that holds a matrix instruction."""
    for body in re.split(r"\n(?=[0-9a-f]{16} <)", listing)[1:]:
        if "v_mfma" not in body:
            continue
        lines = body.splitlines()
        start, name = re.match(r"([0-9a-f]+) <(.*)>:", lines[0]).groups()
        by_addr, order, jumps = {}, [], []
        for line in lines[1:]:
            m = re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]{12}): [0-9A-F ]+(?:<.*\+0x([0-9a-f]+)>)?", line)
            if not m:
                continue
            op, operands, addr, target = m.groups()
            inst = Inst(op, operands)
            by_addr[int(addr, 16)] = inst
            if op.startswith(("s_branch", "s_cbranch")):
                jumps.append((inst, int(start, 16) + int(target or "0", 16)))
            order.append(inst)
        for a, b in zip(order, order[1:]):
            if not a.name.startswith(("s_endpgm", "s_branch", "s_setpc")):
                a.next.append(b)
        for inst, to in jumps:
            inst.next.append(by_addr[to])
        yield name, order


def reached(inst, limit):
    """(instruction, wait states in between) for everything that may run fewer than `limit` wait states behind inst."""
    best, work = {}, [(n, 0) for n in inst.next]
    while work:
        at, gap = work.pop()
        if gap >= limit or best.get(at, limit) <= gap:
            continue
        best[at] = gap
        work += [(n, gap + at.states) for n in at.next]
    return best.items()


def operand_faults(order):
    for inst in order:
        if not is_vector(inst.name):
            continue
        vector = {r for r in inst.writes if r[0] in "va" and r != "vcc"}
        scalar = inst.writes - vector
        for at, gap in reached(inst, 5 if scalar else 2):
            if at.mfma and gap < 2 and at.reads & vector:
                yield "operand of a matrix instruction", inst, at, gap
            if is_memory(at.name) and at.reads & scalar:
                yield "scalar register of a memory instruction", inst, at, gap


def result_faults(order):
    for inst in order:
        if not inst.mfma:
            continue
        for at, gap in reached(inst, inst.result_wait):
            if at.mfma:
                touched = at.factors & inst.writes or (at.c & inst.writes and at.c != inst.writes)
            else:
                touched = at.reads & inst.writes or (is_vector(at.name) and at.writes & inst.writes)
            if touched:
                yield "result of a matrix instruction", inst, at, gap


@pytest.fixture(scope="module")
def built_kernels(tmp_path_factory):
    if not os.path.exists(B.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("needs the built library and llvm-objdump")
    file, out = tmp_path_factory.mktemp("code") / "code.elf", {}
    for blob in code_objects(B.LIB_PATH):
        file.write_bytes(blob)
        out.update(kernels(subprocess.run([OBJDUMP, "-d", str(file)], capture_output=True, text=True, check=True).stdout))
    assert len(out) > 50
    return out


def check(built, faults):
    found = [f"{name}: {what}: {a.name} {sorted(a.writes)[:4]} -> {b.name}, {gap} wait states"
             for name, order in built.items() for what, a, b, gap in faults(order)]
    assert not found, f"{len(found)} in {len({f.split(':')[0] for f in found})} kernels:\n" + "\n".join(found[:40])


def test_operands_are_written_early_enough(built_kernels):
    check(built_kernels, operand_faults)


def test_results_are_touched_late_enough(built_kernels):
    check(built_kernels, result_faults)
