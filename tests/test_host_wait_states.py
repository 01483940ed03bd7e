"""Wait states around the requests that are written as inline assembly.

The compiler keeps the distances that the hardware asks of a program for its own instructions, not
for those inside an assembly string.  The direct-to-LDS requests are such strings, so their
distances are checked in the machine code of the built library: between a vector-unit write of a scalar
register (v_readfirstlane, compares, carries) and a memory instruction that reads it lie five
wait states (a stale descriptor word would drop valid rows or lift the bounds check), between a scalar write
of m0 and a direct-to-LDS request one."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_18710_amd import binding as mb

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def registers(text, kind="s"):
    out = set()
    for one, lo, hi in re.findall(r"(?<![a-z_0-9])%s(?:(\d+)|\[(\d+):(\d+)\])" % kind, text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def kernels(listing):
    """[(name, [(address, opcode, operands, branch target or None)])] of an llvm-objdump listing."""
    out = []
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if head:
            out.append((head.group(2), int(head.group(1), 16), []))
            continue
        text, _, note = line.partition("//")
        at = re.match(r"\s*([0-9A-F]+):", note)
        if not out or not text.strip() or not at:
            continue
        op, _, operands = text.strip().partition(" ")
        to = re.search(r"\+0x([0-9a-f]+)>\s*$", note) if op.startswith(("s_cbranch", "s_branch")) else None
        out[-1][2].append((int(at.group(1), 16), op, operands, out[-1][1] + int(to.group(1), 16) if to else None))
    return [(name, ins) for name, _, ins in out]


def vector_unit_scalar_writes(op, operands):
    if not op.startswith("v_"):
        return set()
    parts = operands.split(", ")
    if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
        return registers(parts[0])
    if ("_co_" in op or op.startswith(("v_div_scale", "v_mad_u64", "v_mad_i64"))) and len(parts) > 1:
        return registers(parts[1])
    return set()


def too_close(ins):
    """Descriptions of the memory instructions that come too soon after the write of what they read."""
    place = {x[0]: i for i, x in enumerate(ins)}
    jumps = {}
    for i, x in enumerate(ins):
        if x[3] in place:
            jumps.setdefault(place[x[3]], []).append(i)

    def found(i, states, hit):                          # on some way to instruction i, within `states` wait states
        work, seen = [(i, states)], set()
        while work:
            i, left = work.pop()
            if left <= 0 or (i, left) in seen:
                continue
            seen.add((i, left))
            before = list(jumps.get(i, []))
            if i > 0 and ins[i - 1][1] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                before.append(i - 1)
            for b in before:
                if hit(ins[b]):
                    return True
                work.append((b, left - (int(ins[b][2].split()[0], 0) + 1 if ins[b][1] == "s_nop" else 1)))
        return False

    bad = []
    for i, (at, op, operands, _) in enumerate(ins):
        if not op.startswith(("buffer_load", "buffer_store", "buffer_atomic", "global_", "scratch_")):
            continue
        reads = registers(operands)
        if found(i, 5, lambda x: vector_unit_scalar_writes(x[1], x[2]) & reads):
            bad.append("%x %s %s: a scalar register written by the vector unit" % (at, op, operands))
        if operands.endswith(" lds") and found(i, 1, lambda x: x[1].startswith("s_") and x[2].startswith("m0,")):
            bad.append("%x %s %s: m0" % (at, op, operands))
    return bad


def listing_of(*lines):
    return "0000000000001000 <k>:\n" + "".join("\t%s // %012X: 00000000\n" % (l, 0x1000 + 4 * i) for i, l in enumerate(lines))


@pytest.mark.parametrize("lines,bad", [
    (("v_readfirstlane_b32 s6, v3", "s_add_i32 s20, s21, 4", "s_mov_b32 m0, s20", "s_nop 0", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"), 1),
    (("v_readfirstlane_b32 s6, v3", "s_nop 4", "s_mov_b32 m0, s20", "s_nop 0", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"), 0),
    (("v_readfirstlane_b32 s8, v3", "s_mov_b32 m0, s20", "s_nop 0", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"), 0),
    (("s_mov_b32 m0, s20", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"), 1),
    (("v_cmp_gt_u32_e64 s[2:3], v0, v1", "s_nop 3", "global_load_dword v1, v2, s[2:3]"), 1),
])
def test_the_check_itself(lines, bad):
    (_, ins), = kernels(listing_of(*lines))
    assert len(ins) == len(lines) and len(too_close(ins)) == bad


def test_requests_keep_their_distance(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    mb.lib()                                            # the library is built
    so = shutil.copy(mb.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(so)], check=True, capture_output=True, cwd=tmp_path)
    requests, bad = 0, []
    for f in sorted(tmp_path.glob("lib.so.*gfx950")):
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, capture_output=True, text=True).stdout
        for name, ins in kernels(listing):
            requests += sum(x[2].endswith(" lds") for x in ins)
            bad += ["%s: %s" % (name[:60], b) for b in too_close(ins)]
    assert requests > 1000, "the listings hold the direct-to-LDS requests"
    assert not bad, "%d in all, the first: %s" % (len(bad), bad[:3])
