"""Wait states around the requests that are written as inline assembly.

The compiler keeps the distances that the hardware asks of a program for its own instructions, not
for those inside an assembly string.  The direct-to-LDS requests are such strings, so their
distances are checked in the machine code of the built library: between a vector-unit write of a scalar
register (v_readfirstlane, compares, carries) and a memory instruction that reads it lie five
wait states (a stale descriptor word would drop valid rows or lift the bounds check), between a scalar write
of m0 and a direct-to-LDS request one.  The dK/dV kernel at head size 64 writes its matrix instructions as strings too and
keeps its accumulators in registers that only those strings name: a vector instruction may read the
result of a 32x32x16 matrix instruction after 12 wait states, a matrix instruction that of a vector instruction after
two, and nothing but the strings may write these registers."""
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


def looking_back(ins):
    """found(i, states, hit): whether hit(instruction) holds on some way to instruction i, within `states` wait states."""
    place = {x[0]: i for i, x in enumerate(ins)}
    jumps = {}
    for i, x in enumerate(ins):
        if x[3] in place:
            jumps.setdefault(place[x[3]], []).append(i)

    def found(i, states, hit):
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
    return found


def vector_registers(text):
    return {(kind, r) for kind in "va" for r in registers(text, kind)}


def matrix_too_close(ins):
    """Descriptions of instructions that come too soon after a matrix instruction, or a matrix instruction too soon after
    a vector instruction."""
    found, bad = looking_back(ins), []
    for i, (at, op, operands, _) in enumerate(ins):
        first, _, rest = operands.partition(", ")
        if op.startswith("v_mfma"):
            reads = vector_registers(rest)
            if found(i, 2, lambda x: x[1].startswith("v_") and not x[1].startswith("v_mfma") and vector_registers(x[2].split(", ")[0]) & reads):
                bad.append("%x %s %s: written by the vector unit" % (at, op, operands))
        elif op.startswith(("v_", "ds_write", "global_store", "buffer_store", "scratch_store")):
            uses = vector_registers(operands)
            if found(i, 12, lambda x: x[1].startswith("v_mfma") and vector_registers(x[2].split(", ")[0]) & uses):
                bad.append("%x %s %s: result of a matrix instruction" % (at, op, operands))
    return bad


def accumulator_writes(ins):
    """(registers a0 .. a95 that anything but a matrix instruction writes, matrix instructions that write other ones of them than a whole
    accumulator).  Loads and reads of LDS may write accumulator registers directly; a swap writes both its operands."""
    plain, odd = [], []
    for at, op, operands, _ in ins:
        if op.startswith("v_mfma"):
            to = {r for r in registers(operands.partition(", ")[0], "a") if r < 96}
            if to and to not in [set(range(i, i + 16)) for i in (0, 16, 32, 48)]:
                odd.append("%x %s %s" % (at, op, operands))
        elif op.startswith("v_") or re.match(r"(ds|buffer|global|flat|scratch)_", op) and "store" not in op and "write" not in op:
            written = operands.split(", ")[:2 if "swap" in op else 1]
            plain += [r for x in written for r in registers(x, "a") if r < 96]
    return plain, odd


def too_close(ins):
    """Descriptions of the memory instructions that come too soon after the write of what they read."""
    found = looking_back(ins)
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


@pytest.mark.parametrize("lines,bad", [
    (("v_cvt_pk_bf16_f32 v8, v0, v1", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"), 1),
    (("v_cvt_pk_bf16_f32 v8, v0, v1", "s_nop 1", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"), 0),
    (("v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], a[64:67], v[16:31]", "s_nop 7", "v_exp_f32 v0, v20"), 1),
    (("v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], a[64:67], v[16:31]", "s_nop 7", "s_nop 3", "v_exp_f32 v0, v20"), 0),
    (("v_mfma_f32_32x32x16_bf16 a[16:31], v[4:7], v[8:11], a[16:31]", "v_exp_f32 v0, v20", "v_accvgpr_read_b32 v1, a16"), 1),
])
def test_the_check_of_matrix_instructions(lines, bad):
    (_, ins), = kernels(listing_of(*lines))
    assert len(matrix_too_close(ins)) == bad


@pytest.mark.parametrize("lines,plain,odd", [
    (("v_accvgpr_write_b32 a3, 0", "v_accvgpr_read_b32 v1, a16", "ds_write_b128 v0, a[4:7]", "global_store_dwordx4 v[0:1], a[8:11], off"), [3], 0),
    (("ds_read_b128 a[0:3], v0",), [0, 1, 2, 3], 0),
    (("buffer_load_dwordx4 a[92:95], v0, s[0:3], 0 offen",), [92, 93, 94, 95], 0),
    (("global_load_dword a7, v[0:1], off", "scratch_load_dword a9, off, off offset:16"), [7, 9], 0),
    (("v_accvgpr_mov_b32 a5, a96", "v_swap_b32 v0, a6"), [5, 6], 0),
    (("ds_read_b128 a[96:99], v0", "v_mfma_f32_32x32x16_bf16 a[16:31], v[4:7], v[8:11], a[16:31]"), [], 0),
    (("v_mfma_f32_32x32x16_bf16 a[64:79], v[4:7], v[8:11], a[64:79]", "v_mfma_f32_16x16x32_bf16 a[4:7], v[4:7], v[8:11], a[4:7]"), [], 2),
])
def test_the_check_of_accumulator_writes(lines, plain, odd):
    (_, ins), = kernels(listing_of(*lines))
    got = accumulator_writes(ins)
    assert sorted(got[0]) == plain and len(got[1]) == odd


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    mb.lib()                                            # the library is built
    d = tmp_path_factory.mktemp("listing")
    so = shutil.copy(mb.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(so)], check=True, capture_output=True, cwd=d)
    return [k for f in sorted(d.glob("lib.so.*gfx950"))
            for k in kernels(subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, capture_output=True, text=True).stdout)]


def test_requests_keep_their_distance(listings):
    requests, bad = 0, []
    for name, ins in listings:
        requests += sum(x[2].endswith(" lds") for x in ins)
        bad += ["%s: %s" % (name[:60], b) for b in too_close(ins)]
    assert requests > 1000, "the listings hold the direct-to-LDS requests"
    assert not bad, "%d in all, the first: %s" % (len(bad), bad[:3])


def test_matrix_instructions_of_the_dkv_kernel_keep_their_distance(listings):
    (ins,) = [ins for name, ins in listings if "attn_bwd_dkv_skew" in name]
    assert sum(x[1].startswith("v_mfma") for x in ins) >= 40
    assert not matrix_too_close(ins)
    # dK, dV and the K and V fragments, a0 .. a95: written once per item (cleared, loaded), otherwise by matrix instructions
    plain, odd = accumulator_writes(ins)
    assert sorted(plain) == list(range(96)) and not odd
