"""Loads issued by inline assembly are waited for by hand, so the compiler takes their destination for valid
at the statement itself: a copy or a spill that it puts behind the load reads the register before the data is
there, and the load then lands in a register that holds something else by that time, an address for
instance.  Reads the code generated for every kernel that has such loads: nothing moves a loaded register
before a wait.  (Moves only: whether a wait is the right one for a use that the source has is for the source
to say, and the walk below also takes paths that no execution takes.)"""
import os
import re
import subprocess

import pytest

from paper_2605_08527_amd import build

FILES = ["gemm_mid", "gemm_decode", "gemm_bf16", "lora_small", "gemm_wide"]


def _registers(operand):
    m = re.match(r"^-?\|?([va])\[(\d+):(\d+)\]", operand)
    if m:
        return [m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)]
    m = re.match(r"^-?\|?([va]\d+)\b", operand)
    return [m.group(1)] if m else []


def _functions(text):
    """(name, basic blocks in order) of the kernels: {label: [(text, op, operands, inline assembly)]}"""
    name = None
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m and name is None:
            name, blocks, label, asm = m.group(1), {"": []}, "", False
            continue
        if name is None:
            continue
        if line.startswith(".Lfunc_end"):
            yield name, blocks
            name = None
            continue
        asm = "#ASMSTART" in line or (asm and "#ASMEND" not in line)
        s = line.split(";")[0].strip()
        m = re.match(r"^(\.\w+):", s)
        if m:
            label = m.group(1)
            blocks[label] = []
        elif s and not s.startswith("."):
            op, _, rest = s.partition(" ")
            blocks[label].append((s, op, [t.strip() for t in rest.split(",")], asm))


MOVES = re.compile(r"v_mov|v_swap|v_pk_mov|v_accvgpr|scratch_store|v_writelane")


def early_moves(blocks):
    """Moves of a register that an inline-assembly load writes, on some path with no wait in between."""
    order = list(blocks)
    after = dict(zip(order, order[1:]))
    state, work, found = {"": frozenset()}, [""], []

    def reach(label, pending):
        if label is not None and not (label in state and pending <= state[label]):
            state[label] = state.get(label, frozenset()) | pending
            work.append(label)

    while work:
        label = work.pop()
        pending = state[label]                       # {(counter, register)}
        for s, op, operands, asm in blocks[label]:
            if op == "s_waitcnt":
                pending = frozenset(p for p in pending if p[0] not in s)
                continue
            if op == "s_barrier":                    # (the kernels meet with their own requests waited for)
                pending = frozenset()
            if op == "s_branch":
                reach(operands[0], pending)
                break
            if op.startswith("s_cbranch"):
                reach(operands[0], pending)
            if op == "s_endpgm":
                break
            stores = "store" in op or op.startswith(("ds_write", "s_"))
            sources = {r for t in (operands if stores else operands[1:]) for r in _registers(t)}
            if MOVES.match(op) and any(r in sources for _, r in pending):
                found.append(s)
            if not stores:
                pending = frozenset(p for p in pending if p[1] not in _registers(operands[0]))
            if asm:
                counter = "vmcnt" if re.match(r"global_load_dword", op) else "lgkmcnt" if op.startswith("ds_read") else None
                if counter:
                    pending = pending | {(counter, r) for r in _registers(operands[0])}
        else:
            reach(after.get(label), pending)
    return found


def overwritten_reads(blocks):
    """Writes into a register that an inline-assembly LDS read is still to fill: a read whose value nobody uses
    looks done to the compiler as soon as it is issued, and its registers free."""
    order = list(blocks)
    after = dict(zip(order, order[1:]))
    seen, work, found = set(), [("", ())], []

    def reach(label, pending):
        if label is not None and (label, pending) not in seen:
            seen.add((label, pending))
            work.append((label, pending))

    while work:
        label, pending = work.pop()                  # registers of the LDS requests under way, oldest first
        for s, op, operands, asm in blocks[label]:
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", s)
                if m:
                    pending = pending[max(0, len(pending) - int(m.group(1))):]
                continue
            if op == "s_branch":
                reach(operands[0], pending)
                break
            if op.startswith("s_cbranch"):
                reach(operands[0], pending)
            if op == "s_endpgm":
                break
            read = asm and op.startswith("ds_read")
            if not read and "store" not in op and not op.startswith(("ds_write", "s_")):
                if any(r in p for r in _registers(operands[0]) for p in pending):
                    found.append(s)
            if op.startswith("ds_"):
                pending = (pending + (tuple(_registers(operands[0])) if read else (),))[-16:]
        else:
            reach(after.get(label), pending)
    return found


def masked_waits(blocks):
    """Waits for a part of the requests under way behind a branch on the exec mask: the lanes' own values decide."""
    text = [i for instructions in blocks.values() for i in instructions]
    return [s for (_, before, _, _), (s, op, _, _) in zip(text, text[1:])
            if before in ("s_cbranch_execz", "s_cbranch_execnz") and op == "s_waitcnt" and re.search(r"vmcnt\([1-9]", s)]


def unsettled_products(blocks):
    """Matrix products by inline assembly, for which the compiler counts no wait states: an accumulator read by anything but a
    product less than SETTLE instructions behind one, a product whose operand vector arithmetic wrote less than two before."""
    order = list(blocks)
    after = dict(zip(order, order[1:]))
    seen, work, found = set(), [("", SETTLE, ())], []

    def reach(label, since, fresh):
        if label is not None and (label, since, fresh) not in seen:
            seen.add((label, since, fresh))
            work.append((label, since, fresh))

    while work:
        label, since, fresh = work.pop()             # instructions since the last product; registers written by the last two
        for s, op, operands, asm in blocks[label]:
            if op == "s_branch":
                reach(operands[0], since, fresh)
                break
            if op.startswith("s_cbranch"):
                reach(operands[0], since, fresh)
            if op == "s_endpgm":
                break
            touched = [_registers(t) for t in operands]
            if op.startswith("v_mfma"):
                if asm and any(r in f for t in touched[1:] for r in t for f in fresh):
                    found.append(s)
                since, wrote = 0, ()
            else:
                if since < SETTLE and any(r[0] == "a" for t in touched for r in t):
                    found.append(s)
                wrote = tuple(touched[0]) if op.startswith("v_") and touched else ()
            waits = int(operands[0]) + 1 if op == "s_nop" else 1
            since = min(SETTLE, since + (waits if not op.startswith("v_mfma") else 0))
            fresh = ((wrote,) + fresh)[:2] if waits == 1 else ()
        else:
            reach(after.get(label), since, fresh)
    return found


def mixed_destinations(blocks):
    """Requests into LDS by inline assembly whose m0 something else has written since: (m0 set in an earlier statement)"""
    found = []
    for instructions in blocks.values():
        ours = False
        for s, op, operands, asm in instructions:
            if operands[0] == "m0" and op.startswith("s_"):
                ours = asm
            if asm and op.startswith("global_load_lds") and not ours:
                found.append(s)
    return found


SETTLE = 19


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    out = tmp_path_factory.mktemp("listings")
    procs = {}
    for f in FILES:
        cmd = [build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", os.path.join(build.CSRC, f + ".hip"), "-o", str(out / f)]
        procs[f] = subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    assert all(p.wait() == 0 for p in procs.values())
    return {f: (out / f).read_text() for f in FILES}


@pytest.mark.parametrize("f", FILES)
def test_no_move_of_a_load_before_a_wait(listings, f):
    seen = 0
    for name, blocks in _functions(listings[f]):
        seen += 1
        assert not early_moves(blocks), name
    assert seen > 0


# A value kept in memory between the loop and the end of the some-rows kernel is a trip for every wave.
def test_some_rows_keep_their_registers(listings):
    spills = re.findall(r"\.vgpr_spill_count: +(\d+)", listings["gemm_mid"])
    assert len(spills) == 4 and all(n == "0" for n in spills)


# The large-batch kernel's accumulators take half of the registers, and its products are inline assembly.
def test_large_batches_keep_their_accumulators(listings):
    spills = re.findall(r"\.vgpr_spill_count: +(\d+)", listings["gemm_wide"])
    assert len(spills) == 20 and all(n == "0" for n in spills)
    kernels = [(name, blocks) for name, blocks in _functions(listings["gemm_wide"]) if "gemm_wide_kernel" in name]
    assert len(kernels) == 18
    for name, blocks in kernels:
        assert not unsettled_products(blocks), name
        assert not mixed_destinations(blocks), name


# The reductions of both gradients share a launch; the arguments of each storage form stay its own.
def test_reductions_keep_their_scalars(listings):
    spills = dict(re.findall(r"\.name: +(_ZN7marlaas18reduce_bf16_kernelILi\d+E\w+)\n(?:.*\n)*?.*\.sgpr_spill_count: +(\d+)", listings["lora_small"]))
    assert len(spills) == 4
    for name, n in spills.items():
        assert "ILi8E" in name or n == "0", name


@pytest.mark.parametrize("f", ["gemm_mid", "gemm_decode"])
def test_no_write_over_a_pending_lds_read(listings, f):
    for name, blocks in _functions(listings[f]):
        assert not overwritten_reads(blocks), name


# The rank of a workgroup's adapter is one value for all its lanes: how many requests its ring waits for is no
# matter of masks.
def test_ring_waits_are_uniform(listings):
    rings = [(name, blocks) for name, blocks in _functions(listings["lora_small"]) if "shrink_ring_kernel" in name]
    assert len(rings) == 16
    for name, blocks in rings:
        assert not masked_waits(blocks), name


def test_overwritten_read_is_seen():
    text = """_Zk:
\t;;#ASMSTART
\tds_read_b128 v[4:7], v0
\t;;#ASMEND
\t;;#ASMSTART
\tds_read_b128 v[8:11], v0
\t;;#ASMEND
%s
\tv_add_u32_e32 v6, v1, v2
.LBB0_1:
\ts_endpgm
.Lfunc_end0:
"""
    for wait, seen in {"": 1, "\ts_waitcnt lgkmcnt(1)": 0, "\ts_waitcnt lgkmcnt(2)": 1, "\ts_waitcnt vmcnt(0)": 1}.items():
        (_, blocks), = _functions(text % wait)
        assert len(overwritten_reads(blocks)) == seen, wait


def test_early_move_is_seen():
    text = """_Zk:
\t;;#ASMSTART
\tglobal_load_dwordx4 v[4:7], v0, s[2:3]
\t;;#ASMEND
%s
\tv_mov_b64_e32 v[8:9], v[6:7]
.LBB0_1:
\ts_endpgm
.Lfunc_end0:
"""
    waits = {"": 1, "\ts_waitcnt vmcnt(2)": 0, "\ts_waitcnt lgkmcnt(0)": 1, "\ts_cbranch_vccz .LBB0_1": 1}
    for wait, moves in waits.items():
        (_, blocks), = _functions(text % wait)
        assert len(early_moves(blocks)) == moves, wait


def test_unsettled_product_is_seen():
    text = """_Zk:
%s
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]
\t;;#ASMEND
%s
\tv_accvgpr_read_b32 v1, a2
.LBB0_1:
\ts_endpgm
.Lfunc_end0:
"""
    for before, behind, n in (("", "", 1), ("", "\ts_nop 15", 1), ("", "\ts_nop 15\n\ts_nop 15", 0), ("\tv_mov_b32_e32 v5, v1", "\ts_nop 15\n\ts_nop 15", 1),
                              ("\tv_mov_b32_e32 v5, v1\n\ts_nop 1", "\ts_nop 15\n\ts_nop 15", 0)):
        (_, blocks), = _functions(text % (before, behind))
        assert len(unsettled_products(blocks)) == n, (before, behind)
