"""The bf16 products' fragment reads from LDS are written out in assembly, with the waits for them: the compiler takes a
read's registers as written at once.  A build is sound if nothing touches them between a read and the wait that covers
it, which the listing of the build shows; a result shows a breach now and then at most."""
import collections
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from __graft_entry__ import HIPCC_FLAGS  # noqa: E402

REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def blocks_of(lines):
    """[(label, [instruction], [labels that follow])] of a kernel's listing."""
    blocks, label, body = [], "entry", []
    for line in lines:
        line = line.split(";")[0].strip()
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            blocks.append((label, body))
            label, body = m.group(1), []
        elif line and not line.startswith(".") and not line.endswith(":"):
            body.append(line)
            if line.startswith("s_cbranch"):  # (what follows is a block without a label)
                blocks.append((label, body))
                label, body = "%s+%d" % (label, len(blocks)), []
    blocks.append((label, body))
    out = []
    for i, (label, body) in enumerate(blocks):
        last = body[-1] if body else ""
        to = re.findall(r"\.LBB\w+", last) if last.startswith(("s_cbranch", "s_branch")) else []
        if not last.startswith(("s_branch", "s_endpgm", "s_setpc")) and i + 1 < len(blocks):
            to.append(blocks[i + 1][0])
        out.append((label, body, to))
    return out


def breaches(lines):
    """(instructions that touch a register of an LDS read that no wait has covered yet, LDS reads seen) of one kernel.

    LDS answers in order: a wait for `lgkmcnt(n)` leaves at most the newest n operations open, those without a result counted
    too.  (Scalar loads share the counter: with some of them on their way the wait leaves fewer.)
    """
    blocks = {label: (body, to) for label, body, to in blocks_of(lines)}
    todo, seen, bad, reads = collections.deque([("entry", ())]), set(), [], 0
    while todo:
        state = todo.popleft()
        if state in seen:
            continue
        seen.add(state)
        assert len(seen) < 20000
        label, open_ = state[0], list(state[1])
        body, to = blocks[label]
        for ins in body:
            op = ins.split()[0]
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", ins)
                n = int(m.group(1)) if m else 0 if re.fullmatch(r"s_waitcnt 0", ins) else None
                if n is not None:
                    open_ = open_[max(len(open_) - n, 0):]
                continue
            touched = registers(ins) & set().union(*open_)
            if touched:
                bad.append((label, ins, sorted(touched)))
            if op.startswith("ds_"):
                reads += op.startswith("ds_read")
                open_.append(frozenset(registers(ins.split(None, 1)[1].split(",")[0])) if op.startswith("ds_read") else frozenset())
            open_ = open_[-63:]
        todo.extend((t, tuple(open_)) for t in to)
    return bad, reads


def kernels(text):
    return re.findall(r"^(_Z\w+):[^\n]*\n(.*?)^\.Lfunc_end", text, re.M | re.S)


LOOP = """
	ds_read_b128 v[0:3], v20
.LBB0_1:
	ds_read_b64_tr_b16 v[4:5], v21 offset:64
	%s
	s_waitcnt lgkmcnt(%d)
	v_mfma_f32_32x32x16_bf16 v[30:45], v[0:3], v[0:3], v[30:45]
	s_waitcnt lgkmcnt(0)
	v_mov_b32_e32 v6, v5
	ds_read_b128 v[0:3], v20
	s_cbranch_scc1 .LBB0_1
; %%bb.2:
	%s
	v_mov_b32_e32 v1, v9
"""


@pytest.mark.parametrize("between,count,behind,found", [
    ("v_mov_b32_e32 v7, v8", 1, "s_waitcnt vmcnt(0) lgkmcnt(0)", 0),
    ("v_mov_b32_e32 v7, v3", 1, "s_waitcnt lgkmcnt(0)", 1),   # a copy in front of the wait
    ("v_add_u32_e32 v4, s0, v7", 1, "s_waitcnt lgkmcnt(0)", 1),  # a value in a register that is still to be written
    ("s_nop 0", 2, "s_waitcnt lgkmcnt(0)", 1),                # a wait that leaves the read open
    ("s_nop 0", 1, "s_waitcnt vmcnt(0)", 1),                  # the last read is never waited for
    ("s_load_dword s4, s[2:3], 0x0", 1, "s_waitcnt lgkmcnt(0)", 0),
])
def test_the_check_finds_what_it_is_for(between, count, behind, found):
    bad, reads = breaches((LOOP % (between, count, behind)).splitlines())
    assert len({b[1] for b in bad}) == found and reads >= 3, bad


def test_no_fragment_is_touched_before_its_wait(tmp_path):
    out = str(tmp_path / "listing.s")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", "-o", out,
                           os.path.join(ROOT, "paper_2009_02701_amd", "csrc", "gemm_bf16_nt.hip")])
    with open(out) as f:
        found = {name: breaches(body.splitlines()) for name, body in kernels(f.read())}
    written_out = [n for n in found if "gemm_bf16_dlx" in n]
    assert len(written_out) >= 3 * 7 and all(found[n][1] > 0 for n in written_out), sorted(found)
    assert not {n: b[:3] for n, (b, _) in found.items() if b}


def test_updates_of_whole_columns_have_no_loads_of_single_words(tmp_path):
    """Every form of an 8-wave update has a kernel for widths of whole pieces of four: the early loads of the last one to three
    columns make the old values of all columns wait for each other."""
    out = str(tmp_path / "listing.s")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", "-o", out,
                           os.path.join(ROOT, "paper_2009_02701_amd", "csrc", "gemm_bf16_nt.hip")])
    forms = collections.defaultdict(list)
    with open(out) as f:
        for name, body in kernels(f.read()):
            m = re.search(r"gemm_bf16_dlx_(kernel|pair_kernel)ILb1E((?:L[ib]\d+E)+)E", name)
            if m:  # shape, gate blocks and (not of a pair) how the operands lie
                form = re.findall(r"L[ib]\d+E", m.group(2))[:8 if m.group(1) == "kernel" else 6]
                forms[m.group(1), tuple(form)].append(len(re.findall(r"\bglobal_load_dword v", body)))
    assert len(forms) == 3 * 3 + 2, sorted(forms)
    assert all(min(n) == 0 for n in forms.values()), dict(forms)
