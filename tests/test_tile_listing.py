"""What the compiler does not check for the tile bodies, whose accumulators are accumulation registers named by number and
whose score MFMAs are assembly: read from the kernels' assembly listing (hipcc cross-compiles; no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2402_01869_amd import build

REG = re.compile(r"\b([va])\[(\w+):(\w+)\]|\b([va])\[(\w+)\]|\b([va])(\d+)\b")

# Wait states from an MFMA to another access of its result, by its passes of four cycles, as the compiler keeps them on this
# target; and from a vector instruction to an MFMA that reads what it wrote.
MFMA_WAIT = {"4x4x4": 5, "16x16x32": 8, "16x16x16": 8, "32x32x16": 12, "32x32x8": 20}
VALU_WAIT = 2


def _regs(text):
    out = []
    for m in REG.finditer(text):
        if m.group(1):
            out += [(m.group(1), r) for r in range(int(m.group(2), 0), int(m.group(3), 0) + 1)]
        else:
            out.append((m.group(4) or m.group(6), int(m.group(5) or m.group(7), 0)))
    return out


class Inst:
    """One instruction: what it reads and writes, how many wait states it stands for, where it may go on."""

    def __init__(self, code, asm):
        self.code, self.asm = code, asm
        self.op, _, rest = code.partition(" ")
        ops = rest.split(",")
        self.waits = int(rest, 0) + 1 if self.op == "s_nop" else 1
        self.target = rest.strip() if self.op.startswith(("s_branch", "s_cbranch")) else None
        self.falls = self.op not in ("s_branch", "s_endpgm")
        self.mfma = next((n for k, n in MFMA_WAIT.items() if "_" + k + "_" in self.op), 20) if "v_mfma" in self.op else 0
        self.valu = self.op.startswith("v_") and not self.mfma
        if self.op.startswith("s_"):
            self.dst, self.src = [], []
        elif self.op.startswith(("ds_write", "global_store", "scratch_store", "buffer_store", "flat_store")) or "_load_lds_" in self.op:
            self.dst, self.src = [], _regs(rest)
        elif "_swap_b32" in self.op:
            self.dst = self.src = _regs(rest)
        else:
            self.dst, self.src = _regs(ops[0]), _regs(",".join(ops[1:]))
        if self.mfma:
            self.ab, self.c = _regs(",".join(ops[1:3])), _regs(ops[3])


def parse(text):
    """Instructions and label positions of one kernel."""
    insts, labels, in_asm = [], {}, False
    for line in text.split("\n"):
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
        code = line.split(";")[0].strip()
        if code.endswith(":"):
            labels[code[:-1]] = len(insts)
        elif code and not code.startswith("."):
            insts.append(Inst(code, in_asm))
    return insts, labels


def check(insts, labels):
    """Follows every branch.  The state in front of an instruction: for each register that an MFMA (a vector instruction) has
    written, the wait states since, the fewest over all ways there; older writes are dropped.  Returns what breaks the rules."""
    keep = max(MFMA_WAIT.values())
    seen, work, bad = [None] * len(insts), [(0, {})], {}
    while work:
        at, state = work.pop()
        while at < len(insts):
            old = seen[at]
            if old is not None:
                merged = dict(old)
                for k, v in state.items():
                    if k not in merged or v < merged[k]:
                        merged[k] = v
                if merged == old:
                    break
                state = merged
            seen[at] = dict(state)
            i = insts[at]
            # keys: ("mfma", register, its result's registers, wait states it asks for) or ("valu", register)
            touched = set(i.src) | set(i.dst)
            for k, age in state.items():
                if k[1] not in touched:
                    continue
                if k[0] == "valu":
                    if i.mfma and k[1] in i.src and age < VALU_WAIT:
                        bad[at] = "%s: vector write %d before" % (i.code, age)
                elif i.mfma and k[1] not in i.ab and tuple(i.c if k[1] in i.c else i.dst) == k[2]:   # a sum goes on
                    if k[3] == MFMA_WAIT["4x4x4"] and i.c and age < 2:
                        bad[at] = "%s: sum %d after its last" % (i.code, age)
                elif age < k[3]:
                    bad[at] = "%s: MFMA result %d before, %d asked" % (i.code, age, k[3])
            state = {k: v + i.waits for k, v in state.items() if k[1] not in i.dst and v + i.waits < keep}
            for r in i.dst:
                if i.mfma:
                    state[("mfma", r, tuple(i.dst), i.mfma)] = 0
                elif i.valu:
                    state[("valu", r)] = 0
            if i.target is not None and i.falls:
                work.append((labels[i.target], dict(state)))
            if not i.falls:
                if i.target is None:
                    break
                at = labels[i.target]
            else:
                at += 1
    return [bad[k] for k in sorted(bad)]


def overwritten(insts, labels, own):
    """Instructions of the compiler's own that write one of the accumulation registers a0 .. a(own - 1) while the assembly blocks
    still want what is in it."""
    live = [frozenset()] * (len(insts) + 1)      # in front of each instruction
    after = lambda k, i: (live[k + 1] if i.falls else frozenset()) | (live[labels[i.target]] if i.target is not None else frozenset())
    mine = lambda regs: {n for t, n in regs if t == "a" and n < own}
    changed = True
    while changed:
        changed = False
        for k in range(len(insts) - 1, -1, -1):
            i = insts[k]
            now = after(k, i)
            if i.asm:
                now = (now - mine(i.dst)) | mine(i.src)
            if now != live[k]:
                live[k], changed = frozenset(now), True
    return [i.code for k, i in enumerate(insts) if not i.asm and mine(i.dst) & after(k, i)]


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not shutil.which("hipcc"):
        pytest.skip("hipcc not on PATH")
    out = str(tmp_path_factory.mktemp("tile") / "tile.s")
    r = subprocess.run(["hipcc"] + [f for f in build.FLAGS if f != "-shared"] + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "attn_tile.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("kernel,D,own", [(k, D, own) for D, own in ((64, 56), (128, 104), (256, 104))
                                          for k in ("tile_persist_kernelILi{}ELb0E", "tile_persist_kernelILi{}ELb1E")]
                         + [("tile_attn_kernelILi{}E", 256, 104)])      # the builds that a plan can launch
def test_accumulation_registers_and_wait_states_of_the_tile_body(listing, kernel, D, own):
    start = re.search(r"^\S*%s\S*:" % kernel.format(D), listing, re.M).start()
    text = listing[start:listing.index(".section", start)]
    # two waves of the tile kernel beside a 96-register row or group workgroup: 2 x 208 + 96 = 512 registers a lane
    meta = listing[listing.index(".amdhsa_kernel", start):]
    total = int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", meta).group(1))
    assert total <= (208 if "persist" in kernel else 256), total
    insts, labels = parse(text)
    mine = [i for i in insts if i.asm and re.search(r"\ba\[", i.code)]
    assert sum("mfma" in i.code for i in mine) >= 60      # the four fast stages and the serial step
    assert overwritten(insts, labels, own) == []
    assert sum(i.target is not None for i in insts) > 20  # branches, all of them to labels of the kernel
    assert check(insts, labels) == []


def test_the_check_follows_branches():
    """A result read too early only on the way back to the head of a loop, or only where a branch skips what stands between."""
    loop = """
.LBB0_1:
    v_add_f32_e32 v40, v2, v2
    s_nop 11
    v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]
    s_nop %d
    s_cbranch_scc1 .LBB0_1
    s_endpgm"""
    assert check(*parse(loop % 10)) == [] and len(check(*parse(loop % 9))) == 1
    skip = """
    v_mfma_f32_16x16x32_bf16 a[0:3], v[16:19], v[20:23], a[0:3]
    s_cbranch_scc1 .LBB0_2
    s_nop 15
.LBB0_2:
    %s
    v_accvgpr_read_b32 v0, a1
    s_endpgm"""
    assert check(*parse(skip % "s_nop 6")) == [] and len(check(*parse(skip % "s_nop 5"))) == 1
    feed = """
    v_accvgpr_write_b32 a7, v0
    s_nop %d
    v_mfma_f32_16x16x32_bf16 a[0:3], a[4:7], v[20:23], a[0:3]
    v_mfma_f32_16x16x32_bf16 a[0:3], a[4:7], v[20:23], a[0:3]
    s_endpgm"""
    assert check(*parse(feed % 1)) == [] and len(check(*parse(feed % 0))) == 1
    held = """
    ;;#ASMSTART
    v_accvgpr_write_b32 a[3], v0
    ;;#ASMEND
.LBB0_3:
    s_cbranch_scc0 .LBB0_4
    v_accvgpr_write_b32 a%d, v0
    s_branch .LBB0_3
.LBB0_4:
    ;;#ASMSTART
    v_accvgpr_read_b32 v0, a[3]
    ;;#ASMEND
    v_accvgpr_write_b32 a3, v0
    s_endpgm"""
    assert overwritten(*parse(held % 4), 4) == [] and len(overwritten(*parse(held % 3), 4)) == 1
