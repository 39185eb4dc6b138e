"""What the compiler does not check for the tile bodies, whose accumulators are accumulation registers named by number and
whose score MFMAs are assembly: read from the kernels' assembly listing (hipcc cross-compiles; no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
REG = re.compile(r"\b([va])\[(\w+):(\w+)\]|\b([va])\[(\w+)\]|\b([va])(\d+)\b")


def _regs(text):
    out = []
    for m in REG.finditer(text):
        if m.group(1):
            out += [(m.group(1), r) for r in range(int(m.group(2), 0), int(m.group(3), 0) + 1)]
        else:
            out.append((m.group(4) or m.group(6), int(m.group(5) or m.group(7), 0)))
    return out


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not shutil.which("hipcc"):
        pytest.skip("hipcc not on PATH")
    src = os.path.join(ROOT, "paper_2402_01869_amd", "csrc", "attn_tile.hip")
    out = str(tmp_path_factory.mktemp("tile") / "tile.s")
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "--cuda-device-only", "-S", src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("kernel", ["tile_persist_kernelILi{}ELb0E", "tile_persist_kernelILi{}ELb1E", "tile_attn_kernelILi{}E"])
@pytest.mark.parametrize("D,own", [(64, 56), (128, 104), (256, 104)])
def test_accumulation_registers_and_wait_states_of_the_tile_body(listing, kernel, D, own):
    start = re.search(r"^\S*%s\S*:" % kernel.format(D), listing, re.M).start()
    text = listing[start:listing.index(".section", start)]
    # two waves of the tile kernel beside a 96-register row or group workgroup: 2 x 208 + 96 = 512 registers a lane
    meta = listing[listing.index(".amdhsa_kernel", start):]
    total = int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", meta).group(1))
    assert total <= (208 if "persist" in kernel else 256), total
    lines, in_asm = [], False      # (code, from an asm block)
    for line in text.split("\n"):
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
        code = line.split(";")[0].strip()
        if code and not code.startswith(".") and not code.endswith(":"):
            lines.append((code, in_asm))
    mine = [i for i, (c, a) in enumerate(lines) if a and re.search(r"\ba\[", c)]
    assert sum("mfma" in lines[i][0] for i in mine) >= 60      # the four fast stages and the serial step
    # From the first to the last use of the body's accumulation registers nothing else touches them; what reads or
    # overwrites an MFMA's result waits for 8 passes + 3 wait states, and an MFMA 2 for an operand a vector instruction wrote.
    at, by_mfma, by_valu = 0, {}, {}
    for code, asm in lines[mine[0]:mine[-1] + 1]:
        op, _, rest = code.partition(" ")
        if not asm:
            assert not any(r[0] == "a" and r[1] < own for r in _regs(rest)), code
        at += int(rest, 0) + 1 if op == "s_nop" else 1
        if op.startswith("s_"):
            continue
        ops = rest.split(",")
        store = op.startswith(("ds_write", "global_store", "scratch_store"))
        dst = [] if store else _regs(ops[0])
        src = _regs(rest if store else ",".join(ops[1:]))
        if "mfma" in op:
            for r in _regs(",".join(ops[1:3])):
                assert at - by_valu.get(r, -99) - 1 >= 2 and at - by_mfma.get(r, -99) - 1 >= 11, code
            for r in dst:
                by_mfma[r] = at
                by_valu.pop(r, None)
            continue
        for r in src + dst:
            assert at - by_mfma.get(r, -99) - 1 >= 11, code
        for r in dst:
            by_mfma.pop(r, None)
            if op.startswith("v_"):
                by_valu[r] = at
            else:
                by_valu.pop(r, None)
