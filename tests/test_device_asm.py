"""Wait states of the inline assembly, read off the assembly built here.

On gfx950 a vector instruction may read a scalar register two wait states
after a vector instruction wrote it at the earliest. The compiler inserts the
waits between its own instructions but does not look into inline assembly, so
a block that reads or writes scalar registers with vector instructions has to
keep the distance by itself: from its start, inside, and to its end (whatever
the compiler puts there, a spill of a mask among it)."""
import os
import re
import subprocess

import pytest

from paper_2606_02982_amd import build

WAIT = 2


def _scalars(operand):
    regs = {"vcc"} if "vcc" in operand else set()
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", operand):
        regs |= {"s%d" % r for r in range(int(a), int(b) + 1)}
    return regs | {"s" + r for r in re.findall(r"\bs(\d+)\b", operand)}


def _violations(block):
    """Of one block's instructions: reads closer than WAIT to their write."""
    bad, since, start = [], {}, 0      # wait states since each register's write, and the block's start
    for ins in block:
        op, _, rest = ins.partition(" ")
        args = rest.split(",")
        if op.startswith("v_"):
            n_out = 2 if "_co_" in op else 1
            for r in set().union(set(), *map(_scalars, args[n_out:])):
                if since.get(r, start) < WAIT:
                    bad.append("%s: %s %s" % (ins, r, "written" if r in since else "at the block's start"))
            written = set().union(*map(_scalars, args[:n_out]))
        else:
            written = set()
        step = int(rest, 0) + 1 if op == "s_nop" else 1
        start += step
        since = {r: w + step for r, w in since.items()}
        since.update({r: 0 for r in written})
    return bad + ["the block ends %d after the write of %s" % (w, r) for r, w in sorted(since.items()) if w < WAIT]


@pytest.mark.parametrize("src", ["norder.hip"])
def test_masks_of_inline_assembly_wait(src, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "device.s")
    subprocess.run([build.HIPCC] + build.HIP_FLAGS + ["--cuda-device-only", "-S", "-o", out,
                                                      os.path.join(build.CSRC, src)], check=True, timeout=300,
                   capture_output=True)
    with open(out) as f:
        text = f.read()
    blocks = [[x.strip().replace("\t", " ") for x in b.split("\n") if x.strip() and not x.strip().startswith(";")]
              for b in re.findall(r";;#ASMSTART\n(.*?);;#ASMEND", text, re.S)]
    blocks = [b for b in blocks if any(x.startswith("v_subb") for x in b)]
    assert len(blocks) > 50
    bad = [v for b in blocks for v in _violations(b)]
    assert not bad, "\n".join(bad[:8])
