"""The INT2 producer of the fused kernel waits for its direct-to-LDS loads with hand-counted s_waitcnt.  Here the
generated assembly is walked with the hardware's rule (loads return in the order they were issued) and every read-back of a pass
must find that pass's load among the returned ones: the single-round kernels (seven passes, all in flight), and the others over
three rounds with requests and the last one without."""
import os
import re
import subprocess

import pytest

from paper_2505_05950_amd.build import CSRC, FLAGS, HIPCC  # the product's own compiler line

STEADY_ROUNDS = 3


def late_read_backs(lines):
    """Passes whose codes are read back before their load is known to have arrived (loads, stores: the fewest that can be
    outstanding, so a store - it depends on the channel or the workgroup - is left out)."""
    issued, landed, requests, reads, bad, in_asm = 0, 0, [], 0, [], False
    for raw in lines:
        s = raw.strip()
        if s.startswith(";;#ASMSTART") or s.startswith(";APP"):
            in_asm = True
        elif s.startswith(";;#ASMEND") or s.startswith(";NO_APP"):
            in_asm = False
        elif re.match(r"(global|flat|buffer|scratch)_load", s):
            issued += 1
            if s.startswith("global_load_lds"):
                requests.append(issued)
        elif s.startswith("s_waitcnt") and "vmcnt(" in s:
            landed = max(landed, issued - int(re.search(r"vmcnt\((\d+)\)", s).group(1)))
        elif in_asm and s.startswith("ds_read_b128"):
            if requests[reads] > landed:
                bad.append(reads)
            reads += 1
    return bad, reads


def steady_loop(body, first, depth):
    """(first, last line) of the loop over rounds that request: the tightest one behind the prologue's requests with `depth` of them."""
    labels = {l.split(":")[0]: i for i, l in enumerate(body) if re.match(r"\.LBB\w+:", l)}
    loads = [i for i, l in enumerate(body) if "global_load_lds_dwordx4" in l]
    loops = []
    for i, l in enumerate(body):
        m = re.search(r"s_c?branch\w* (\.LBB\w+)", l)
        if m and loads[depth - 1] < labels[m.group(1)] <= i:
            if sum(labels[m.group(1)] <= k <= i for k in loads) == depth:
                loops.append((labels[m.group(1)], i))
    return min(loops, key=lambda r: r[1] - r[0])


def check(asm):
    seen = 0
    for m in re.finditer(r"^(_ZN4floe16fused_ffn_kernelILi2E\w*Li(7|448)ELi(\d+)EE\w+):(.*?)^\.Lfunc_end", asm, re.M | re.S):
        body = m.group(4).split("\n")
        first = next(i for i, l in enumerate(body) if "global_load_lds_dwordx4" in l)
        depth, rounds = int(m.group(3)), 1
        walk = body[first:]
        if m.group(2) != "7":
            begin, end = steady_loop(body, first, depth)
            walk = body[first:begin] + STEADY_ROUNDS * body[begin:end + 1] + body[end + 1:]
            rounds += STEADY_ROUNDS
        bad, reads = late_read_backs(walk)
        assert reads == depth * rounds, (m.group(1), reads)
        assert not bad, (m.group(1), "read back too early: passes", bad)
        seen += 1
    return seen


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs the compiler")
def test_every_pass_has_landed_before_it_is_read_back(tmp_path):
    out = tmp_path / "fused_int2.s"
    subprocess.run([HIPCC, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, "fused_int2.hip"), "-o", str(out)], check=True)
    assert check(out.read_text()) == 36


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs the compiler")
def test_the_same_at_widths_between_the_powers_of_two(tmp_path):
    out = tmp_path / "fused_between_int2.s"
    subprocess.run([HIPCC, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, "fused_between_int2.hip"), "-o", str(out)], check=True)
    assert check(out.read_text()) == 36
