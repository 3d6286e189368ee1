"""Kernels that load straight into LDS wait for it with hand-counted s_waitcnt.  Here the generated assembly is walked with the
hardware's rule (loads return in the order they were issued).

The INT2 producer of the fused kernel: every read-back of a pass must find that pass's load among the returned ones: the
single-round kernels (seven passes, all in flight), and the others over three rounds with requests and the last one without.

The rings of the wide kernels: the barrier that makes a slot everybody's must find the slot's loads of every wave returned, and no
wait inside the loop may empty the ring."""
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


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs the compiler")
def test_the_same_with_consumers_one_entry_ahead(tmp_path):
    out = tmp_path / "fused_ahead_int2.s"
    subprocess.run([HIPCC, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, "fused_ahead_int2.hip"), "-o", str(out)], check=True)
    seen = 0
    for m in re.finditer(r"^(_ZN4floe16fused_ffn_kernelILi2E\w*Li448ELi14EE\w+):(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S):
        body = m.group(2).split("\n")
        first = next(i for i, l in enumerate(body) if "global_load_lds_dwordx4" in l)
        begin, end = steady_loop(body, first, 14)
        head, tail = body[first:begin], body[end + 1:]
        if late_read_backs(head)[1] > 1:  # the last round stands in front of the loop: from the label behind the first read back on
            read = next(i for i, l in enumerate(head) if l.strip().startswith("ds_read_b128") and "ASMSTART" in head[i - 1])
            cut = next(i for i, l in enumerate(head) if i > read and l.startswith(".LBB"))
            head, tail = head[:cut], head[cut:]
        bad, reads = late_read_backs(head + STEADY_ROUNDS * body[begin:end + 1] + tail)
        assert reads == 14 * (1 + STEADY_ROUNDS), (m.group(1), reads)
        assert not bad, (m.group(1), "read back too early: passes", bad)
        seen += 1
    assert seen == 6


def ring_loops(body):
    """(first, last line, barriers, direct loads) of the innermost loops that meet once per slot of a ring of three or four."""
    labels = {l.split(":")[0]: i for i, l in enumerate(body) if re.match(r"\.LBB\w+:", l)}
    loops = []
    for i, l in enumerate(body):
        m = re.search(r"s_c?branch\w* (\.LBB\w+)", l)
        if m and labels[m.group(1)] <= i:
            part = body[labels[m.group(1)]:i + 1]
            barriers, loads = sum("s_barrier" in x for x in part), sum("global_load_lds" in x for x in part)
            if barriers in (3, 4) and loads:
                loops.append((labels[m.group(1)], i, barriers, loads))
    return [a for a in loops if not any(b[0] >= a[0] and b[1] <= a[1] and b != a for b in loops)]


def check_ring(body, begin, end, barriers, loads):
    """Slots are loaded in turn, `per` requests of a wave each, and barrier k of the loop hands out slot k."""
    assert loads % barriers == 0
    per = loads // barriers
    ahead = [i for i, l in enumerate(body[:begin]) if "global_load_lds" in l]
    first = ahead[-(barriers - 1) * per]  # all slots but one are requested in front of the loop
    # (a loop may be entered past its first lines, which then belong to the end of a round)
    jump = next((re.match(r"\s*s_branch (\.LBB\w+)", l) for l in reversed(body[:begin]) if l.split(";")[0].strip()), None)
    entry = next((i for i in range(begin, end + 1) if jump and body[i].startswith(jump.group(1) + ":")), begin)
    walk = body[first:begin] + body[entry:end + 1] + (STEADY_ROUNDS - 1) * body[begin:end + 1]
    issued, landed, requests, met, emptied = 0, 0, [], 0, 0
    in_loop = begin - first
    for i, raw in enumerate(walk):
        s = raw.strip()
        if re.match(r"(global|flat|buffer|scratch)_load", s):
            issued += 1
            if s.startswith("global_load_lds"):
                requests.append(issued)
        elif s.startswith("s_waitcnt") and "vmcnt(" in s:
            landed = max(landed, issued - int(re.search(r"vmcnt\((\d+)\)", s).group(1)))
            emptied += i >= in_loop and landed >= requests[-1]
        elif s.startswith("s_barrier") and i >= in_loop:
            assert requests[(met + 1) * per - 1] <= landed, ("slot handed out too early", met)
            met += 1
    assert met == STEADY_ROUNDS * barriers
    return emptied


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs the compiler")
@pytest.mark.parametrize("source,kernel,instances", [("up_wide.hip", "up_wide", 21), ("wide_batch.hip", "gate_wide", 6)])
def test_ring_slots_have_landed_when_they_are_handed_out(tmp_path, source, kernel, instances):
    out = tmp_path / "ring.s"
    subprocess.run([HIPCC, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, source), "-o", str(out)], check=True)
    seen = 0
    for m in re.finditer(rf"^(_ZN4floe\w*{kernel}_kernel\w+):(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S):
        body = m.group(2).split("\n")
        loops = ring_loops(body)
        assert len(loops) >= 2, m.group(1)  # waves at work, and those that only help to load
        for loop in loops:
            assert check_ring(body, *loop) == 0, (m.group(1), "a wait inside the loop leaves nothing under way")
        seen += 1
    assert seen == instances
