"""Widened draft kernel: what the wait in front of the prologue's barrier lets through, from the order of issue that the source
states.  Group 0 reads the first operands of group 1 under its last token tile, before its own closing wait, and those
rows come in by other wavefronts' transfers, so the prologue's barrier has to publish both stages.  Loads complete in order and a wait
for n of them lets the n youngest be on their way.  Needs no GPU."""
import os
import re

import pytest

from paper_2410_11305_amd import build

SOURCE = os.path.join(build.HERE, "csrc", "gemm_tile4.hpp")


def _body(text, start):
    """The braces that open behind `start`."""
    begin = text.index("{", text.index(start)) + 1
    depth, end = 1, begin
    while depth:
        depth += {"{": 1, "}": -1}.get(text[end], 0)
        end += 1
    return text[begin:end - 1]


def in_flight(text, PN, UD):
    """Transfers that may be under way behind the prologue's wait, as the groups they belong to."""
    NW = 3
    prologue = re.sub(r"//.*", "", _body(text[text.index("load_sa3(0);"):], "if constexpr (WIDE)"))
    pending = ["scales"]                                   # load_sa3(0)
    for name, args in re.findall(r"(dma_x|load_w|waitcnt_vm)\(((?:[^()]|\([^()]*\))*)\)", prologue):
        if name == "dma_x":
            pending += [int(args.split(",")[0])] * UD
        elif name == "load_w":
            pending += ["weights"] * (3 * PN)
        else:
            n = eval(args, {}, dict(PN=PN, NW=NW, UD=UD))
            pending = pending[max(0, len(pending) - n):]
    return {p for p in pending if isinstance(p, int)}


@pytest.mark.parametrize("BM,waves", [(128, 4), (64, 4), (64, 2), (128, 8)])       # the workgroup shapes
def test_the_first_barrier_publishes_what_group_0_reads(BM, waves):
    text = open(SOURCE).read()
    group = _body(text, "auto group_body")
    assert 0 < group.index("read_operand(xl_next, 0, st)") < group.rindex("__syncthreads()")
    assert in_flight(text, 1, BM // 8 // waves) == set()


def test_the_check_sees_a_wait_that_is_too_lax():
    text = open(SOURCE).read()
    for lax, expected in (("3 * PN * NW + UD", {1}), ("3 * PN * NW + 2 * UD", {0, 1})):
        planted = re.sub(r"(s_waitcnt\(waitcnt_vm\()[^;]*(\)\);)", lambda m: m.group(1) + lax + m.group(2), text, count=1)
        assert in_flight(planted, 1, 2) == expected
