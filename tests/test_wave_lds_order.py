"""LDS that the lanes of one wavefront pass values through, without a barrier: between a write and the read of what another lane
wrote, and between a read and the write that replaces it, the source names the order (wave_lds_order), or the workgroup
waits.  Needs no GPU."""
import os
import re

import pytest

from paper_2410_11305_amd import build

KINDS = [("order", r"wave_lds_order\(\)|__syncthreads\(\)"), ("write", r"\*reinterpret_cast<[^<>]*>\((?!p\.y)[^;=]*\) = [^;]*;|\bstage\(\);|\bput_scales\([^)]*\);"),
         ("read", r"= (?:unpack_i8\(|half_bits_to_float\()?\*reinterpret_cast<const ")]


def _function(file, start):
    text = re.sub(r"//.*", "", open(os.path.join(build.HERE, "csrc", file)).read())
    begin = text.index("{", text.index(start)) + 1
    depth, end = 1, begin
    while depth:
        depth += {"{": 1, "}": -1}.get(text[end], 0)
        end += 1
    return text[begin:end - 1]


def unordered(text, loops):
    """Neighbouring accesses of different kinds with no order between them, the text run through `loops` times."""
    text = text * loops
    events = sorted((m.start(), kind) for kind, pattern in KINDS for m in re.finditer(pattern, text))
    kinds = [kind for _, kind in events]
    assert "write" in kinds and "read" in kinds
    return [(a, b) for a, b in zip(kinds, kinds[1:]) if {a, b} == {"read", "write"}]


PLACES = [("tile_common.hpp", "tile_write_rows(", "for (int t"), ("tile_common.hpp", "tile_write_columns(", "for (int j"),
          ("gemm_stream.hpp", "auto step = ", None)]


@pytest.mark.parametrize("file,function,loop", PLACES)
def test_lanes_hand_over_in_a_stated_order(file, function, loop):
    body = _function(file, function)
    body = body[body.index(loop):] if loop else body
    assert unordered(body, 2) == []
    assert len(unordered(body.replace("wave_lds_order();", ""), 2)) >= 3          # (the check sees a missing one)


def test_streaming_kernel_between_its_loop_and_its_sums():
    text = _function("gemm_stream.hpp", "void stream_product(")
    chunks = text[text.index("put_scales(0);"):]
    sums = chunks.index("mine + o * 1024")
    assert re.search(r"break;\s*\}\s*load_scales\(c0 \+ CH\);\s*wave_lds_order\(\);\s*put_scales\(c0 \+ CH\);", chunks)
    assert chunks.rindex("wave_lds_order();", 0, sums) > chunks.index("step(s, c0, std::integral_constant<bool, false>{});")
