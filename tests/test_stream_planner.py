"""The choice between the streaming and tiled kernels, and of their plans, against timed plans
(profiles/stream_plan_times.txt): draft mode at 17 to 600 tokens, verify mode at 17 to 32.  Needs no GPU: the
choice is a pure function of the sizes.  Bounds: the timings repeat within 3 %; the cost tables leave 1 % on
average and 15 % at most on problems they were not fitted to."""
import math
import os
import re

import pytest

from paper_2410_11305_amd import binding as B

TABLE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles", "stream_plan_times.txt")
BLOCK4 = [(128, 128, "1, 4, 4"), (128, 64, "1, 2, 4"), (64, 64, "1, 2, 2"), (256, 128, "1, 4, 8")]


def _chosen(draft, M, N, K):
    name = B.describe_kernel(draft, M, N, K)
    m = re.match(r"gemm_stream_kernel<\w+, (\d+), (\d+)>", name)
    if m:
        return f"stream{m.group(1)}.{m.group(2)}"
    need = B.workspace_bytes(M, N, K)
    for shape, (bn, bm, args) in enumerate(BLOCK4):
        if f"<{args}, 1," in name:
            return f"tile{shape}.{max(1, (need - 16384) // (-(-N // bn) * -(-M // bm) * bn * bm * 4))}"


def test_chosen_plans_are_near_the_best(plan):
    plan("QSPEC_TILE_W4A16", "0,1")                       # (the verify mode's own workspace need is kept at none)
    logs, slower, n = [], [], 0
    for line in open(TABLE):
        if line.startswith("#"):
            continue
        size, before, plans = line.split("|")
        mode, M, N, K = size.split()
        M, N, K, before = int(M), int(N), int(K), float(before)
        times = {k: float(v) for k, v in (p.split(":") for p in plans.split())}
        t = times.get(_chosen(mode == "draft", M, N, K), math.inf)    # a plan more than 20 % off the best is not listed
        logs.append(math.log(t / min(times.values())))
        if t > 1.12 * before:
            slower.append((size, t, before))
        n += 1
    assert n == 320 and not slower, slower[:5]
    assert max(logs) <= math.log(1.2) and sum(logs) / n <= math.log(1.02)


@pytest.mark.parametrize("M", [17, 33, 48, 64, 65, 128, 129, 256, 512, 600, 2050, 20001])
@pytest.mark.parametrize("N,K", [(16, 128), (16, 130944), (1024, 1024), (4096, 2048), (57344, 8192), (128256, 4096)])
def test_draft_partial_sums_fit_the_built_in_scratch(plan, M, N, K):
    """qspec_gemm_w4a16_noalloc holds its scratch against the larger of the two modes' needs."""
    plan("QSPEC_TILE_W4A16", "0,1")
    if M * K * 2 < 2 ** 31:
        assert B.workspace_bytes(M, N, K) <= (32 << 20) + 16384
