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


@pytest.mark.parametrize("M", [33, 48, 64, 65, 100, 128, 200, 300, 600, 2000])
@pytest.mark.parametrize("N,K", [(400, 1408), (1024, 1024), (4096, 4096), (22016, 4096)])
def test_generic_override_leaves_nothing_above_32_tokens_to_the_other_kernels(plan, M, N, K):
    plan("QSPEC_KERNEL", "generic")
    for draft in (True, False):
        assert re.match(r"gemm_w4a(4|16)_generic<", B.describe_kernel(draft, M, N, K))
    assert not B.w4a4_takes_wide(M, N, K) and B.workspace_bytes(M, N, K) == 0
    assert B.describe_kernel(True, 32, N, K).startswith("gemm_stream") and B.describe_kernel(False, 32, N, K).startswith("gemm_stream")


@pytest.mark.parametrize("bound", [32, 64, 100, 128])
@pytest.mark.parametrize("N,K", [(400, 1408), (1024, 1024), (4096, 4096), (22016, 4096), (57344, 8192)])
def test_stream_max_override_is_a_bound_from_both_sides(plan, bound, N, K):
    plan("QSPEC_STREAM_MAX_W4A4", str(bound))
    for M in (17, 30, bound - 1, bound):
        m = re.match(r"gemm_stream_kernel<true, (\d+), (\d+)>", B.describe_kernel(True, M, N, K))
        assert m and int(m.group(1)) > 0 and int(m.group(2)) > 0       # (0: a plan that the launch refuses)
    for M in (bound + 1, 300, 1500):
        assert B.describe_kernel(True, M, N, K).startswith("gemm_tile4w_kernel")
