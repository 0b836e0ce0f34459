"""Streaming kernels (small M) where their loop over the K groups can go wrong: fewer groups than
wavefronts, odd numbers of groups per wavefront, more groups than the scales of one fill of LDS cover
(16 per wavefront, 8 from 64 tokens on), numbers of tile blocks that do not divide by the eight XCDs."""
import numpy as np
import pytest

from oracle import device_layout as lay
from oracle import qspec_oracle as orc
from paper_2410_11305_amd import synth

pytestmark = pytest.mark.gpu
TOL = 2e-3           # max |y - y_ref| / max |y_ref| against the float64 oracle


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2410_11305_amd import binding as B
    assert torch.cuda.is_available()
    B.lib()
    return torch, B


@pytest.mark.parametrize("G", [1, 7, 9, 33, 131, 258])
@pytest.mark.parametrize("tm,nt", [(1, 1), (1, 3), (2, 2), (2, 6), (4, 4), (8, 2)])
def test_draft_mode_bit_exact_over_group_counts(env, plan, tm, nt, G):
    """One live group per token row and power-of-two scales: y = fp16(P sa sw) in any summation order."""
    torch, B = env
    M, N = 16 * tm - 3, 16 * (9 * nt + 1)                # ten tile blocks, the last one ragged
    plan("QSPEC_STREAM_MAX_W4A4", "128")
    plan("QSPEC_STREAM_W4A4", f"{nt},1")
    rng = np.random.default_rng(G * 100 + tm * 10 + nt)
    qw = rng.integers(-8, 8, size=(N, 128 * G), dtype=np.int8)
    qa = np.zeros((M, 128 * G), np.int8)
    for m in range(M):
        g = G - 1 if m == 0 else (m * 37) % G            # the last group is always among them
        qa[m, 128 * g:128 * g + 128] = rng.integers(-7, 8, size=128, dtype=np.int8)
    sa = (2.0 ** rng.integers(-3, 3, size=(M, G))).astype(np.float32)
    sw = (2.0 ** rng.integers(-9, -5, size=(N, G))).astype(np.float16)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    assert B.describe_kernel(True, M, N, 128 * G) == f"gemm_stream_kernel<true, {tm}, {nt}>"
    y = B.gemm_w4a4(B.pack_weights(to(qw), to(sw)), to(lay.act_bytes(qa)), to(sa), N).cpu().numpy()
    ref = orc.gemm_w4a4(qa, sa, qw, sw)
    assert np.array_equal(y.view(np.uint16), ref.view(np.uint16))


@pytest.mark.parametrize("G", [1, 7, 9, 33, 131, 258])
@pytest.mark.parametrize("M,forced", [(13, "1,1"), (16, "3,1"), (29, "1,1"), (32, "6,1"), (29, "2,1,2")])
def test_verify_mode_over_group_counts(env, plan, M, forced, G):
    """Against the oracle; and an infinite activation in the last group reaches its own token row only
    (a group that does not exist is skipped, not multiplied by zero weights)."""
    torch, B = env
    nt = int(forced.split(",")[0])
    N, K = 16 * (9 * nt + 1), 128 * G
    plan("QSPEC_STREAM_W4A16", forced)
    codes, scales, x = synth.generic_case(G * 100 + M, M, N, K)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    blob = B.pack_weights(to(codes), to(scales))
    y = B.gemm_w4a16(blob, to(x), N).cpu().numpy().astype(np.float64)
    ref = orc.gemm_w4a16(x, codes, scales).astype(np.float64)
    assert np.max(np.abs(y - ref)) / np.max(np.abs(ref)) <= TOL
    x2 = x.copy()
    x2[M // 2, K - 1] = np.inf
    codes[:, K - 1] = 3                                  # inf times a non-zero code
    blob = B.pack_weights(to(codes), to(scales))
    y2 = B.gemm_w4a16(blob, to(x2), N).cpu().numpy()
    assert np.isinf(y2[M // 2]).all() and np.isfinite(np.delete(y2, M // 2, axis=0)).all()
