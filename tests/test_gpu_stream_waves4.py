"""Streaming kernels on four wavefronts: every instance over group counts that leave wavefronts without a group, give them
odd numbers of groups and run past the scales of one fill of LDS (16 groups a wavefront, 8 from 64 tokens on), and
the library's own choice of them."""
import numpy as np
import pytest

from oracle import device_layout as lay
from oracle import qspec_oracle as orc
from paper_2410_11305_amd import synth

pytestmark = pytest.mark.gpu
TOL = 2e-3           # max |y - y_ref| / max |y_ref| against the float64 oracle
INSTANCES = [(tm, nt) for tm in (1, 2, 4) for nt in (2, 3, 4, 6) if tm * nt <= 16]


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2410_11305_amd import binding as B
    assert torch.cuda.is_available()
    B.lib()
    return torch, B


def to(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def draft_case(M, N, G, seed):
    """One live group per token row and power-of-two scales: y = fp16(P sa sw) in any summation order."""
    rng = np.random.default_rng(seed)
    qw = rng.integers(-8, 8, size=(N, 128 * G), dtype=np.int8)
    qa = np.zeros((M, 128 * G), np.int8)
    for m in range(M):
        g = G - 1 if m == 0 else (m * 37) % G
        qa[m, 128 * g:128 * g + 128] = rng.integers(-7, 8, size=128, dtype=np.int8)
    sa = (2.0 ** rng.integers(-3, 3, size=(M, G))).astype(np.float32)
    sw = (2.0 ** rng.integers(-9, -5, size=(N, G))).astype(np.float16)
    return qa, sa, qw, sw


@pytest.mark.parametrize("G", [1, 3, 9, 67, 131])
@pytest.mark.parametrize("tm,nt", INSTANCES)
def test_draft_mode_bit_exact(env, plan, tm, nt, G):
    torch, B = env
    M, N = 16 * tm - 3, 16 * (5 * nt + 1)
    plan("QSPEC_STREAM_MAX_W4A4", "128")
    plan("QSPEC_STREAM_W4A4", f"{nt},1,1,4")
    qa, sa, qw, sw = draft_case(M, N, G, G * 100 + tm * 10 + nt)
    y = B.gemm_w4a4(B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), N).cpu().numpy()
    assert np.array_equal(y.view(np.uint16), orc.gemm_w4a4(qa, sa, qw, sw).view(np.uint16))


@pytest.mark.parametrize("G", [1, 3, 9, 67])
@pytest.mark.parametrize("tm,nt", [i for i in INSTANCES if i[0] <= 2])
def test_verify_mode(env, plan, tm, nt, G):
    torch, B = env
    M, N, K = 16 * tm - 3, 16 * (5 * nt + 1), 128 * G
    plan("QSPEC_STREAM_W4A16", f"{nt},1,1,4")
    codes, scales, x = synth.generic_case(G * 100 + M, M, N, K)
    x[M // 2, K - 1] = np.inf                            # reaches its own token row only: no group is multiplied by zeros
    codes[:, K - 1] = 3
    y = B.gemm_w4a16(B.pack_weights(to(torch, codes), to(torch, scales)), to(torch, x), N).cpu().numpy()
    rows = np.arange(M) != M // 2
    ref = orc.gemm_w4a16(x[rows], codes, scales).astype(np.float64)
    assert np.isinf(y[M // 2]).all()
    assert np.max(np.abs(y[rows].astype(np.float64) - ref)) / np.max(np.abs(ref)) <= TOL


@pytest.mark.parametrize("M,N,K", [(5, 27648, 640), (16, 22016, 256), (30, 27648, 640), (48, 22016, 640), (64, 27648, 384)])
def test_more_than_one_round_of_workgroups(env, M, N, K):
    """The library's own plans, all outputs, twice."""
    torch, B = env
    qa, sa, qw, sw = draft_case(M, N, K // 128, M)
    args = B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), N
    y = B.gemm_w4a4(*args, workspace=B.alloc_workspace(B.workspace_bytes(M, N, K)))
    assert np.array_equal(y.cpu().numpy().view(np.uint16), orc.gemm_w4a4(qa, sa, qw, sw).view(np.uint16))
    assert torch.equal(y, B.gemm_w4a4(*args))


def test_an_instance_that_does_not_exist_is_refused(env, plan):
    torch, B = env
    qa, sa, qw, sw = draft_case(5, 64, 2, 0)
    args = B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), 64
    for forced in ("1,1,1,4", "2,1,1,5"):
        plan("QSPEC_STREAM_W4A4", forced)
        with pytest.raises(B.QSpecError):
            B.gemm_w4a4(*args)
