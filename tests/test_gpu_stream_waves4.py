"""Streaming kernels on four wavefronts: every instance over group counts that leave wavefronts without a group, give them
odd numbers of groups and run past the scales of one fill of LDS (16 groups a wavefront, 8 from 64 tokens on), in K-slices and
blocks of token rows, and the library's own choice of them in both modes."""
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


@pytest.mark.parametrize("G", [5, 67])
@pytest.mark.parametrize("S", [2, 5])
@pytest.mark.parametrize("tm,nt", INSTANCES)
def test_k_slices(env, plan, tm, nt, S, G):
    """More slices than groups for some wavefronts; the counters are left at zero."""
    torch, B = env
    M, N = 16 * tm - 3, 16 * (3 * nt + 1)
    plan("QSPEC_STREAM_MAX_W4A4", "128")
    plan("QSPEC_STREAM_W4A4", f"{nt},{S},1,4")
    qa, sa, qw, sw = draft_case(M, N, G, G * 100 + tm * 10 + nt)
    args = B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), N
    ws = B.alloc_workspace(B.workspace_bytes(M, N, 128 * G))
    y = B.gemm_w4a4(*args, workspace=ws)
    assert np.array_equal(y.cpu().numpy().view(np.uint16), orc.gemm_w4a4(qa, sa, qw, sw).view(np.uint16))
    assert torch.equal(y, B.gemm_w4a4(*args, workspace=ws)) and not ws[:16384].any()


@pytest.mark.parametrize("tm,nt,ms", [(tm, nt, ms) for tm, nt in INSTANCES for ms in (2, 4) if 16 * tm * ms <= 128])
def test_row_blocks(env, plan, tm, nt, ms):
    """A ragged last block of token rows, and one that starts past M (four blocks of three blocks' rows)."""
    torch, B = env
    M = 16 * tm * ms - (3 if ms == 2 else 16 * tm + 5)
    N, G = 16 * (5 * nt + 1), 9
    plan("QSPEC_STREAM_MAX_W4A4", "128")
    plan("QSPEC_STREAM_W4A4", f"{nt},1,{ms},4")
    assert B.describe_kernel(True, M, N, 128 * G) == f"waves4::gemm_stream_kernel<true, {tm}, {nt}>"
    qa, sa, qw, sw = draft_case(M, N, G, ms * 100 + tm * 10 + nt)
    y = B.gemm_w4a4(B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), N).cpu().numpy()
    assert np.array_equal(y.view(np.uint16), orc.gemm_w4a4(qa, sa, qw, sw).view(np.uint16))


# sizes at which the library itself takes four wavefronts, by token tiles, weight tiles and token-row blocks
OWN_DRAFT = [(1, 25104, 256, "1, 4"), (33, 8528, 384, "1, 4"), (65, 5568, 256, "1, 4"), (17, 32208, 1024, "2, 4"), (49, 16816, 2048, "2, 3"),
             (60, 18592, 2048, "2, 6"), (96, 10896, 2048, "2, 3"), (33, 22144, 4096, "4, 3"), (100, 12672, 4096, "4, 4")]
OWN_VERIFY = [(1, 25104, 4096, "1, 4"), (17, 25104, 256, "2, 4"), (23, 36944, 256, "2, 6"), (17, 32800, 2048, "2, 3")]


def sample_of(N):
    """Columns of the first tile block, of the last ones and some between."""
    return np.unique(np.r_[0:100, N // 2:N // 2 + 50, N - 130:N])


@pytest.mark.parametrize("M,N,K,instance", OWN_DRAFT)
def test_the_librarys_own_draft_plans(env, plan, M, N, K, instance):
    """Sampled columns bit for bit against the oracle, all of them against the kernel of eight wavefronts."""
    torch, B = env
    assert B.describe_kernel(True, M, N, K) == f"waves4::gemm_stream_kernel<true, {instance}>"
    qa, sa, qw, sw = draft_case(M, N, K // 128, M)
    args = B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), N
    y = B.gemm_w4a4(*args, workspace=B.alloc_workspace(B.workspace_bytes(M, N, K)))
    cols = sample_of(N)
    assert np.array_equal(y.cpu().numpy()[:, cols].view(np.uint16), orc.gemm_w4a4(qa, sa, qw[cols], sw[cols]).view(np.uint16))
    assert torch.equal(y, B.gemm_w4a4(*args))
    tm, nt = map(int, instance.split(", "))
    if M <= 16 * tm:
        plan("QSPEC_STREAM_W4A4", f"{nt},1")
        assert B.describe_kernel(True, M, N, K) == f"gemm_stream_kernel<true, {instance}>"
        assert torch.equal(y, B.gemm_w4a4(*args))


@pytest.mark.parametrize("M,N,K,instance", OWN_VERIFY)
def test_the_librarys_own_verify_plans(env, M, N, K, instance):
    torch, B = env
    assert B.describe_kernel(False, M, N, K) == f"waves4::gemm_stream_kernel<false, {instance}>"
    codes, scales, x = synth.generic_case(M, M, N, K)
    args = B.pack_weights(to(torch, codes), to(torch, scales)), to(torch, x), N
    y = B.gemm_w4a16(*args)
    cols = sample_of(N)
    ref = orc.gemm_w4a16(x, codes[cols], scales[cols]).astype(np.float64)
    assert np.max(np.abs(y.cpu().numpy()[:, cols].astype(np.float64) - ref)) / np.max(np.abs(ref)) <= TOL
    assert torch.equal(y, B.gemm_w4a16(*args))


def test_an_instance_that_does_not_exist_is_refused(env, plan):
    torch, B = env
    qa, sa, qw, sw = draft_case(5, 64, 2, 0)
    args = B.pack_weights(to(torch, qw), to(torch, sw)), to(torch, lay.act_bytes(qa)), to(torch, sa), 64
    for forced in ("1,1,1,4", "2,1,1,5"):
        plan("QSPEC_STREAM_W4A4", forced)
        with pytest.raises(B.QSpecError):
            B.gemm_w4a4(*args)
