"""Sizes at the edge of what the entry points accept: a packed weight tensor just under
the 2 GiB that the kernels' 32-bit byte offsets reach, the largest input dimension that
goes with it, and a token count far beyond any decoding batch.  The weights are drawn on
the device (seeded); the oracle sees the sampled rows only."""
import numpy as np
import pytest

from oracle import qspec_oracle as orc

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2410_11305_amd import binding as B
    assert torch.cuda.is_available()
    B.lib()
    return torch, B


def rel_err(y, ref):
    return float(np.max(np.abs(y.astype(np.float64) - ref)) / max(np.max(np.abs(ref)), 1e-30))


def test_weight_tensor_just_under_two_gib(env, plan):
    torch, B = env
    N, K = 32800, 130944                      # N*K/2 = 2 147 481 600 bytes of codes (limit: 2^31 - 2)
    assert N * K // 2 < 2 ** 31 - 1 <= (N + 16) * K // 2
    G = K // 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    codes = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    scales = (torch.rand((N, G), device="cuda", generator=gen) * 0.008 + 0.002).half()
    blob = B.pack_weights(codes, scales)
    assert blob.numel() == B.packed_weight_bytes(N, K) == N * K // 2 + N * G * 2
    cols = np.unique(np.concatenate([np.arange(16), np.arange(N - 16, N), [N // 2, N // 2 + 17, 12345, 30001, 32767, 32768]]))
    c_h = codes[torch.from_numpy(cols).cuda()].cpu().numpy()
    s_h = scales[torch.from_numpy(cols).cuda()].cpu().numpy()
    # the round trip of the sampled rows (first tile, last tile, middle)
    back_c, back_s = B.unpack_weights(blob, N, K)
    assert torch.equal(back_c[-16:], codes[-16:]) and torch.equal(back_c[:16], codes[:16])
    assert torch.equal(back_s, scales)
    del back_c, back_s, codes
    rng = np.random.default_rng(78)
    for M in (8, 96):                          # the streaming and the tiled kernels
        x = rng.standard_normal((M, K)).astype(np.float16)
        x[:, rng.choice(K, K // 100, replace=False)] *= 20
        xd = torch.from_numpy(x).cuda()
        qa, sa = B.quant_act(xd)
        q_ref, s_ref = orc.quant_act(x)
        assert np.array_equal(sa.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
        y4 = B.gemm_w4a4(blob, qa, sa, N)
        y16 = B.gemm_w4a16(blob, xd, N)
        torch.cuda.synchronize()
        print(M, B.describe_kernel(True, M, N, K), B.describe_kernel(False, M, N, K), flush=True)
        y4, y16 = y4.cpu().numpy(), y16.cpu().numpy()
        assert np.isfinite(y4).all() and np.isfinite(y16).all()
        e4 = rel_err(y4[:, cols], orc.gemm_w4a4(q_ref, s_ref, c_h, s_h))
        e16 = rel_err(y16[:, cols], orc.gemm_w4a16(x, c_h, s_h))
        print(f"   rel err w4a4 {e4:.2e}  w4a16 {e16:.2e}", flush=True)
        assert e4 <= TOL and e16 <= TOL
    # the last M again on the shapes of the verify mode that its plan does not take: 512 x 128 blocks, the K
    # groups dealt to sets of wavefronts, alone and in slices
    ref16 = orc.gemm_w4a16(x, c_h, s_h)
    for forced in ("7,1", "0,1", "1,1", "2,1", "3,1", "5,2", "6,1"):
        plan("QSPEC_TILE_W4A16", forced)
        y16 = B.gemm_w4a16(blob, xd, N).cpu().numpy()
        e16 = rel_err(y16[:, cols], ref16)
        print(f"   {forced}: {B.describe_kernel(False, M, N, K)} {e16:.2e}", flush=True)
        assert np.isfinite(y16).all() and e16 <= TOL


def test_one_row_too_many_is_refused(env):
    torch, B = env
    a = torch.zeros(64, dtype=torch.uint8, device="cuda")
    assert B.packed_weight_bytes(32800 + 16, 130944) == 0
    with pytest.raises(B.QSpecError):
        B.gemm_w4a16(a, torch.zeros((1, 130944), dtype=torch.float16, device="cuda"), 32800 + 16,
                     y=torch.zeros((1, 32800 + 16), dtype=torch.float16, device="cuda"))
    torch.cuda.synchronize()


def test_twenty_thousand_tokens(env, plan):
    torch, B = env
    M, N, K = 20001, 48, 1024                 # 157 token blocks of 128 or 313 of 64, the last with one or 33 rows
    rng = np.random.default_rng(79)
    codes = rng.integers(-8, 8, (N, K), dtype=np.int8)
    scales = rng.uniform(0.002, 0.01, (N, K // 128)).astype(np.float16)
    x = rng.standard_normal((M, K)).astype(np.float16)
    blob = B.pack_weights(torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda())
    xd = torch.from_numpy(x).cuda()
    qa, sa = B.quant_act(xd)
    q_ref, s_ref = orc.quant_act(x)
    assert np.array_equal(sa.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
    y4 = B.gemm_w4a4(blob, qa, sa, N).cpu().numpy()
    y16 = B.gemm_w4a16(blob, xd, N).cpu().numpy()
    assert rel_err(y4, orc.gemm_w4a4(q_ref, s_ref, codes, scales)) <= TOL
    ref16 = orc.gemm_w4a16(x, codes, scales)
    assert rel_err(y16, ref16) <= TOL
    for shape in range(8):                    # whatever the plan, every block shape of the verify mode
        plan("QSPEC_TILE_W4A16", f"{shape},1")
        assert rel_err(B.gemm_w4a16(blob, xd, N).cpu().numpy(), ref16) <= TOL, shape


def test_activations_just_under_two_gib(env, plan):
    """Row offsets near 2^31: every block shape on the last rows of an activation matrix of 2 GiB."""
    torch, B = env
    K, N = 16384, 16
    M = (2 ** 31 - 2) // (2 * K)              # 65535 tokens: M * K * 2 = 2^31 - 32768 bytes
    gen = torch.Generator(device="cuda")
    gen.manual_seed(80)
    x = torch.randn((M, K), device="cuda", generator=gen, dtype=torch.float16)
    rng = np.random.default_rng(81)
    codes = rng.integers(-8, 8, (N, K), dtype=np.int8)
    scales = rng.uniform(0.002, 0.01, (N, K // 128)).astype(np.float16)
    blob = B.pack_weights(torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda())
    rows = np.r_[0:8, M // 2:M // 2 + 8, M - 140:M]
    ref = orc.gemm_w4a16(x[torch.from_numpy(rows).cuda()].cpu().numpy(), codes, scales)
    for forced in [None] + [f"{shape},1" for shape in range(8)]:
        plan("QSPEC_TILE_W4A16", forced)
        y = B.gemm_w4a16(blob, x, N).cpu().numpy()
        assert np.isfinite(y).all() and rel_err(y[rows], ref) <= TOL, forced


@pytest.mark.parametrize("blocks", [37837, 37838])
def test_more_token_blocks_than_the_reciprocal_covers(env, plan, blocks):
    """Tiled kernels find their output block by a reciprocal while blocks of tokens squared times blocks of outputs stays below
    2^32, by a division from there on: the last size of the one and the first of the other, 64 x 64 blocks.  Token
    rows repeat with a period that is no multiple of a block, so every row has to equal the same row of a small call."""
    torch, B = env
    M, N, K, period = 64 * blocks - 40, 176, 128, 8191
    assert (blocks * blocks * 3 >= 2 ** 32) == (blocks == 37838)
    rng = np.random.default_rng(83)
    codes = rng.integers(-8, 8, (N, K), dtype=np.int8)
    scales = rng.uniform(0.002, 0.01, (N, 1)).astype(np.float16)
    x = rng.standard_normal((period, K)).astype(np.float16)
    blob = B.pack_weights(torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda())
    few = torch.from_numpy(x).cuda()
    rows = torch.arange(M, device="cuda") % period
    many = few[rows]
    plan("QSPEC_TILE_W4A16", "2,1")
    plan("QSPEC_TILE_W4A4", "2,1")
    for product, ref in ((lambda t: B.gemm_w4a16(blob, t, N), orc.gemm_w4a16(x, codes, scales)),
                         (lambda t: B.gemm_w4a4(blob, *B.quant_act(t), N), orc.gemm_w4a4(*orc.quant_act(x), codes, scales)),
                         (lambda t: B.gemm_w4a4_wide(blob, *B.quant_act_wide(t), N), orc.gemm_w4a4(*orc.quant_act(x), codes, scales))):
        y = product(few)
        assert rel_err(y.cpu().numpy(), ref) <= TOL
        assert torch.equal(product(many), y[rows])
