"""Tiled draft-mode kernel: every workgroup shape and both activation formats at group counts with none,
one and two groups left over behind the loop over threes, alone and in two K-slices.  One live group per
token row and power-of-two scales make y = fp16(P sa sw) in any summation order: bit for bit."""
import numpy as np
import pytest

from oracle import device_layout as lay
from oracle import qspec_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("G", [2, 3, 4, 5, 7, 11])
@pytest.mark.parametrize("shape", range(4))
def test_groups_left_over_behind_the_loop(plan, shape, G, S):
    import torch
    from paper_2410_11305_amd import binding as B
    M, N = 133, 272
    plan("QSPEC_TILE_W4A4", f"{shape},{S}")
    rng = np.random.default_rng(G * 10 + shape)
    qw = rng.integers(-8, 8, size=(N, 128 * G), dtype=np.int8)
    qa = np.zeros((M, 128 * G), np.int8)
    for m in range(M):
        g = (G - 1 - m) % G
        qa[m, 128 * g:128 * g + 128] = rng.integers(-7, 8, size=128, dtype=np.int8)
    sa = (2.0 ** rng.integers(-3, 3, size=(M, G))).astype(np.float32)
    sw = (2.0 ** rng.integers(-9, -5, size=(N, G))).astype(np.float16)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    assert B.describe_kernel(True, M, N, 128 * G).startswith("gemm_tile4w_kernel")
    blob, ws = B.pack_weights(to(qw), to(sw)), B.alloc_workspace(B.workspace_bytes(M, N, 128 * G))
    ref = orc.gemm_w4a4(qa, sa, qw, sw).view(np.uint16)
    packed = B.gemm_w4a4(blob, to(lay.act_bytes(qa)), to(sa), N, workspace=ws).cpu().numpy()
    wide = B.gemm_w4a4_wide(blob, to(lay.act_wide_bytes(qa)), to(sa), N, workspace=ws).cpu().numpy()
    assert np.array_equal(packed.view(np.uint16), ref) and np.array_equal(wide.view(np.uint16), ref)
