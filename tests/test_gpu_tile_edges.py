"""The verify-mode tiled kernels where their splits run out: fewer K groups than sets of wavefronts
that deal them, an odd number of groups under the two-group loop, last blocks of one row or
sixteen columns.  Against the float64 oracle at the tolerance of the fp16 outputs (2e-3 of the
largest: one fp16 rounding of the result and one of each dequantised weight)."""
import numpy as np
import pytest

from oracle import qspec_oracle as orc
from paper_2410_11305_amd import synth

pytestmark = pytest.mark.gpu
TOL = 2e-3


def _case(plan, shape, S, M, N, G):
    import torch
    from paper_2410_11305_amd import binding as B
    plan("QSPEC_TILE_W4A16", f"{shape},{S}")
    K = 128 * G
    codes, scales, x = synth.generic_case(1000 * shape + 10 * G + M % 10, M, N, K)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    blob = B.pack_weights(to(codes), to(scales))
    buf = torch.full((M * N + 512,), 321.0, dtype=torch.float16, device="cuda")
    ws = B.alloc_workspace(B.workspace_bytes(M, N, K))
    y = B.gemm_w4a16(blob, to(x), N, y=buf[256:256 + M * N].view(M, N), workspace=ws)
    torch.cuda.synchronize()
    ref = orc.gemm_w4a16(x, codes, scales).astype(np.float64)
    err = np.max(np.abs(y.cpu().numpy().astype(np.float64) - ref)) / np.max(np.abs(ref))
    assert err <= TOL, (B.describe_kernel(False, M, N, K), err)
    assert (buf[:256] == 321.0).all() and (buf[-256:] == 321.0).all()
    assert int(ws[:16384].count_nonzero()) == 0 or S == 1


@pytest.mark.parametrize("G", [1, 2, 3, 8])
@pytest.mark.parametrize("M,N", [(129, 16), (160, 528), (257, 1040)])
def test_512_by_128_blocks(plan, M, N, G):
    _case(plan, 7, 1, M, N, G)


@pytest.mark.parametrize("S,G", [(1, 1), (1, 2), (1, 3), (1, 5), (2, 5), (2, 9), (4, 13)])
@pytest.mark.parametrize("shape", [1, 2, 3, 5])
def test_k_groups_dealt_to_sets_of_wavefronts(plan, shape, S, G):
    _case(plan, shape, S, 129, 208, G)
