"""Verify-mode products that run as two launches, the whole blocks of 128 tokens and the rows left over: the row
where they meet, the last row, what lies behind it, and every kind of second launch."""
import ctypes

import numpy as np
import pytest

from oracle import qspec_oracle as orc
from paper_2410_11305_amd import synth

pytestmark = pytest.mark.gpu
TOL = 2e-3           # max |y - y_ref| / max |y_ref| against the float64 oracle


@pytest.mark.parametrize("M,N,K,second", [(2061, 4080, 768, "stream_kernel<false, 1, 1>"), (661, 12000, 768, "stream_kernel<false, 2, 3>"),
                                          (566, 14544, 1024, "tile16w_kernel<1, 2, 2"), (1924, 8672, 640, "stream_kernel<false, 1, 3>"),
                                          (217, 16, 1408, "stream_kernel<false, 1, 1>")])
def test_both_launches_against_the_oracle(M, N, K, second):
    import torch
    from paper_2410_11305_amd import binding as B
    name = ctypes.create_string_buffer(128)
    assert B.lib().qspec_describe_kernel(5, M, N, K, 128, name, 128) == 0 and second in name.value.decode()
    rows = M // 128 * 128
    codes, scales, x = synth.generic_case(M, M, N, K)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    blob, xd = B.pack_weights(to(codes), to(scales)), to(x)
    ws = B.alloc_workspace(B.workspace_bytes(M, N, K))
    guarded = torch.full((M + 8, N), 7.0, dtype=torch.float16, device="cuda")
    y = B.gemm_w4a16(blob, xd, N, y=guarded[:M], workspace=ws)
    again = B.gemm_w4a16(blob, xd, N, workspace=ws)
    sample = np.unique(np.r_[0, 127, rows - 128, rows - 1:min(rows + 34, M), M - 1])
    ref = orc.gemm_w4a16(x[sample], codes, scales).astype(np.float64)
    err = np.max(np.abs(y.cpu().numpy()[sample].astype(np.float64) - ref)) / np.max(np.abs(ref))
    assert err <= TOL
    assert torch.equal(y, again) and bool((guarded[M:] == 7.0).all())
    own = torch.empty((M, N), dtype=torch.float16, device="cuda")
    assert B.lib().qspec_gemm_w4a16_noalloc(blob.data_ptr(), xd.data_ptr(), M, N, K, 128, own.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(own, y)
