"""Host rules of the library: which kernel a call takes, and how much scratch it accepts (no GPU needed)."""
import ctypes

import pytest
import torch

from paper_2605_10886_amd import binding as B


def _check(desc, nbytes):
    """loka_fp8_gemm_norm_check on a clear workspace of `nbytes`: on the device where there is one; without one the size is
    still judged, and an accepted workspace then ends in LOKA_ERR_HIP at the copy of its header."""
    dev = "cuda:0" if torch.cuda.is_available() else "cpu"
    ws = torch.zeros(max(nbytes, 16) + 256, dtype=torch.uint8, device=dev)
    p = (ws.data_ptr() + 255) // 256 * 256
    return B.lib().loka_fp8_gemm_norm_check(ctypes.byref(desc), p, nbytes, None)


# (the FP8-output form needs less than the bf16 call, more, the same, or is the only one of the two that waits)
@pytest.mark.parametrize("M,N,K", [(1024, 2560, 4096), (1000, 1536, 4096), (512, 1024, 2048), (300, 4096, 4096), (2048, 4096, 4096),
                                   (5013, 720, 1024), (65536, 1024, 1024)])
def test_wait_check_takes_the_workspace_of_either_call(M, N, K):
    L, d = B.lib(), B.make_desc(M, N, K, norm=B.NORM_LAYERNORM)
    sizes = [int(L.loka_fp8_gemm_norm_workspace(ctypes.byref(d))), int(L.loka_fp8_gemm_norm_fp8out_workspace(ctypes.byref(d)))]
    for n in sizes:
        assert _check(d, n) != B.LOKA_ERR_WORKSPACE, (sizes, n)
