"""The native marshalling of the per-step calls: what it rejects before anything is allocated (no GPU), and, on the GPU,
that given outputs and workspaces are the ones written and that a failed call raises with the library's status."""
import pytest
import torch

from paper_2605_10886_amd import binding as B


def test_rejects_before_allocating():
    with pytest.raises(AssertionError):
        B.loka_quantize(torch.zeros(8, 16), B.SCALE_ROW)                          # not bf16
    with pytest.raises(AssertionError):
        B.loka_quantize(torch.zeros(16, 8, dtype=torch.bfloat16).t(), B.SCALE_ROW)   # columns strided
    with pytest.raises(B.LokaError) as e:
        B.loka_quantize(torch.zeros(16, 200, dtype=torch.bfloat16), B.SCALE_BLOCK_1x128)
    assert e.value.status == B.LOKA_ERR_SHAPE
    with pytest.raises(Exception):
        B.loka_fp8_gemm_norm(object(), *(torch.zeros(1),) * 4)                    # not a descriptor
    with pytest.raises(AssertionError):
        B.loka_probe_error(torch.zeros(4, 8), torch.zeros(8, 4))


@pytest.mark.gpu
def test_given_outputs_and_errors():
    M, K, N = 96, 128, 256
    x = torch.randn(M, K, device="cuda").bfloat16()
    wq, sw = B.loka_quantize((torch.randn(K, N, device="cuda") / 11).bfloat16(), B.SCALE_COL, transpose_out=True)
    xq, sx = B.loka_quantize(x, B.SCALE_ROW)
    d = B.make_desc(M, N, K)
    ref, none = B.loka_fp8_gemm_norm(d, xq, sx, wq, sw)
    out, y = torch.empty_like(ref), torch.empty(M, N, device="cuda")
    o2, y2 = B.loka_fp8_gemm_norm(d, xq, sx, wq, sw, want_y=True, out=out, y=y)
    assert none is None and o2.data_ptr() == out.data_ptr() and y2.data_ptr() == y.data_ptr()
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    wide = B.make_desc(M, 2048, K, norm=B.NORM_LAYERNORM, variant=B.variant_id("panel32_256x256"))
    with pytest.raises(B.LokaError) as e:
        B.loka_fp8_gemm_norm(wide, xq, sx, torch.zeros(2048, K, dtype=torch.uint8, device="cuda"),
                             torch.ones(2048, device="cuda"), workspace=ws)
    assert e.value.status == B.LOKA_ERR_WORKSPACE


@pytest.mark.gpu
def test_tensor_without_storage_raises():
    # a batched view has a shape and a device but no address of its own: the error leaves the call as a Python exception
    x = torch.randn(2, 32, 128, device="cuda").bfloat16()
    with pytest.raises(RuntimeError):
        torch.vmap(lambda t: B.loka_quantize(t, B.SCALE_ROW)[0])(x)
    y = torch.zeros(2, 32, 128, device="cuda")
    with pytest.raises(RuntimeError):
        torch.vmap(lambda t: B.loka_probe_error(t, t, sync=False)[1])(y)
    codes, _ = B.loka_quantize(x[0], B.SCALE_ROW)                                 # and the next call runs
    assert codes.shape == (32, 128)


def test_variant_ids_keep_their_place():
    # callers keep ids (a dispatch choice, a descriptor): entries are added at the end
    names = ["row32x128", "row64x128", "row64x256", "row128x256", "row64x512", "row64x1024", "exact64x256", "exact64x512",
             "exact64x1024", "wreg32", "strip32", "twopass128x128", "twopass256x256", "twopass256x256w8", "splitk128x128",
             "splitk128x128s2", "panel256x256w8", "panel32_256x256"]
    assert [B.variant_id(n) for n in names] == list(range(len(names)))
