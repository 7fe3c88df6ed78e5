"""Bit parity of loka_quantize where its tiles and row shares end: partial last tiles of the TENSOR / COL passes in both
layouts (including a strided input), and rows held by one workgroup."""
import numpy as np
import pytest
import torch

from paper_2605_10886_amd import binding as B
from paper_2605_10886_amd import synth

pytestmark = pytest.mark.gpu


def _check(orc, x, mode, transpose_out=False, ld=None):
    xg = x.to("cuda:0")
    if ld:
        wide = torch.full((x.shape[0], ld), 9.0e9, dtype=torch.bfloat16, device="cuda:0")    # what lies beyond is not read
        wide[:, :x.shape[1]] = xg
        xg = wide[:, :x.shape[1]]
    q_o, s_o = orc.quantize(synth.bf16_bits(x), mode, transpose_out=transpose_out)
    q, s = B.loka_quantize(xg, mode, transpose_out)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), s_o.view(np.uint32))
    assert np.array_equal(q.cpu().numpy(), q_o)


@pytest.mark.parametrize("rows,cols", [(16, 16), (112, 144), (128, 128), (144, 48), (272, 400), (8208, 80), (16, 4112)])
@pytest.mark.parametrize("mode", [B.SCALE_TENSOR, B.SCALE_COL])
@pytest.mark.parametrize("transpose_out", [False, True])
def test_tensor_and_column_tiles(orc, rows, cols, mode, transpose_out):
    x = synth.student_t4(rows, cols, seed=rows * 3 + cols)
    x[:, 5] = 0
    _check(orc, x, mode, transpose_out, ld=None if rows % 32 else cols + 24)


@pytest.mark.parametrize("rows,cols", [(1, 48), (77, 208), (129, 1008)])
@pytest.mark.parametrize("mode", [B.SCALE_TENSOR, B.SCALE_COL])
def test_rows_of_any_number_without_transposition(orc, rows, cols, mode):
    _check(orc, synth.normal(rows, cols, seed=rows), mode)


@pytest.mark.parametrize("rows,cols", [(3, 8208), (513, 8224), (2, 16384), (2, 16400), (515, 32784), (1, 65552), (2, 131072),
                                       (259, 65536), (2, 131088)])
def test_rows_longer_than_a_wave_holds(orc, rows, cols):
    x = synth.normal(rows, cols, seed=cols)
    x[0, cols - 1] = 300.0              # the maximum in the last chunk
    if rows > 1:
        x[1] = 0
    _check(orc, x, B.SCALE_ROW, ld=cols + 8 if rows < 4 else None)


# every share of a row (lanes, chunks per lane, rows per wave) of the one-pass kernel, whose groups' scales are taken by different
# lanes: rows that do not fill a wave's share, a row of zeros, the maximum at the end of the first group and the start of the last
@pytest.mark.parametrize("rows,cols", [(1, 128), (7, 128), (11, 256), (70003, 256), (5, 512), (33001, 512), (9, 1024), (17003, 1024),
                                       (6, 2048), (9, 4096), (3, 8192)])
@pytest.mark.parametrize("mode", [B.SCALE_ROW, B.SCALE_BLOCK_1x128, B.SCALE_BLOCK_1x128_POW2])
def test_groups_whose_scales_other_lanes_take(orc, rows, cols, mode):
    x = synth.student_t4(rows, cols, seed=cols + rows)
    x[:, 127] *= 64
    x[-1, cols - 128] = -500.0
    if rows > 2:
        x[1] = 0
    _check(orc, x, mode, ld=cols + 8 if rows < 8 else None)


# tensors that are read past the caches give what their parts, which are not, give
@pytest.mark.parametrize("rows,cols", [(131072, 256), (65536, 512), (8192, 4096)])
@pytest.mark.parametrize("mode", [B.SCALE_ROW, B.SCALE_BLOCK_128x128, B.SCALE_TENSOR])
def test_streamed_reads_change_nothing(rows, cols, mode):
    x = synth.student_t4(rows // 8, cols, seed=7).to("cuda:0").repeat(8, 1)
    q, s = B.loka_quantize(x, mode)
    q1, s1 = B.loka_quantize(x[:rows // 8], mode)
    assert torch.equal(q.view(8, rows // 8, cols), q1.expand(8, -1, -1))
    assert torch.equal(s if mode == B.SCALE_TENSOR else s.view(8, -1), s1 if mode == B.SCALE_TENSOR else s1.reshape(1, -1).expand(8, -1))
