"""The estimate by which batched products read the tile-based sections or the section of four-row steps (16-bit operands: in panels,
always), and how wide a workgroup's share of the right-hand sides is, at sizes where both were measured (us on MI355X): it takes the
faster one.  No GPU."""
import ctypes

import numpy as np
import pytest

import csb_inputs
from paper_2005_05758_amd import CsbMatrix, VAL_BF16, VAL_F32, load_library


def form(R, C, block, rate, law, fmt, batch):
    A = np.random.default_rng(3).standard_normal((R, C), np.float32) if rate == 1.0 else csb_inputs.make_mat(csb_inputs.MatConfig("t", R, C, block, rate, law, 0.05), 3).A
    M = CsbMatrix(A, block, block)
    M.set_value_format(fmt)
    M.plan()
    out = (ctypes.c_int32 * 3)()
    assert load_library().csb_debug_spmm_form(M._h, batch, int(fmt != VAL_F32), out) == 0
    return list(out)


@pytest.mark.parametrize("R,C,block,rate,fmt,batch,tiles,quads", [
    (4096, 4096, 32, 1.0, VAL_F32, 128, 45.0, 63.7), (4096, 4096, 32, 4.0, VAL_F32, 128, 30.6, 28.0),
    (4096, 4096, 32, 1.0, VAL_BF16, 512, 58.9, 39.0), (4096, 4096, 32, 4.0, VAL_BF16, 512, 45.9, 23.9),
    (8192, 2048, 16, 1.25, VAL_BF16, 192, 47.8, 30.9), (9252, 2045, 16, 2.0, VAL_BF16, 12, 24.4, 18.0),
    (2048, 2048, 16, 2.0, VAL_F32, 16, 12.1, 14.2), (2048, 2048, 16, 4.0, VAL_F32, 64, 13.8, 10.2),
    (4100, 2048, 24, 4.0, VAL_F32, 4, 11.5, 16.8), (4100, 2048, 24, 4.0, VAL_F32, 32, 19.5, 16.4),
    (16384, 1024, 32, 8.0, VAL_F32, 4, 10.0, 12.4), (16384, 1024, 32, 4.0, VAL_F32, 64, 23.6, 19.2),
    (2048, 2048, 64, 1.0, VAL_BF16, 64, 33.6, 6.6)])
def test_the_faster_section(R, C, block, rate, fmt, batch, tiles, quads):
    assert (form(R, C, block, rate, "binomial", fmt, batch)[0] == 0) == (tiles < quads)


# us by (rows of a tile, right-hand sides, wavefronts of a workgroup)
@pytest.mark.parametrize("R,C,block,rate,law,fmt,batch,measured", [
    (8192, 8192, 32, 12.0, "heavy", VAL_F32, 512, {(32, 128, 16): 128.0, (32, 128, 8): 115.0}),
    (8192, 8192, 32, 12.0, "heavy", VAL_F32, 16, {(32, 32, 16): 21.7, (32, 64, 16): 25.4}),
    (8192, 8192, 32, 12.0, "heavy", VAL_BF16, 512, {(32, 64, 8): 59.6, (32, 128, 8): 44.9}),
    (8192, 8192, 32, 12.0, "heavy", VAL_BF16, 64, {(32, 64, 8): 10.5, (32, 128, 8): 13.8}),
    (4096, 4096, 16, 8.0, "binomial", VAL_F32, 64, {(16, 32, 16): 23.5, (16, 64, 16): 15.3}),
    (4096, 4096, 16, 8.0, "binomial", VAL_BF16, 64, {(16, 64, 8): 7.0, (16, 128, 8): 9.0}),
    (4096, 4096, 16, 8.0, "binomial", VAL_BF16, 256, {(16, 64, 8): 19.3, (16, 128, 8): 15.5}),
    (2048, 2048, 32, 12.0, "binomial", VAL_BF16, 64, {(32, 64, 4): 5.6, (32, 64, 8): 5.8, (16, 64, 4): 5.1, (16, 64, 8): 4.8, (16, 128, 8): 5.9}),
    (4096, 2048, 64, 25.0, "binomial", VAL_BF16, 256, {(32, 64, 4): 6.5, (32, 64, 8): 7.1, (32, 128, 4): 6.8, (16, 64, 4): 7.3, (16, 128, 4): 7.1}),
    (2048, 2048, 32, 12.0, "binomial", VAL_F32, 64, {(32, 32, 16): 7.4, (16, 32, 16): 6.0}),
    (4096, 2048, 64, 25.0, "binomial", VAL_F32, 64, {(32, 32, 16): 5.7, (16, 64, 16): 5.2})])
def test_the_faster_share(R, C, block, rate, law, fmt, batch, measured):
    assert tuple(form(R, C, block, rate, law, fmt, batch)) == min(measured, key=measured.get)
