"""The section of the device image that the batched products read: csb_plan_validate walks it the way
the kernels do and rebuilds the matrix from it.  No GPU."""
import numpy as np
import pytest

import csb_inputs
from paper_2005_05758_amd import CsbMatrix, CsbRnn, load_library
from paper_2005_05758_amd import binding as csb


# Blocks lower and taller than a row tile (16 or 32 rows), passes of 1 to 8 columns, kernel rows in fours and not,
# rows and columns that end inside a tile, a block, a pass.
@pytest.mark.parametrize("R,C,br,bc", [(33, 70, 1, 9), (37, 53, 8, 8), (64, 65, 16, 16), (150, 77, 33, 40), (200, 90, 64, 64),
                                       (130, 100, 128, 128), (8200, 33, 16, 32), (300, 17, 256, 8)])
@pytest.mark.parametrize("fmt", [csb.VAL_F32, csb.VAL_F16, csb.VAL_BF16])
def test_section_holds_the_matrix(fmt, R, C, br, bc):
    for rate in (1.0, 3.0) if R < 1000 else (3.0,):
        M = CsbMatrix(csb_inputs.small_matrix(R + C, R, C, br, bc, rate=rate).A, br, bc)
        M.set_value_format(fmt)
        for mode in (0, 1, 2) if R < 1000 else (0,):
            M.plan(mode=mode)
            M.validate()
        M.plan_rows()
        M.validate()


# A recurrent handle's matrices: passes end where the input's two sources meet, the GRU's candidate rows are
# summed in two parts.
@pytest.mark.parametrize("cell,gates", [(csb.CELL_LSTM, 4), (csb.CELL_GRU, 3), (csb.CELL_LIGRU, 2), (csb.CELL_LSTMP, 4), (csb.CELL_GRU_RB, 3)])
@pytest.mark.parametrize("inputs,hidden,block", [(5, 40, 16), (39, 33, 32), (64, 100, 64)])
def test_section_of_a_recurrent_handle(cell, gates, inputs, hidden, block):
    state = 24 if cell == csb.CELL_LSTMP else hidden
    A = csb_inputs.small_matrix(7, gates * hidden, inputs + state, block, block, rate=3.0).A.copy()
    second = []
    if cell == csb.CELL_GRU_RB:
        A[2 * hidden:, inputs:] = 0.0
        second = [CsbMatrix(csb_inputs.small_matrix(8, hidden, hidden, block, block, rate=3.0).A, block, block)]
    if cell == csb.CELL_LSTMP:
        second = [CsbMatrix(csb_inputs.small_matrix(8, state, hidden, block, block, rate=3.0).A, block, block)]
    W = CsbMatrix(A, block, block)
    CsbRnn(cell, inputs, hidden, [W], proj=state if cell == csb.CELL_LSTMP else 0, Wp=second or None)
    for m in [W] + second:
        m.validate()


# The handle's plan cuts no pass where a gate ends: with an input that ends with a block it has those of a plain plan.
@pytest.mark.parametrize("hidden,block", [(100, 32), (301, 32), (500, 64), (77, 16)])
def test_gates_do_not_cut_tiles(hidden, block):
    inputs = 2 * block
    A = csb_inputs.small_matrix(5, 4 * hidden, inputs + hidden, block, block, rate=3.0).A
    plain, W = CsbMatrix(A, block, block), CsbMatrix(A, block, block)
    plain.plan()
    CsbRnn(csb.CELL_LSTM, inputs, hidden, [W])
    for rows in (16, 32):
        passes = [load_library().csb_debug_quad_passes(m._h, rows) for m in (plain, W)]
        assert passes[0] == passes[1]
    assert any(load_library().csb_debug_quad_passes(W._h, rows) for rows in (16, 32))


# What a 16-bit gate matrix of a handle holds for products of right-hand sides: the tile-based sections.
@pytest.mark.parametrize("fmt", [csb.VAL_F16, csb.VAL_BF16])
@pytest.mark.parametrize("cell,gates", [(csb.CELL_LSTM, 4), (csb.CELL_GRU, 3)])
def test_no_section_that_nothing_reads(cell, gates, fmt):
    A = csb_inputs.small_matrix(5, gates * 64, 96, 32, 32, rate=3.0).A
    W, plain = CsbMatrix(A, 32, 32), CsbMatrix(A, 32, 32)
    for m in (W, plain):
        m.set_value_format(fmt)
    plain.plan()
    CsbRnn(cell, 32, 64, [W])
    W.validate()
    passes = [[load_library().csb_debug_quad_passes(m._h, rows) for rows in (16, 32)] for m in (W, plain)]
    assert passes[0] == [0, 0] and all(passes[1])


# A matrix that was planned before its handle was created, or is planned again after, has the section that a handle's own
# plan has: cut where the input's two sources meet, inside a block here.
@pytest.mark.parametrize("plan", ["plan", "mode1", "mode2", "rows"])
@pytest.mark.parametrize("cell,gates", [(csb.CELL_LSTM, 4), (csb.CELL_GRU, 3), (csb.CELL_LIGRU, 2), (csb.CELL_LSTMP, 4), (csb.CELL_GRU_RB, 3)])
def test_section_of_a_matrix_planned_by_its_caller(cell, gates, plan):
    inputs, hidden, state = 39, 64, 48 if cell == csb.CELL_LSTMP else 64
    A = csb_inputs.small_matrix(7, gates * hidden, inputs + state, 32, 32, rate=2.0).A.copy()
    B = csb_inputs.small_matrix(8, state, hidden, 32, 32, rate=2.0).A
    if cell == csb.CELL_GRU_RB:
        A[2 * hidden:, inputs:] = 0.0

    def handle(before, after):
        W = CsbMatrix(A, 32, 32)
        second = [CsbMatrix(B, 32, 32)] if cell in (csb.CELL_GRU_RB, csb.CELL_LSTMP) else []
        call = {"plan": W.plan, "mode1": lambda: W.plan(mode=1), "mode2": lambda: W.plan(mode=2), "rows": W.plan_rows}[plan]
        if before:
            call()
        CsbRnn(cell, inputs, hidden, [W], proj=state if cell == csb.CELL_LSTMP else 0, Wp=second or None)
        if after:
            call()
        for m in [W] + second:
            m.validate()
        return [load_library().csb_debug_quad_passes(W._h, rows) for rows in (16, 32)]

    own = handle(False, False)
    assert handle(True, False) == own and all(own)
    if not (cell == csb.CELL_GRU and plan == "rows"):                     # (the rows of a GRU step are laid out by its handle alone)
        assert handle(False, True) == own
