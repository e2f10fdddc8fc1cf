"""Parity of the batched products where their route changes: rows of the input so far apart that they take
the tile-based form, and a matrix planned by a recurrent handle (tiles end with a gate, the input comes as two
sources), against the oracle's float64 product with the float32 dot-product bound."""
import numpy as np
import pytest

import csb_inputs
import oracle
from paper_2005_05758_amd import CsbMatrix, CsbRnn
from paper_2005_05758_amd import binding as csb

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def bound_of(A, X):
    return 2.0 * np.maximum(np.count_nonzero(A, axis=1)[:, None], 1) * 2.0 ** -24 * oracle.matmat(np.abs(A), np.abs(X)) + 1e-30


# 16383 is the largest stride of the quad form; both sides of it, at the edges of 32, 64 and 128 right-hand sides.
@pytest.mark.parametrize("batch", [1, 31, 32, 33, 64, 65, 127, 129])
@pytest.mark.parametrize("ldx", [16383, 16384])
def test_strides_on_both_sides_of_the_limit(ldx, batch):
    R, C = 150, 90
    A = csb_inputs.small_matrix(3, R, C, 32, 32, rate=3.0).A
    M = CsbMatrix(A, 32, 32)
    M.plan()
    M.upload()
    X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
    wide = torch.full((C, ldx), float("nan"), device="cuda")        # what lies beside the batch is never used
    wide[:, 2:2 + batch] = torch.from_numpy(X).cuda()
    Y = M.spmm(wide[:, 2:2 + batch])
    torch.cuda.synchronize()
    assert np.all(np.abs(Y.cpu().numpy().astype(np.float64) - oracle.matmat(A, X)) <= bound_of(A, X))


@pytest.mark.parametrize("inputs,hidden,block", [(39, 33, 32), (64, 100, 64), (5, 520, 16)])
@pytest.mark.parametrize("batch", [3, 40, 130])
def test_product_with_a_recurrent_handles_matrix(inputs, hidden, block, batch):
    A = csb_inputs.small_matrix(7, 4 * hidden, inputs + hidden, block, block, rate=3.0).A
    M = CsbMatrix(A, block, block)
    CsbRnn(csb.CELL_LSTM, inputs, hidden, [M])
    M.upload()
    X = csb_inputs.make_vectors(batch, inputs + hidden, batch).reshape(inputs + hidden, batch)
    Y = M.spmm(torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert np.all(np.abs(Y.cpu().numpy().astype(np.float64) - oracle.matmat(A, X)) <= bound_of(A, X))
