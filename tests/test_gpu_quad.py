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


# Tiles of 16 rows up to 256 of them, of 32 where those would take another turn over the CUs: 4090 rows at 64 and 65 right-hand
# sides, one row more than there are such tiles for, blocks that they cut in two, in four and unevenly.
@pytest.mark.parametrize("R,C,block", [(4090, 70, 32), (4096, 130, 64), (4097, 50, 33), (2050, 90, 24)])
@pytest.mark.parametrize("batch", [4, 64, 68, 132, 260])
@pytest.mark.parametrize("fmt", [csb.VAL_F32, csb.VAL_F16, csb.VAL_BF16])
def test_both_tile_heights(R, C, block, batch, fmt):
    A = csb_inputs.small_matrix(R + C, R, C, block, block, rate=3.0).A
    M = CsbMatrix(A, block, block)
    M.set_value_format(fmt)
    M.plan()
    M.validate()
    M.upload()
    X = torch.from_numpy(csb_inputs.make_vectors(batch, C, batch).reshape(C, batch))
    to = {csb.VAL_F32: torch.float32, csb.VAL_F16: torch.float16, csb.VAL_BF16: torch.bfloat16}[fmt]
    X = X.to(to)
    Y = {csb.VAL_F32: M.spmm, csb.VAL_F16: M.spmm_half, csb.VAL_BF16: M.spmm_bfloat}[fmt](X.cuda())
    torch.cuda.synchronize()
    Ar, Xr = torch.from_numpy(A).to(to).float().numpy(), X.float().numpy()      # (the rounded operands: their products are exact in float32)
    assert np.all(np.abs(Y.cpu().numpy().astype(np.float64) - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr))


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


# The last layer's outputs are turned over a ring of steps at a time: 16 here, so 40 steps fill it twice and a half; on
# either side of the size from which on they are (65536 words a step, 450000 in all), and with the projected cell, where they always are.
@pytest.mark.parametrize("cell,layers,batch,T", [(csb.CELL_LSTM, 2, 2048, 40), (csb.CELL_LSTM, 1, 2048, 16), (csb.CELL_GRU, 1, 2048, 17),
                                                 (csb.CELL_LIGRU, 2, 47, 3), (csb.CELL_LIGRU, 2, 48, 3), (csb.CELL_LSTMP, 2, 5, 4),
                                                 (csb.CELL_LSTM, 1, 64, 1), (csb.CELL_LSTMP, 1, 2100, 35), (csb.CELL_LIGRU, 2, 1024, 6),
                                                 (csb.CELL_LIGRU, 2, 1024, 7), (csb.CELL_GRU, 1, 1023, 9)])
def test_output_sequence_of_a_batch(cell, layers, batch, T):
    inputs, hidden, state = 10, 64, 40 if cell == csb.CELL_LSTMP else 64
    gates = {csb.CELL_LSTM: 4, csb.CELL_GRU: 3, csb.CELL_LIGRU: 2, csb.CELL_LSTMP: 4}[cell]
    A = [csb_inputs.small_matrix(20 + l, gates * hidden, (inputs if l == 0 else state) + state, 16, 16, rate=4.0).A * 0.1 for l in range(layers)]
    P = [csb_inputs.small_matrix(40 + l, state, hidden, 16, 16, rate=2.0).A * 0.1 for l in range(layers)] if cell == csb.CELL_LSTMP else []
    W, Wp = [CsbMatrix(a, 16, 16) for a in A], [CsbMatrix(p, 16, 16) for p in P]
    rnn = CsbRnn(cell, inputs, hidden, W, proj=state if P else 0, Wp=Wp or None)
    for m in W + Wp:
        m.upload()
    x = np.random.default_rng(T).uniform(-1, 1, (T, batch, inputs)).astype(np.float32)
    ref = oracle.lstmp_forward(A, P, None, x, inputs, hidden, state) if P else oracle.rnn_forward(cell, A, None, x, inputs, hidden)
    for _ in range(2):                                              # (the second call finds the first one's ring)
        got = rnn.forward(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        for g, r in zip(got, ref):
            if g is not None:
                assert np.max(np.abs(g.cpu().numpy() - r)) <= 1e-4
    alone = rnn.forward(torch.from_numpy(x).cuda(), want_hseq=False)  # without the sequence: the state in place
    assert alone[0] is None and torch.equal(alone[1], got[1])


# Matrices that their caller planned before the handle was created: not uploaded yet (their section is cut anew), uploaded (they
# keep the image on the GPU), and uploaded after into a buffer of the size that was asked for before.
# (A GRU handle plans its matrices itself: an upload before it is void, and so is a size that was asked for before.)
@pytest.mark.parametrize("cell,gates,upload", [(csb.CELL_LSTM, 4, "after"), (csb.CELL_LSTM, 4, "before"), (csb.CELL_LSTM, 4, "told"),
                                               (csb.CELL_LIGRU, 2, "told"), (csb.CELL_GRU, 3, "after")])
@pytest.mark.parametrize("batch", [3, 70])
def test_batch_with_matrices_planned_by_the_caller(cell, gates, upload, batch):
    inputs, hidden = 39, 100
    A = [csb_inputs.small_matrix(20 + l, gates * hidden, (inputs, hidden)[l] + hidden, 32, 32, rate=4.0).A * 0.1 for l in range(2)]
    W = [CsbMatrix(a, 32, 32) for a in A]
    for m in W:
        m.plan()
    told = [m.device_bytes() for m in W]
    if upload == "before":
        for m in W:
            m.upload()
    rnn = CsbRnn(cell, inputs, hidden, W)
    bufs = [torch.zeros(n, dtype=torch.uint8, device="cuda") for n in told]
    for m, n, buf in zip(W, told, bufs):
        if upload == "after":
            m.upload()
        elif upload == "told":
            assert csb.lib().csb_upload(m._h, buf.data_ptr(), n - 1, None) == -2      # CSB_ENOMEM
            assert csb.lib().csb_upload(m._h, buf.data_ptr(), n, None) == 0
            m.validate()
    x = np.random.default_rng(batch).uniform(-1, 1, (5, batch, inputs)).astype(np.float32)
    got, ref = rnn.forward(torch.from_numpy(x).cuda()), oracle.rnn_forward(cell, A, None, x, inputs, hidden)
    torch.cuda.synchronize()
    for g, r in zip(got, ref):
        if g is not None:
            assert np.max(np.abs(g.cpu().numpy() - r)) <= 1e-4


# Layers whose blocks are of different heights: their matrices' tiles have 16 or 32 rows, and share a launch.
@pytest.mark.parametrize("blocks", [(16, 64), (32, 16), (64, 24)])
@pytest.mark.parametrize("batch", [3, 33, 130])
def test_layers_of_different_block_heights(blocks, batch):
    inputs, hidden = 40, 100
    A = [csb_inputs.small_matrix(30 + l, 4 * hidden, (inputs, hidden)[l] + hidden, b, b, rate=4.0).A * 0.1 for l, b in enumerate(blocks)]
    W = [CsbMatrix(a, b, b) for a, b in zip(A, blocks)]
    rnn = CsbRnn(csb.CELL_LSTM, inputs, hidden, W)
    for m in W:
        assert csb.lib().csb_debug_spmm_force(m._h, 2) == 0
        m.upload()
    x = np.random.default_rng(batch).uniform(-1, 1, (6, batch, inputs)).astype(np.float32)
    got, ref = rnn.forward(torch.from_numpy(x).cuda()), oracle.rnn_forward(csb.CELL_LSTM, A, None, x, inputs, hidden)
    torch.cuda.synchronize()
    for g, r in zip(got, ref):
        assert np.max(np.abs(g.cpu().numpy() - r)) <= 1e-4
