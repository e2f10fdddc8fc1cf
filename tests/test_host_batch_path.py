"""The estimate by which csb_rnn_forward runs a batch on the resident kernel or on the batched products, at
sizes where both were measured (us per step on MI355X): it takes the faster one.  No GPU."""
import pytest

import csb_inputs
from paper_2005_05758_amd import CELL_GRU, CELL_LSTM, CELL_LSTMP, CsbMatrix, CsbRnn, load_library


def handle(cell, L, I, H, block, rate, law):
    if cell == CELL_LSTMP:
        wl = csb_inputs.make_lstmp(3, L, I, H, H // 2, block, rate, 1, 1, sigma=0.05)
        return CsbRnn(cell, I, H, [CsbMatrix(m.A, m.br, m.bc) for m in wl.W], None, proj=H // 2,
                      Wp=[CsbMatrix(m.A, m.br, m.bc) for m in wl.Wp])
    wl = csb_inputs.make_rnn(csb_inputs.RnnConfig("t", cell, L, I, H, block, rate, law, 0.05, 1, 1, 3))
    return CsbRnn(cell, I, H, [CsbMatrix(m.A, m.br, m.bc) for m in wl.W], None)


# model, then batch: (us on the resident kernel, us on the batched products)
@pytest.mark.parametrize("cell,L,I,H,block,rate,law,measured", [
    (CELL_LSTM, 1, 153, 512, 32, 10.0, "binomial", {8: (1.5, 8.3), 32: (5.9, 8.9), 64: (11.8, 9.0)}),
    (CELL_GRU, 1, 256, 1024, 32, 16.0, "beta", {8: (3.3, 9.0), 16: (6.7, 9.2), 32: (13.3, 9.6), 64: (26.6, 10.9)}),
    (CELL_LSTM, 2, 1024, 1024, 64, 25.0, "binomial", {4: (4.0, 11.4), 8: (8.0, 12.9), 16: (16.0, 11.7), 64: (64.8, 14.4)}),
    (CELL_LSTM, 1, 64, 128, 16, 8.0, "binomial", {2: (1.2, 8.2), 64: (1.2, 8.3)}),
    (CELL_LSTM, 2, 153, 256, 16, 8.0, "binomial", {16: (5.9, 8.7), 64: (23.4, 9.8)}),
    (CELL_LSTMP, 1, 153, 512, 32, 13.0, "binomial", {16: (5.8, 16.2), 32: (11.6, 16.7), 64: (23.0, 16.3)}),
    (CELL_LSTM, 1, 512, 1024, 32, 12.0, "binomial", {4: (3.5, 10.8), 8: (6.9, 9.9), 16: (13.9, 10.2), 64: (55.4, 12.3)}),
    (CELL_LSTM, 4, 64, 256, 16, 8.0, "binomial", {4: (1.5, 8.4), 64: (24.1, 10.9)}),
    (CELL_LSTM, 6, 64, 256, 16, 8.0, "binomial", {4: (3.2, 15.9), 64: (51.0, 19.4)})])
def test_the_faster_path(cell, L, I, H, block, rate, law, measured):
    rnn = handle(cell, L, I, H, block, rate, law)
    got = {b: load_library().csb_debug_rnn_prefers_resident(rnn._h, b) for b in measured}
    assert got == {b: int(res < bat) for b, (res, bat) in measured.items()}


# The ring of the last layer's outputs is part of the workspace where the call uses it: from about half a million words of output
# on, and at least 65536 a step.  (A model whose input is too wide for the resident layout: what else grows with the steps
# are its input frames.)
@pytest.mark.parametrize("hidden,batch,T,ring", [(16, 4, 64, False), (64, 40, 64, False), (64, 48, 64, False), (1024, 47, 16, False), (1024, 64, 6, False),
                                                 (1024, 64, 7, True), (1024, 256, 1, False), (1024, 256, 2, True), (1024, 512, 1, True)])
def test_workspace_of_a_batch(hidden, batch, T, ring):
    W = CsbMatrix(csb_inputs.small_matrix(3, 4 * hidden, 2100 + hidden, 64, 64, rate=25.0).A, 64, 64)
    rnn = CsbRnn(CELL_LSTM, 2100, hidden, [W], None)
    assert rnn.device_bytes() == 0
    # (gate sums, cell and output states, frames, the merge words of a mat-vec; every part rounded up to 256 bytes)
    plain = W.workspace_bytes(1) + 4 * batch * (4 * hidden + 3 * hidden + 2100 * min(T, max(1, (8 << 20) // (4 * batch * 2100))))
    extra = rnn.workspace_bytes(batch, T) - plain
    assert (extra > 4 * batch * hidden if ring and T > 1 else extra >= 4 * batch * hidden if ring else extra < 8192)
