"""The estimate by which csb_rnn_forward runs a batch on the resident kernel or on the batched products, at
sizes where both were measured (us per step on MI355X): it takes the faster one.  No GPU."""
import pytest

import csb_inputs
from paper_2005_05758_amd import CELL_GRU, CELL_LIGRU, CELL_LSTM, CELL_LSTMP, CsbMatrix, CsbRnn, load_library


def handle(cell, L, I, H, block, rate, law):
    if cell == CELL_LSTMP:
        wl = csb_inputs.make_lstmp(3, L, I, H, H // 2, block, rate, 1, 1, sigma=0.05)
        return CsbRnn(cell, I, H, [CsbMatrix(m.A, m.br, m.bc) for m in wl.W], None, proj=H // 2,
                      Wp=[CsbMatrix(m.A, m.br, m.bc) for m in wl.Wp])
    wl = csb_inputs.make_rnn(csb_inputs.RnnConfig("t", cell, L, I, H, block, rate, law, 0.05, 1, 1, 3))
    return CsbRnn(cell, I, H, [CsbMatrix(m.A, m.br, m.bc) for m in wl.W], None)


# model, then batch: (us on the resident kernel, us on the batched products)
@pytest.mark.parametrize("cell,L,I,H,block,rate,law,measured", [
    (CELL_LSTM, 1, 153, 512, 32, 10.0, "binomial", {8: (1.4, 7.1), 32: (5.3, 7.2), 64: (10.5, 7.6)}),
    (CELL_GRU, 1, 256, 1024, 32, 16.0, "beta", {8: (3.1, 7.5), 16: (6.1, 7.4), 24: (9.1, 7.6), 32: (12.1, 7.8), 64: (24.1, 8.4)}),
    (CELL_LSTM, 2, 1024, 1024, 64, 25.0, "binomial", {4: (3.6, 9.3), 8: (7.1, 9.3), 16: (14.0, 9.4), 64: (56.1, 10.8)}),
    (CELL_LSTM, 1, 64, 128, 16, 8.0, "binomial", {2: (0.9, 6.1), 64: (0.9, 6.3)}),
    (CELL_LSTM, 2, 153, 256, 16, 8.0, "binomial", {16: (5.3, 7.6), 32: (10.5, 7.8), 64: (21.1, 8.0)}),
    (CELL_LSTMP, 1, 153, 512, 32, 13.0, "binomial", {16: (5.0, 10.1), 24: (7.5, 10.3), 48: (15.1, 10.4), 64: (20.3, 10.5)}),
    (CELL_LSTM, 1, 512, 1024, 32, 12.0, "binomial", {4: (3.2, 8.4), 8: (6.3, 8.4), 16: (12.6, 8.4), 64: (50.8, 9.5)}),
    (CELL_LSTM, 4, 64, 256, 16, 8.0, "binomial", {4: (2.9, 7.9), 8: (5.7, 8.0), 16: (11.2, 7.9), 64: (45.3, 8.9)}),
    (CELL_LSTM, 6, 64, 256, 16, 8.0, "binomial", {4: (3.1, 15.1), 16: (12.2, 15.0), 64: (49.6, 16.3)}),
    (CELL_GRU, 2, 512, 512, 32, 20.0, "binomial", {8: (2.7, 7.6), 16: (5.4, 7.5), 32: (10.7, 7.9)}),
    (CELL_LIGRU, 2, 39, 512, 32, 7.1, "binomial", {8: (3.1, 8.3), 16: (6.3, 8.2), 33: (14.8, 8.5)})])
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
