"""Parity of the batched products at the edges of their batch tiles, against the oracle's float64 product, with the
float32 dot-product bound of tests/test_gpu_spmm.py.  Every test runs in both forms, whichever the estimate favours at its
size: from the tile-based sections (the general form, and the one that keeps its results in registers, at up to 128
right-hand sides per workgroup) and from the section of four-row steps (16-bit operands: in panels)."""
import numpy as np
import pytest

import csb_inputs
import oracle

from paper_2005_05758_amd import CsbMatrix
from paper_2005_05758_amd import binding as csb

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from test_gpu_spmm import check_spmm            # noqa: E402
from test_gpu_val16 import FORMATS, packed      # noqa: E402


@pytest.fixture(autouse=True, params=["tiles", "quads"])
def form(request, monkeypatch):
    upload = CsbMatrix.upload

    def forced(M, *args, **kwargs):
        assert csb.lib().csb_debug_spmm_force(M._h, {"tiles": 1, "quads": 2}[request.param]) == 0
        return upload(M, *args, **kwargs)

    monkeypatch.setattr(CsbMatrix, "upload", forced)
    return request.param


# 256 row tiles and more: every compute unit gets a workgroup of 128 columns.  Batches one step
# below, at and above a tile; 16- and 32-row tiles; blocks of one and of several column passes.
@pytest.mark.parametrize("R,C,br,bc,batch", [(8192, 70, 32, 16, 68), (8192, 40, 32, 40, 128), (8190, 33, 32, 32, 132),
                                             (4100, 130, 16, 32, 124), (2060, 60, 16, 64, 260), (8190, 33, 32, 32, 196),
                                             (4100, 130, 16, 32, 196)])
def test_spmm_128_columns(R, C, br, bc, batch):
    m = csb_inputs.small_matrix(R + C + batch, R, C, br, bc, rate=4.0)
    check_spmm(m.A, br, bc, csb_inputs.make_vectors(batch, C, batch), tag="128-columns")


@pytest.mark.parametrize("fmt,name", FORMATS)
@pytest.mark.parametrize("R,C,br,bc,batch", [(8192, 70, 32, 16, 68), (8190, 33, 32, 32, 132), (4100, 130, 16, 32, 128),
                                             (4100, 130, 16, 32, 196)])
def test_spmm_16bit_128_columns(fmt, name, R, C, br, bc, batch):
    m = csb_inputs.small_matrix(R + C + batch, R, C, br, bc, rate=4.0)
    X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
    Aq, Xq = oracle.round_weights(m.A, name), oracle.round_weights(X, name).astype(np.float32)
    M = packed(m.A, br, bc, fmt)
    Xd = torch.from_numpy(Xq).cuda()
    ref, absr = oracle.matmat(Aq, Xq), oracle.matmat(np.abs(Aq), np.abs(Xq))
    k = np.count_nonzero(m.A, axis=1)[:, None]
    for Y in (M.spmm_bfloat(Xd.to(torch.bfloat16)) if name == "bf16" else M.spmm_half(Xd.to(torch.float16)), M.spmm(Xd)):
        torch.cuda.synchronize()
        got = Y.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= 2.0 * np.maximum(k, 1) * 2.0 ** -24 * absr + 1e-30)


# The general form: any batch, any alignment.  Batches around 16, 32 and 64 columns per workgroup (the last
# lanes move back to the batch's last right-hand sides), block sizes with partial 16-row slices and 16-column
# passes, and tiles taller than 32 rows.
@pytest.mark.parametrize("R,C,br,bc", [(70, 50, 16, 16), (200, 90, 64, 64), (150, 77, 33, 40), (8200, 41, 32, 32), (16400, 40, 64, 8)])
@pytest.mark.parametrize("batch", [2, 15, 17, 31, 49, 63, 66])
def test_spmm_any_batch(R, C, br, bc, batch):
    m = csb_inputs.small_matrix(R + C + batch, R, C, br, bc, rate=3.0)
    X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
    M, Y = check_spmm(m.A, br, bc, X, tag="any-batch")
    wide = torch.zeros((C, batch + 5), device="cuda")               # rows at odd word offsets
    wide[:, 3:3 + batch] = torch.from_numpy(X).cuda()
    wide[:, batch + 3:] = float("nan")                              # what lies beside the batch is never used
    out = torch.full((R, batch + 3), 7.0, device="cuda")
    M.spmm(wide[:, 3:3 + batch], out[:, 1:1 + batch])
    torch.cuda.synchronize()
    assert torch.all(out[:, 0] == 7.0) and torch.all(out[:, batch + 1:] == 7.0)
    ref = oracle.matmat(m.A, X)
    bound = 2.0 * np.maximum(np.count_nonzero(m.A, axis=1)[:, None], 1) * 2.0 ** -24 * oracle.matmat(np.abs(m.A), np.abs(X)) + 1e-30
    assert np.all(np.abs(out[:, 1:1 + batch].cpu().numpy().astype(np.float64) - ref) <= bound)


# What an input that is not finite does, in every form: the general one at 16, 32 and 64 columns, the register ones of
# 64 and 128 right-hand sides, 16 and 32 rows (from 256 row tiles on), and the 16-bit ones.
@pytest.mark.parametrize("R,br,batch", [(96, 32, 5), (96, 32, 33), (96, 32, 70), (8200, 32, 63), (8200, 64, 64), (8192, 32, 64),
                                        (8192, 32, 128), (4100, 16, 64), (4100, 16, 196)])
@pytest.mark.parametrize("fmt,name", [(None, "f32")] + FORMATS)
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_spmm_infinite_input(value, fmt, name, R, br, batch, form):
    """The rows that hold an entry of its column are not finite.  In the general float32 form, in four-row steps and in panels no
    others are touched (and an infinity stays one, with its sign); in the others no rows outside of the row tiles that hold
    the column.  Other right-hand sides are what they are."""
    C = 70
    m = csb_inputs.small_matrix(5, R, C, br, 32, rate=6.0)
    col = int(np.flatnonzero(np.count_nonzero(m.A, axis=0))[-1])
    batch = batch if fmt is None else (batch + 3) // 4 * 4
    general = form == "quads" or fmt is None and (br == 64 or R == 96 or batch % 4 != 0)
    X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
    X[col] = value
    X[col, 1::3] = 1.0                                             # (some right-hand sides are finite throughout)
    A = m.A
    if fmt is None:
        M = CsbMatrix(A, br, 32)
        M.plan()
        M.upload()
    else:
        M, A = packed(A, br, 32, fmt), oracle.round_weights(m.A, name)
        X = oracle.round_weights(X, name).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    Y = M.spmm(Xd) if fmt is None else M.spmm_bfloat(Xd.to(torch.bfloat16)) if name == "bf16" else M.spmm_half(Xd.to(torch.float16))
    got = Y.cpu().numpy().astype(np.float64)
    hit, odd = m.A[:, col] != 0, ~np.isfinite(X[col])
    at = np.ix_(hit, odd)
    assert not np.any(np.isfinite(got[at]))
    if general and np.isinf(value):
        assert np.all(np.isinf(got[at])) and np.all(np.sign(got[at]) == np.sign(m.A[hit, col])[:, None])
    apart = ~hit if general else ~np.isin(np.arange(R) // br, np.unique(np.flatnonzero(hit) // br))
    X[col, odd] = 0.0
    ref, absr = oracle.matmat(A, X), oracle.matmat(np.abs(A), np.abs(X))
    bound = 2.0 * np.maximum(np.count_nonzero(m.A, axis=1)[:, None], 1) * 2.0 ** -24 * absr + 1e-30
    for rows, cols in ((apart, odd), (np.ones(R, bool), ~odd)):
        at = np.ix_(rows, cols)
        assert np.all(np.abs(got[at] - ref[at]) <= bound[at])


# Rows of X beyond 2 GiB (float32) and beyond 1 GiB (16-bit): offsets of more than 31 bits.  Few
# right-hand sides in rows far apart; the general forms and, from 256 row tiles on, the register forms.
@pytest.mark.parametrize("R,br,batch", [(70, 64, 5), (4096, 16, 64), (4096, 16, 68)])
@pytest.mark.parametrize("fmt,name", [(None, "f32")] + FORMATS)
def test_spmm_input_rows_far_apart(fmt, name, R, br, batch):
    C, ld = 16380, 33400
    first = 16192                                                   # entries in the last columns only
    assert C * ld < 2 ** 30 and first * ld * (4 if fmt is None else 2) > 2 ** (31 if fmt is None else 30)
    batch = batch if fmt is None else (batch + 3) // 4 * 4
    m = csb_inputs.small_matrix(R + batch, R, C - first, br, 32, rate=4.0)
    A = np.zeros((R, C), np.float32)
    A[:, first:] = m.A
    X = csb_inputs.make_vectors(batch, C - first, batch).reshape(C - first, batch)
    if fmt is None:
        M = CsbMatrix(A, br, 32)
        M.plan()
        M.upload()
    else:
        M = packed(A, br, 32, fmt)
    A, X = (m.A, X) if fmt is None else (oracle.round_weights(m.A, name), oracle.round_weights(X, name).astype(np.float32))
    wide = torch.empty((C, ld), dtype={"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[name], device="cuda")
    wide[:, 4:4 + batch] = 0.0
    wide[first:, 4:4 + batch] = torch.from_numpy(X).cuda()
    Y = {"f32": M.spmm, "f16": M.spmm_half, "bf16": M.spmm_bfloat}[name](wide[:, 4:4 + batch])
    torch.cuda.synchronize()
    k = np.maximum(np.count_nonzero(A, axis=1)[:, None], 1)
    err = np.abs(Y.cpu().numpy().astype(np.float64) - oracle.matmat(A, X))
    assert np.all(err <= 2.0 * k * 2.0 ** -24 * oracle.matmat(np.abs(A), np.abs(X)) + 1e-30)


# Row tiles of 750 blocks, whose records take several segments, among empty ones up to 256 tiles: the register
# forms of 64 and 128 right-hand sides, whose wavefronts open block after block and start again in every segment.
@pytest.mark.parametrize("R,br", [(8192, 32), (4096, 16)])
@pytest.mark.parametrize("fmt,name", [(None, "f32")] + FORMATS)
def test_spmm_long_row_tiles(fmt, name, R, br):
    C, rows = 12000, 2 * br
    m = csb_inputs.small_matrix(21, rows, C, br, 16, rate=2.0)
    A = np.zeros((R, C), np.float32)
    A[br:br + rows] = m.A
    if fmt is None:
        M = CsbMatrix(A, br, 16)
        M.plan()
        M.upload()
    else:
        M = packed(A, br, 16, fmt)
    Aq = m.A if fmt is None else oracle.round_weights(m.A, name)
    k = np.maximum(np.count_nonzero(m.A, axis=1)[:, None], 1)
    for batch in (64, 128):
        X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
        if fmt is not None:
            X = oracle.round_weights(X, name).astype(np.float32)
        Xd = torch.from_numpy(X).cuda()
        Y = M.spmm(Xd) if fmt is None else M.spmm_bfloat(Xd.to(torch.bfloat16)) if name == "bf16" else M.spmm_half(Xd.to(torch.float16))
        torch.cuda.synchronize()
        got = Y.cpu().numpy().astype(np.float64)
        ref, absr = oracle.matmat(Aq, X), oracle.matmat(np.abs(Aq), np.abs(X))
        assert np.all(np.abs(got[br:br + rows] - ref) <= 2.0 * k * 2.0 ** -24 * absr + 1e-30)
        assert not got[:br].any() and not got[br + rows:].any()


# Two sources (x_t and h_{t-1}), one layer and two per launch: batches that take 64 columns without being
# multiples of four, and the register forms of 64 and 128.  256 row tiles of 16 rows, or 128 of 32 and two layers.
@pytest.mark.parametrize("block", [16, 32])
@pytest.mark.parametrize("batch", [50, 63, 64, 68, 128, 132])
@pytest.mark.parametrize("fmt,name", [(None, "f32"), FORMATS[0]])
def test_rnn_batch_tiles(fmt, name, block, batch):
    from paper_2005_05758_amd import CsbRnn
    T, H = 3, 1024
    wl = csb_inputs.make_rnn(csb_inputs.RnnConfig("t", csb_inputs.LSTM, 2, 40, H, block, 12.0, "binomial", 0.05, batch, T, 90 + batch))
    Ws = [CsbMatrix(w.A, w.br, w.bc) for w in wl.W]
    if fmt is not None:
        for w in Ws:
            w.set_value_format(fmt)
    rnn = CsbRnn(csb_inputs.LSTM, 40, H, Ws, [torch.from_numpy(b).cuda() for b in wl.bias])
    for w in Ws:
        w.upload()
    rng = np.random.default_rng(batch)
    h0, c0 = (rng.uniform(-0.5, 0.5, (2, batch, H)).astype(np.float32) for _ in range(2))
    W = [w.A if fmt is None else oracle.round_weights(w.A, name) for w in wl.W]
    ref = oracle.rnn_forward(csb_inputs.LSTM, W, wl.bias, wl.x, 40, H, h0=h0, c0=c0)
    got = rnn.forward(torch.from_numpy(wl.x).cuda(), torch.from_numpy(h0).cuda(), torch.from_numpy(c0).cuda())
    torch.cuda.synchronize()
    err = [float(np.max(np.abs(g.cpu().numpy() - r))) for g, r in zip(got, ref)]
    print(f"[tiles] rnn block {block} batch {batch} {name}: {err}", flush=True)
    assert max(err) <= 1e-4
