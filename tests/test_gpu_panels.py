"""Parity of the 16-bit products in panels (csb_spmm_bfloat / csb_spmm_half), in every form of a launch, against the oracle's float64
product of the rounded operands with the float32 dot-product bound (their products are exact in float32)."""
import ctypes

import numpy as np
import pytest

import csb_inputs
import oracle
from paper_2005_05758_amd import CsbMatrix
from paper_2005_05758_amd import binding as csb

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
TYPES = {csb.VAL_F16: torch.float16, csb.VAL_BF16: torch.bfloat16}


def product(A, br, bc, fmt, X, ldx=None, form=None, first=0):
    """(result, rounded A, rounded X); `form`: what the call has to take (rows of a tile, right-hand sides, wavefronts); `first`: X's place in
    its rows."""
    M = CsbMatrix(A, br, bc)
    M.set_value_format(fmt)
    M.plan()
    M.upload()
    C, batch = X.shape
    if form is not None:
        got = (ctypes.c_int32 * 3)()
        assert csb.lib().csb_debug_spmm_panel(M._h, batch, got) == 0 and tuple(got) == form
    wide = torch.full((C, ldx or batch), float("nan"), device="cuda").to(TYPES[fmt])      # what lies beside the batch is never used
    wide[:, first:first + batch] = torch.from_numpy(X).cuda().to(TYPES[fmt])
    out = torch.full((A.shape[0], batch + 3), 7.0, device="cuda")
    call = M.spmm_half if fmt == csb.VAL_F16 else M.spmm_bfloat
    call(wide[:, first:first + batch], out[:, 1:1 + batch])
    torch.cuda.synchronize()
    assert torch.all(out[:, 0] == 7.0) and torch.all(out[:, batch + 1:] == 7.0)
    return out[:, 1:1 + batch].cpu().numpy().astype(np.float64), torch.from_numpy(A).to(TYPES[fmt]).float().numpy(), wide[:, first:first + batch].float().cpu().numpy()


def bound_of(A, X):
    return 2.0 * np.maximum(np.count_nonzero(A, axis=1)[:, None], 1) * 2.0 ** -24 * oracle.matmat(np.abs(A), np.abs(X)) + 1e-30


# Every form, at row counts beside a multiple of its tile and at batches one step below, at and above its columns; with 128 the last
# lane has eight right-hand sides (128) or moves back to the last eight (68, 124, 260, 508).
@pytest.mark.parametrize("R,C,block,rate,batch,form", [
    (150, 90, 16, 3.0, 4, (16, 64, 8)), (97, 600, 33, 2.0, 60, (16, 64, 8)), (4090, 70, 32, 3.0, 64, (16, 64, 4)),
    (4090, 70, 32, 3.0, 260, (16, 64, 4)), (4100, 70, 24, 3.0, 8, (32, 64, 4)), (4500, 2600, 32, 1.5, 60, (32, 64, 8)),
    (4097, 2500, 16, 2.0, 124, (16, 128, 8)), (4097, 1500, 16, 4.0, 124, (16, 128, 4)), (4097, 1500, 16, 4.0, 128, (16, 128, 4)),
    (4500, 2600, 32, 1.5, 68, (32, 128, 8)), (5000, 900, 32, 4.0, 260, (32, 128, 4)), (8200, 300, 16, 1.5, 508, (32, 128, 4))])
@pytest.mark.parametrize("fmt", list(TYPES))
def test_every_form(R, C, block, rate, batch, form, fmt):
    A = csb_inputs.small_matrix(3, R, C, block, block, rate=rate).A
    got, Ar, Xr = product(A, block, block, fmt, csb_inputs.make_vectors(batch, C, batch).reshape(C, batch), batch + 12, form)
    assert np.all(np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr))


# X at 8 bytes from a multiple of 16, every row of it or every second one, in the forms of 128 right-hand sides (loads of 16 bytes) and of 64.
@pytest.mark.parametrize("R,C,block,rate,batch,form", [(97, 600, 33, 2.0, 60, (16, 64, 8)), (4097, 2500, 16, 2.0, 124, (16, 128, 8)),
                                                       (4097, 1500, 16, 4.0, 128, (16, 128, 4)), (4500, 2600, 32, 1.5, 68, (32, 128, 8)),
                                                       (5000, 900, 32, 4.0, 260, (32, 128, 4))])
@pytest.mark.parametrize("beside", [8, 12])
def test_x_aligned_to_8_bytes(R, C, block, rate, batch, form, beside):
    A = csb_inputs.small_matrix(3, R, C, block, block, rate=rate).A
    ldx = (batch + 7) // 8 * 8 + beside
    got, Ar, Xr = product(A, block, block, csb.VAL_BF16, csb_inputs.make_vectors(batch, C, batch).reshape(C, batch), ldx, form, first=4)
    assert np.all(np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr))


# Lists of very different lengths are found through a table: one full block row of 1100 that are nearly empty.
@pytest.mark.parametrize("batch", [12, 72])
def test_lists_of_different_lengths(batch):
    R, C = 1100 * 32, 4000
    A = np.zeros((R, C), np.float32)
    A[64:96] = np.random.default_rng(1).standard_normal((32, C), np.float32)
    A[::640, 7] = 1.0
    got, Ar, Xr = product(A, 32, 32, csb.VAL_BF16, csb_inputs.make_vectors(2, C, batch).reshape(C, batch))
    assert np.all(np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr))


# Records of more than 2 GiB: 257 tiles of 16 lists, 8400 records of 64 bytes from one list to the next, are 2.21e9 bytes (32390400 passes; the
# first 32 tiles have half as many as the others).
def test_records_beyond_2_gib():
    R, C = 257 * 32, 4200
    A = np.random.default_rng(1).standard_normal((R, C), np.float32)
    A[:1024, ::2] = 0.0
    got, Ar, Xr = product(A, 1, 1, csb.VAL_BF16, csb_inputs.make_vectors(3, C, 4).reshape(C, 4))
    assert np.all(np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr))


# 65536 tiles by 128 groups of right-hand sides by 512 threads are 2^32 threads, more than a grid's row has: the last right-hand
# sides are a launch of their own.  (288 passes a tile: lists of more than 16, for which there are no workgroups of 256 threads.)
def test_more_threads_than_a_grid_has():
    R, C, batch = 65536 * 32, 9, 16380
    if torch.cuda.mem_get_info()[0] < 4 * R * batch + (8 << 30):
        pytest.skip("no memory for a result of 137 GB")
    A = np.random.default_rng(1).standard_normal((R, C), np.float32)
    M = CsbMatrix(A, 1, 1)
    M.set_value_format(csb.VAL_BF16)
    M.plan()
    M.upload()
    form = (ctypes.c_int32 * 3)()
    assert csb.lib().csb_debug_spmm_panel(M._h, batch, form) == 0 and form[2] == 8
    X = torch.from_numpy(csb_inputs.make_vectors(5, C, batch)).cuda().to(torch.bfloat16)
    Y = M.spmm_bfloat(X)
    torch.cuda.synchronize()
    Ad, Xd = torch.from_numpy(A).cuda().to(torch.bfloat16).float(), X.float()
    for rows in (slice(0, 64), slice(R // 2 - 32, R // 2 + 32), slice(R - 64, R)):
        ref, absr = Ad[rows].double() @ Xd.double(), Ad[rows].abs().double() @ Xd.abs().double()
        assert torch.all((Y[rows].double() - ref).abs() <= 2.0 * C * 2.0 ** -24 * absr + 1e-30)
    del Y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("R,block,batch", [(96, 16, 12), (96, 32, 132), (8200, 32, 196), (4100, 16, 260)])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_an_input_that_is_not_finite_reaches_the_rows_that_use_it_alone(value, R, block, batch):
    C = 300
    A = csb_inputs.small_matrix(5, R, C, block, 32, rate=6.0).A
    X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
    col = int(np.flatnonzero(np.count_nonzero(A, axis=0))[-1])
    X[col, ::3] = value
    got, Ar, Xr = product(A, block, 32, csb.VAL_BF16, X)
    odd, hit = ~np.isfinite(X[col]), Ar[:, col] != 0
    at = np.ix_(hit, odd)
    assert not np.any(np.isfinite(got[at]))
    if np.isinf(value):
        assert np.all(np.sign(got[at]) == np.sign(Ar[hit, col])[:, None])
    Xr[col, odd] = 0.0
    good = np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr)
    good[at] = True
    assert np.all(good)


# Which right-hand sides are computed again: in workgroups of 128 either 64 of them or all, in binary16 as in bfloat16.  `odd`: the
# right-hand sides with such an input, in the first, the second or both halves of a workgroup, among the last four of a batch.
@pytest.mark.parametrize("R,C,block,rate,batch,odd,form", [
    (96, 300, 32, 6.0, 64, [5], (16, 64, 8)), (5000, 900, 32, 4.0, 260, [7], (32, 128, 4)), (5000, 900, 32, 4.0, 260, [127, 259], (32, 128, 4)),
    (5000, 900, 32, 4.0, 260, [63, 64, 129], (32, 128, 4)), (4500, 2600, 32, 1.5, 68, [66], (32, 128, 8)), (4500, 2600, 32, 1.5, 68, [0, 67], (32, 128, 8)),
    (4097, 1500, 16, 4.0, 124, [63, 123], (16, 128, 4)), (4097, 2500, 16, 2.0, 124, [64], (16, 128, 8))])
@pytest.mark.parametrize("fmt", list(TYPES))
def test_right_hand_sides_that_are_computed_again(fmt, R, C, block, rate, batch, odd, form):
    A = csb_inputs.small_matrix(5, R, C, block, block, rate=rate).A
    X = csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)
    col = int(np.argmax(np.count_nonzero(A, axis=0)))
    X[col, odd] = -np.inf
    got, Ar, Xr = product(A, block, block, fmt, X, form=form)
    at = np.ix_(Ar[:, col] != 0, odd)
    assert np.all(got[at] == -np.sign(Ar[Ar[:, col] != 0, col])[:, None] * np.inf)
    Xr[col, odd] = 0.0
    good = np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr)
    good[at] = True
    assert np.all(good)


# Weights that are infinite or undefined, and sums beyond float32's range, reach their own rows.
@pytest.mark.parametrize("R,block,batch", [(96, 32, 64), (4100, 16, 132)])
def test_results_that_are_not_finite_stay_in_their_rows(R, block, batch):
    C = 300
    A = csb_inputs.small_matrix(5, R, C, block, 32, rate=6.0).A
    rows = [int(r) for r in np.flatnonzero(np.count_nonzero(A, axis=1) > 3)[[0, 7, -1]]]
    A[rows[0], np.flatnonzero(A[rows[0]])[1]] = np.inf
    A[rows[1], np.flatnonzero(A[rows[1]])[1]] = np.nan
    A[rows[2], A[rows[2]] != 0] = 3e38                      # (four times that and more)
    X = np.abs(csb_inputs.make_vectors(batch, C, batch).reshape(C, batch)) + 1.0
    got, Ar, Xr = product(A, block, 32, csb.VAL_BF16, X)
    assert np.all(got[[rows[0], rows[2]]] == np.inf) and np.all(np.isnan(got[rows[1]]))
    Ar[rows], got[rows] = 0.0, 0.0
    assert np.all(np.abs(got - oracle.matmat(Ar, Xr)) <= bound_of(Ar, Xr))
