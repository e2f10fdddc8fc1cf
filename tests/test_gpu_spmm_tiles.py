"""Parity of the batched products at the edges of their batch tiles: the forms that take 128
right-hand sides per workgroup, against the oracle's float64 product, with the float32 dot-product
bound of tests/test_gpu_spmm.py."""
import numpy as np
import pytest

import csb_inputs
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from test_gpu_spmm import check_spmm            # noqa: E402
from test_gpu_val16 import FORMATS, packed      # noqa: E402


# 256 row tiles and more: every compute unit gets a workgroup of 128 columns.  Batches one step
# below, at and above a tile; 16- and 32-row tiles; blocks of one and of several column passes.
@pytest.mark.parametrize("R,C,br,bc,batch", [(8192, 70, 32, 16, 68), (8192, 40, 32, 40, 128), (8190, 33, 32, 32, 132),
                                             (4100, 130, 16, 32, 124), (2060, 60, 16, 64, 260)])
def test_spmm_128_columns(R, C, br, bc, batch):
    m = csb_inputs.small_matrix(R + C + batch, R, C, br, bc, rate=4.0)
    check_spmm(m.A, br, bc, csb_inputs.make_vectors(batch, C, batch), tag="128-columns")


@pytest.mark.parametrize("fmt,name", FORMATS)
@pytest.mark.parametrize("R,C,br,bc,batch", [(8192, 70, 32, 16, 68), (8190, 33, 32, 32, 132), (4100, 130, 16, 32, 128)])
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
