"""The measured cases: pruned recurrent inference and the products it is made of.

A case is a dict of plain values.  `kind` picks the path:

  "rnn"      csb_rnn_forward over a sequence (batch 1: resident or streaming; batch > 1: matrix cores)
  "spmv"     csb_spmv, one right-hand side
  "spmm"     csb_spmm / csb_spmm_bfloat / csb_spmm_half, a batch of right-hand sides
  "project"  csb_project, the projection of a dense matrix onto the CSB pattern

Every matrix is drawn with the block structure the library is for: inside each block whole rows
and whole columns survive, the density of the blocks following one of three laws.
"""
import math

import numpy as np
import torch

from paper_2005_05758_amd import CsbMatrix, CsbRnn
from paper_2005_05758_amd import binding as csb

CELLS = {"lstm": csb.CELL_LSTM, "gru": csb.CELL_GRU, "lstmp": csb.CELL_LSTMP, "ligru": csb.CELL_LIGRU,
         "gru_rb": csb.CELL_GRU_RB}
GATES = {"lstm": 4, "gru": 3, "lstmp": 4, "ligru": 2, "gru_rb": 3}
FORMATS = {"f32": csb.VAL_F32, "f16": csb.VAL_F16, "bf16": csb.VAL_BF16}
SIGMA = 0.05                 # standard deviation of the weights, as the repository's workloads have it


def _rnn(name, cell, layers, inputs, hidden, block, rate, law, batch, steps, resident, proj=0, keep=False):
    return {"name": name, "kind": "rnn", "cell": cell, "layers": layers, "input": inputs, "hidden": hidden,
            "proj": proj, "block": block, "rate": rate, "law": law, "batch": batch, "steps": steps,
            "resident": resident, "keep": keep}


def _mat(name, kind, rows, cols, block, rate, law, fmt="f32", batch=1):
    return {"name": name, "kind": kind, "rows": rows, "cols": cols, "block": block, "rate": rate, "law": law,
            "format": fmt, "batch": batch}


def listed():
    return [
        # One frame at a time, as a device that answers while the speaker talks: the smallest call,
        # all launch and host path.  State and output buffers are kept by the caller.
        _rnn("frame_lstm_64x128", "lstm", 1, 64, 128, 16, 8.0, "binomial", 1, 1, True, keep=True),
        # One utterance, one layer, weights on chip: the headline workload of the benchmark.
        _rnn("seq_lstm_153x512", "lstm", 1, 153, 512, 32, 10.0, "binomial", 1, 100, True),
        # The same for a wider GRU whose blocks are unevenly filled.
        _rnn("seq_gru_256x1024", "gru", 1, 256, 1024, 32, 16.0, "beta", 1, 200, True),
        # One utterance through a two-layer LSTM with projections, weights streamed at every step.
        _rnn("stream_lstmp2_153x1024x512", "lstmp", 2, 153, 1024, 32, 13.0, "binomial", 1, 100, False, proj=512),
        # A full batch of sequences on the matrix cores.
        _rnn("batch64_lstm2_1024", "lstm", 2, 1024, 1024, 64, 25.0, "binomial", 64, 256, False),
        # A batch as it happens to fill up (odd) and a narrow, odd input.
        _rnn("batch33_ligru2_39x512", "ligru", 2, 39, 512, 32, 7.1, "binomial", 33, 100, False),
        # One matrix-vector product: the large square matrix with unevenly filled blocks.
        _mat("spmv_8192", "spmv", 8192, 8192, 32, 12.0, "heavy"),
        # A tall matrix of odd sizes (a vocabulary's output layer) with 16-bit weights.
        _mat("spmv_f16_20011x5003", "spmv", 20011, 5003, 32, 12.0, "heavy", "f16"),
        # A batch of right-hand sides: the large matrix, 128 at once.
        _mat("spmm_8192_b128", "spmm", 8192, 8192, 32, 12.0, "heavy", "f32", 128),
        # Odd sizes and an odd batch: a gate matrix applied to the frames of one utterance.
        _mat("spmm_2048x665_b99", "spmm", 2048, 665, 32, 10.0, "binomial", "f32", 99),
        # bfloat16 on both sides, a large batch.
        _mat("spmm_bf16_8192_b512", "spmm", 8192, 8192, 32, 12.0, "heavy", "bf16", 512),
        # The pruning step: a dense matrix onto the pattern.
        _mat("project_8192", "project", 8192, 8192, 32, 12.0, "dense"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rnn", "rnn", "rnn", "spmv", "spmm", "spmm", "project"])
    block, law = rng.choice([16, 32, 32, 64]), rng.choice(["binomial", "beta", "heavy"])
    if kind == "rnn":
        cell = rng.choice(["lstm", "lstm", "gru", "lstmp", "ligru", "gru_rb"])
        batch = 1 if rng.random() < 0.5 else _log(rng, 2, 64)
        hidden = _log(rng, 128, 1024)
        c = _rnn("", cell, rng.choice([1, 2]), _log(rng, 39, 1024), hidden, block, round(rng.uniform(8.0, 25.0), 1),
                 "binomial" if law == "heavy" else law, batch, _log(rng, 1, 200) if batch == 1 else _log(rng, 4, 100),
                 batch == 1 and rng.random() < 0.6, proj=(hidden + 1) // 2 if cell == "lstmp" else 0)
    elif kind == "project":
        c = _mat("", kind, _log(rng, 512, 8192), _log(rng, 192, 8192), block, round(rng.uniform(4.0, 25.0), 1), "dense")
    else:
        fmt = rng.choice(["f32", "f32", "f16", "bf16"])
        rows, cols = _log(rng, 512, 16384), _log(rng, 192, 8192)
        batch = 1
        if kind == "spmm":                                  # 16-bit right-hand sides come in fours
            batch = _log(rng, 4, 512) if fmt == "f32" else 4 * _log(rng, 2, 128)
            rows = min(rows, 8192)
        c = _mat("", kind, rows, cols, block, round(rng.uniform(8.0, 25.0), 1), law, fmt, batch)
    del c["name"]
    return c


def _density(g, rate, law, nb):
    """Density of each of nb blocks, 1 / rate on average."""
    if law == "beta":
        u = g.beta(2.0, 5.0, size=nb)
        return np.minimum(u / (u.mean() * rate), 1.0)
    if law == "heavy":                                       # a tenth of the blocks much fuller than the rest
        light = 0.6 / rate
        heavy = min((1.0 / rate - 0.9 * light) / 0.1, 1.0)
        return np.where(g.random(nb) < 0.1, heavy, light)
    return np.full(nb, 1.0 / rate)


def _pruned(seed, rows, cols, block, rate, law):
    """A pruned weight matrix on the host: N(0, SIGMA) where a block keeps both row and column."""
    g = np.random.Generator(np.random.PCG64(seed))
    t = torch.Generator(device="cuda").manual_seed(seed)
    nbr, nbc = -(-rows // block), -(-cols // block)
    keep = torch.from_numpy(np.sqrt(_density(g, rate, law, nbr * nbc))).float().cuda().view(nbr, nbc, 1)
    r = torch.rand((nbr, nbc, block), generator=t, device="cuda") < keep
    c = torch.rand((nbr, nbc, block), generator=t, device="cuda") < keep
    mask = (r.permute(0, 2, 1).unsqueeze(3) & c.unsqueeze(1)).reshape(nbr * block, nbc * block)[:rows, :cols]
    w = torch.randn((rows, cols), generator=t, device="cuda") * SIGMA
    return (w * mask).cpu().numpy()


def _matrix(seed, case, rows, cols, dense=None):
    if dense is None:
        dense = _pruned(seed, rows, cols, case["block"], case["rate"], case["law"])
    return CsbMatrix(dense, case["block"], case["block"])


def _widths(case):
    """(width of the recurrent state, [inputs of layer 0, 1, ...])"""
    state = case["proj"] or case["hidden"]
    return state, [case["input"]] + [state] * (case["layers"] - 1)


def prepare(case, seed):
    t = torch.Generator(device="cuda").manual_seed(seed + 7919)

    def uniform(*shape):
        return torch.rand(shape, generator=t, device="cuda") * 2.0 - 1.0

    if case["kind"] == "project":
        W = torch.randn((case["rows"], case["cols"]), generator=t, device="cuda") * SIGMA
        return {"case": case, "W": W, "Z": torch.empty_like(W)}
    if case["kind"] != "rnn":
        M = _matrix(seed, case, case["rows"], case["cols"])
        if case["format"] != "f32":
            M.set_value_format(FORMATS[case["format"]])
        M.plan()
        M.upload()
        if case["kind"] == "spmv":
            return {"case": case, "M": M, "x": uniform(case["cols"]), "y": torch.empty(case["rows"], device="cuda")}
        X = uniform(case["cols"], case["batch"])
        X = X.to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[case["format"]])
        return {"case": case, "M": M, "x": X, "y": torch.empty((case["rows"], case["batch"]), device="cuda")}

    cell, H, G = case["cell"], case["hidden"], GATES[case["cell"]]
    S, ins = _widths(case)
    W, second = [], []
    for l, n_in in enumerate(ins):
        dense = _pruned(seed + 101 * l, G * H, n_in + S, case["block"], case["rate"], case["law"])
        if cell == "gru_rb":                                 # the candidate's recurrent side is a matrix of its own
            second.append(_matrix(0, case, H, H, np.ascontiguousarray(dense[2 * H:, n_in:])))
            dense[2 * H:, n_in:] = 0.0
        W.append(_matrix(0, case, G * H, n_in + S, dense))
        if cell == "lstmp":
            second.append(_matrix(seed + 101 * l + 50, case, S, H))
    bias = [torch.randn(G * H, generator=t, device="cuda") * SIGMA for _ in ins]
    rnn = CsbRnn(CELLS[cell], case["input"], H, W, bias, proj=case["proj"], Wp=second or None)
    if case["resident"] and rnn.device_bytes() > 0:
        rnn.upload()
    else:
        for m in W + second:
            m.upload()
    T, B, L = case["steps"], case["batch"], case["layers"]
    st = {"case": case, "rnn": rnn, "x": uniform(T, B, case["input"]), "h0": 0.5 * uniform(L, B, S),
          "c0": 0.5 * uniform(L, B, H) if cell in ("lstm", "lstmp") else None}
    if case["keep"]:
        st["out"] = (torch.empty((T, B, S), device="cuda"), torch.empty((L, B, S), device="cuda"),
                     torch.empty((L, B, H), device="cuda") if st["c0"] is not None else None)
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "rnn":
        if case["keep"]:
            st["rnn"].forward_into(st["x"], st["h0"], st["c0"], *st["out"])
            out = st["out"]
        else:
            out = st["rnn"].forward(st["x"], st["h0"], st["c0"])
        return [o for o in out if o is not None]
    if case["kind"] == "project":
        return csb.project(st["W"], case["block"], case["block"], case["rate"], out=st["Z"])
    if case["kind"] == "spmv":
        return st["M"].spmv(st["x"], st["y"])
    call = {"f32": st["M"].spmm, "f16": st["M"].spmm_half, "bf16": st["M"].spmm_bfloat}[case["format"]]
    return call(st["x"], st["y"])


def _stored(rows, cols, block, rate, size):
    """Bytes of a pruned matrix: its values, a byte for each kept row and column of a block, two counts a block."""
    blocks = -(-rows // block) * -(-cols // block)
    return rows * cols / rate * size + blocks * (2.0 * block * rate ** -0.5 + 2.0)


def work(case):
    if case["kind"] == "project":
        return {"bytes": 8.0 * case["rows"] * case["cols"], "flops": 4.0 * case["rows"] * case["cols"]}
    if case["kind"] != "rnn":
        rows, cols, batch, size = case["rows"], case["cols"], case["batch"], 4 if case["format"] == "f32" else 2
        x_size = size if case["kind"] == "spmm" else 4
        return {"bytes": _stored(rows, cols, case["block"], case["rate"], size) + batch * (cols * x_size + rows * 4.0),
                "flops": 2.0 * rows * cols / case["rate"] * batch}
    H, G = case["hidden"], GATES[case["cell"]]
    S, ins = _widths(case)
    entries = bytes_ = 0.0
    for n_in in ins:
        shapes = [(G * H, n_in + S)] + ([(S, H)] if case["cell"] == "lstmp" else [])
        entries += sum(r * c / case["rate"] for r, c in shapes)
        bytes_ += sum(_stored(r, c, case["block"], case["rate"], 4) for r, c in shapes) + 4.0 * G * H
    T, B = case["steps"], case["batch"]
    states = 2.0 * case["layers"] * B * (S + (H if case["cell"] in ("lstm", "lstmp") else 0))
    return {"bytes": bytes_ + 4.0 * (T * B * (case["input"] + S) + states),
            "flops": T * B * (2.0 * entries + 10.0 * H * case["layers"])}


def tolerance(case):
    """All sums are float32 (16-bit weights and inputs have exact float32 products).  Against the
    same path in float64, over the listed cases and drawn ones: products 0.6e-7 to 1.5e-7 (largest
    element 1.1e-6), sequences 0.6e-7 to 4.2e-7 (largest element 4.3e-6); four times the largest."""
    if case["kind"] == "project":
        return "exact"
    if case["kind"] == "rnn":
        return {"rel": 1.7e-6, "max": 1.7e-5}
    return {"rel": 6e-7, "max": 4.5e-6}
