"""The work that a user of this framework has it do, as cases that can be timed.

A case is one layer with a block-sparse weight W (n, k), stored in blocks of bs_r x bs_c, and m rows of input:

  pass "forward"   Y = X * W^T                                     (`bsr_spmm` on the handle of W)
  pass "backward"  what the layer's backward step needs: the stored values of W^T brought up to date (an optimizer
                   step has changed W), Z = G * W (`bsr_spmm` on the handle of W^T), and the gradient of the stored
                   blocks D (`bsr_sddmm`)

with `dtype` the type of X, G and W, `out` the type of the result, `pattern` "uniform" (exactly round(density * blocks)
stored blocks, anywhere) or "power" (blocks per block-row by a rank power law with exponent 1.2), and `keep` whether the
caller passes an output buffer that it keeps (a serving loop) or lets the call return a new one.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2007_13055_amd as lib
from paper_2007_13055_amd.binding import BSR_BF16, BSR_F16, BSR_F32

_SIZE = {"f32": 4, "f16": 2, "bf16": 2}
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_CODE = {"f32": BSR_F32, "f16": BSR_F16, "bf16": BSR_BF16}


def _case(name, kind, m, k, n, bs_r, bs_c, dtype, density, pattern="uniform", out=None, keep=False):
    c = {"pass": kind, "m": m, "k": k, "n": n, "bs_r": bs_r, "bs_c": bs_c, "dtype": dtype, "out": out or dtype,
         "density": density, "pattern": pattern, "keep": keep}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one request through a small fp32 layer, buffers kept: latency of a single call (the paper's grid, m = 1)
        _case("one row", "forward", 1, 1024, 1024, 16, 16, "f32", 0.15, keep=True),
        # a handful of rows in a new buffer, small blocks (the paper's grid, m = 8)
        _case("eight rows", "forward", 8, 1024, 1024, 8, 8, "f32", 0.20),
        # a small layer at batch 128: launch cost and little else
        _case("tiny", "forward", 128, 256, 256, 16, 16, "f32", 0.25),
        # the feed-forward weight of a transformer at an inference batch, and the same layer's backward step
        _case("ffn", "forward", 128, 3072, 3072, 32, 32, "f32", 0.10),
        _case("ffn backward", "backward", 128, 3072, 3072, 32, 32, "f32", 0.10),
        # an odd number of rows of 16-bit activations, result handed on in fp32
        _case("ragged", "forward", 1003, 1504, 2080, 32, 32, "f16", 0.15, out="f32"),
        # a training batch of bf16 activations against 16x16 blocks, forward and backward
        _case("batched", "forward", 4096, 768, 3072, 16, 16, "bf16", 0.20),
        _case("batched backward", "backward", 4096, 768, 3072, 16, 16, "bf16", 0.20),
        # blocks of one column (fp32), forward and backward
        _case("thin", "forward", 256, 4096, 4096, 16, 1, "f32", 0.05),
        _case("thin backward", "backward", 256, 4096, 4096, 16, 1, "f32", 0.05),
        # the largest: 64x64 fp16 blocks, a few block-rows hold most of W; forward and backward
        _case("skewed", "forward", 8192, 8192, 8192, 64, 64, "f16", 0.05, pattern="power"),
        _case("skewed backward", "backward", 8192, 8192, 8192, 64, 64, "f16", 0.05, pattern="power"),
    ]


def _cost(c):
    """Seconds, roughly, of a case on one GPU: what a drawn case is held to."""
    w = work(c)
    return w["bytes"] / 4e12 + w["flops"] / (3e13 if c["dtype"] == "f32" else 4e14)


def draw(rng):
    """A case of the same ranges: m 1..8192, k and n 128..8192, blocks 8x8 to 64x64 and 16x1, densities 0.03..0.3."""
    most = _cost(listed()[-1])

    def log_between(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    while True:
        bs_r, bs_c = rng.choice([(8, 8), (16, 16), (16, 16), (32, 32), (32, 32), (64, 64), (64, 64), (16, 1)])
        dtype = "f32" if bs_c == 1 else rng.choice(["f32", "f16", "bf16"])
        # most layers' widths are multiples of 64, some only of the block
        unit = 64 if rng.random() < 0.7 else bs_r

        def width():
            return max(2, round(log_between(128, 8192) / unit)) * unit

        kind = rng.choice(["forward", "forward", "backward"])
        out = "f32" if dtype != "f32" and kind == "forward" and rng.random() < 0.25 else dtype
        pattern = "power" if bs_c > 1 and rng.random() < 0.25 else "uniform"
        c = _case(None, kind, round(log_between(1, 8192)), width(), width(), bs_r, bs_c, dtype,
                  round(log_between(0.03, 0.3), 3), pattern, out, rng.random() < 0.3)
        if _cost(c) <= most:
            return c


def _stored(c):
    return max(1, round(c["density"] * (c["n"] // c["bs_r"]) * (c["k"] // c["bs_c"])))


def _pattern(c, rng):
    """index_pointer and block_indices, sorted within a block-row."""
    R, C, total = c["n"] // c["bs_r"], c["k"] // c["bs_c"], _stored(c)
    if c["pattern"] == "uniform":
        at = np.sort(rng.choice(R * C, size=total, replace=False, shuffle=False))
        counts = np.bincount(at // C, minlength=R)
        idx = (at % C).astype(np.int32)
    else:
        share, rest = np.arange(1, R + 1, dtype=np.float64) ** -1.2, np.ones(R, dtype=bool)
        counts = np.zeros(R)
        while True:                                        # rows at their limit hand the rest on to the others
            counts[rest] = (total - C * (~rest).sum()) * share[rest] / share[rest].sum()
            over = rest & (counts > C)
            if not over.any():
                break
            counts[over] = C
            rest &= ~over
        left = counts - np.floor(counts)
        counts = np.floor(counts).astype(np.int64)
        counts[np.argsort(-left, kind="stable")[: total - counts.sum()]] += 1
        counts = counts[rng.permutation(R)]
        idx = np.concatenate([np.sort(rng.permutation(C)[:v]) for v in counts]).astype(np.int32)
    ptr = np.zeros(R + 1, dtype=np.int32)
    np.cumsum(counts, out=ptr[1:])
    return ptr, idx


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * scale).to(_TORCH[c["dtype"]])

    ptr, idx = _pattern(c, np.random.default_rng(seed))
    data = normal(_stored(c), c["bs_r"], c["bs_c"], scale=0.02)
    s = {"pass": c["pass"], "out": c["out"], "X": normal(c["m"], c["k"]), "Y": None, "Z": None, "D": None}
    s["W"] = lib.bsr_create(c["n"], c["k"], data, idx, ptr)
    if c["pass"] == "forward":
        if c["keep"]:
            s["Y"] = torch.empty((c["m"], c["n"]), dtype=_TORCH[c["out"]], device="cuda")
    else:
        s["G"] = normal(c["m"], c["n"])
        s["WT"] = lib.bsr_create_transposed(c["n"], c["k"], data, idx, ptr)
        perm = lib.bsr_transpose_pattern(c["n"], c["k"], c["bs_r"], c["bs_c"], ptr, idx)[2]
        s["perm"] = torch.from_numpy(perm).cuda()
        s["blocks"] = (_CODE[c["dtype"]], c["bs_r"], c["bs_c"], _stored(c))
        if c["keep"]:
            s["Z"] = torch.empty((c["m"], c["k"]), dtype=_TORCH[c["out"]], device="cuda")
            s["D"] = torch.empty((_stored(c), c["bs_r"], c["bs_c"]), dtype=_TORCH[c["out"]], device="cuda")
    return s


def run(state):
    s = state
    if s["pass"] == "forward":
        return lib.bsr_spmm(s["W"], s["X"], s["Y"], y_dtype=s["out"])
    st = lib.load_library().bsr_transpose_values(*s["blocks"], s["perm"].data_ptr(), s["W"].block_data.data_ptr(),
                                                 s["WT"].block_data.data_ptr(), torch.cuda.current_stream().cuda_stream)
    if st != 0:
        raise lib.BsrError(st, "bsr_transpose_values")
    return {"Z": lib.bsr_spmm(s["WT"], s["G"], s["Z"], y_dtype=s["out"]),
            "D": lib.bsr_sddmm(s["W"], s["G"], s["X"], s["D"], d_dtype=s["out"]),
            "WT": s["WT"].block_data}


def work(case):
    """The referenced parts of the operands, the stored blocks and the index arrays read once, the results written once."""
    c = case
    s_in, s_out, nnzb = _SIZE[c["dtype"]], _SIZE[c["out"]], _stored(c)
    R, C, block = c["n"] // c["bs_r"], c["k"] // c["bs_c"], c["bs_r"] * c["bs_c"]
    used_cols = C * (1.0 - (1.0 - nnzb / (R * C)) ** R)          # block-columns that hold a block, expected
    x_bytes = c["m"] * used_cols * c["bs_c"] * s_in
    w_bytes, i_bytes, flops = nnzb * block * s_in, 4 * (nnzb + R + 1), 2 * c["m"] * nnzb * block
    if c["pass"] == "forward":
        return {"bytes": x_bytes + w_bytes + i_bytes + c["m"] * c["n"] * s_out, "flops": flops}
    # G and X and W's values once, W^T's values, Z and D written
    return {"bytes": x_bytes + c["m"] * c["n"] * s_in + 2 * w_bytes + 2 * i_bytes + c["m"] * c["k"] * s_out
            + nnzb * block * s_out, "flops": 2 * flops}


def tolerance(case):
    """Sums are in fp32 in any order; a 16-bit result is rounded once."""
    return {"rel": {"f32": 1e-5, "f16": 2e-3, "bf16": 1e-2}[case["out"]]}
