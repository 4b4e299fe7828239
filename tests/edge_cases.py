"""Streams at the sizes where an execution path changes its shape of work: remainders of vectors, rows
and passes, the smallest and largest of a path's range, every alignment of the operands."""
import numpy as np

from paper_2604_17861_amd import streams as S
from helpers import Builder, np_dtype
from parity_cases import to_dtype


def values(rng, shape, code, scale=2.0):
    if code == S.I32:
        return rng.integers(-(1 << 30), 1 << 30, size=shape, dtype=np.int32)
    return to_dtype((rng.standard_normal(shape) * scale).astype(np.float32), code)


def reduction_edges(code):
    """Contiguous rows whose length and first element lie anywhere in a vector: spans of one vector, of
    exactly and just over 64, 256 and 1,024 vectors, rows fewer and more than one pass holds."""
    rng = np.random.default_rng(700 + code)
    b = Builder()
    V = 4 if code in (S.F32, S.I32) else 8
    odt = np.int32 if code == S.I32 else np.float32
    for rows, n in ((1, 1), (3, 2), (700, V - 1), (65, V), (513, V + 1), (40, 22), (129, 64 * V), (130, 64 * V + 3),
                    (9, 63 * V + 1), (17, 256 * V - 1), (6, 256 * V + 1), (67, 1023 * V), (3, 1024 * V + 5), (1, 5000 * V + 1)):
        for lead in (0, 1, V - 1):
            x = b.pool(values(rng, rows * n + lead, code))[lead:].reshape(rows, n)
            if code != S.I32 and rows > 2:
                x[1, n // 2] = to_dtype(np.array([np.nan], np.float32), code)[0]
                x[2, :] = to_dtype(np.array([-np.inf], np.float32), code)[0]
            for name in ("SUM_LAST", "MAX_LAST", "MIN_LAST"):
                b.add(name, b.pool(np.zeros(rows, odt)), [x])
    return b.stream("reduction_edges_%d" % code)


def rows_edges(code):
    """Rows contiguous in every operand under outer dims of any strides: slices read and written, head
    splits, per-row scalars of any dtype, repeated rows, unaligned bases; rows of exactly one vector, of
    one vector and a remainder, of many; fewer and more vectors than a round of the workgroup holds;
    operators by arity, copies of bits, casts.  Outputs lie inside larger buffers."""
    rng = np.random.default_rng(710 + code)
    b = Builder()
    V = 4 if code in (S.F32, S.I32) else 8
    dt = np_dtype(code)
    unary = ["COPY"] if code == S.I32 else ["COPY", "SCALE", "RELU", "EXP", "GELU_ERF", "GELU_TANH"]
    binary = ["ADD", "SUB", "MUL"] if code == S.I32 else ["ADD", "SUB", "MUL", "DIV", "SUB_EXP"]
    for i, (A, B, R, C) in enumerate(((1, 1, 1, V), (1, 1, 3, V + 1), (1, 1, 700, 2 * V - 1), (1, 1, 37, 17 * V + 3), (1, 3, 5, 9 * V),
                                      (2, 3, 70, 8 * V), (3, 2, 5, 3 * V + 2), (2, 5, 3, 300 * V + 1), (1, 1, 2, 5000 * V + 5))):
        lead = i % (V + 1)
        x = b.pool(values(rng, (A, R, B, C + 3), code))[..., :C].transpose(0, 2, 1, 3)          # a head split of a slice
        flat = b.pool(values(rng, A * B * R * C + lead, code))[lead:].reshape(A, B, R, C)
        row = np.broadcast_to(b.pool(values(rng, (B, 1, C), code)), (A, B, R, C))               # repeated over A and R
        col = np.broadcast_to(b.pool(values(rng, (A, B, R, 1), code)), (A, B, R, C))            # one scalar per row
        other = S.I32 if code == S.I32 else S.F32 if code != S.F32 else S.BF16
        col2 = np.broadcast_to(b.pool(values(rng, R + 1, other))[1:].reshape(R, 1), (A, B, R, C))

        def out(c=code):
            return b.pool(np.zeros((A, B, R, C + 2), np_dtype(c)))[..., 1:C + 1]
        for name in unary:
            b.add(name, out(), [x], alpha=0.75)
        for name in binary:
            b.add(name, out(), [x, flat])
            b.add(name, out(), [row, x])
        b.add(binary[1], out(), [flat, col])
        b.add(binary[0], out(), [col, x])
        b.add(binary[1], b.pool(np.zeros((A, B, R, C), dt)), [flat, col2])
        if code != S.I32:
            b.add("FMA", out(), [x, flat, row])
            b.add("FMA", out(), [x, col2, flat])
            for c in (S.F32, S.F16, S.BF16):
                if c != code:
                    b.add("COPY", out(c), [x])
                    b.add("COPY", b.pool(np.zeros((A, B, R, C), np_dtype(c))), [flat])
    return b.stream("rows_edges_%d" % code)
