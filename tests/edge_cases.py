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
