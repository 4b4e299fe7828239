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


def reduction_shares(code):
    """Contiguous rows that wavefronts share out and read densely: row lengths at either side of each shape of
    work (rows put into LDS by the piece, one piece a row and many; rows that end within a group of 64
    vectors, at its end, several in one; more than 64 rows a wavefront), rows that no piece or share
    divides, a NaN in a row's first or last element, between rows that have none."""
    rng = np.random.default_rng(720 + code)
    b = Builder()
    V = 4 if code in (S.F32, S.I32) else 8
    odt = np.int32 if code == S.I32 else np.float32
    for rows, n, lead in ((1030, 3, 1), (411, 2 * V + 1, 0), (197, 14 * V - 1, 2), (77, 126 * V + 2, 0), (78, 127 * V - 1, 1), (79, 127 * V, 1),
                          (45, 127 * V + 1, 0), (46, 128 * V, 0), (47, 65 * V, 0), (13, 223 * V + 1, 1), (9, 447 * V + 1, 0), (9, 448 * V, 0),
                          (300, 64 * V, 0), (260, 63 * V, 0), (50, 34 * V, 0), (90, V, 0), (21, 1022 * V, 0), (9000, 65 * V, 0)):
        x = b.pool(values(rng, rows * n + lead, code))[lead:].reshape(rows, n)
        if code != S.I32:
            nan = to_dtype(np.array([np.nan], np.float32), code)[0]
            x[1::7, -1] = nan
            x[3::7, 0] = nan
        for name in ("SUM_LAST", "MAX_LAST", "MIN_LAST"):
            b.add(name, b.pool(np.zeros(rows, odt)), [x])
    return b.stream("reduction_shares_%d" % code)


def reduction_long_rows(code):
    """Contiguous rows that wavefronts take a quarter each of, the next vectors or the next row's first on their way: quarters of
    one group of 4 x 64 vectors and of many, of whole groups and not, the last one shorter; one row, a few, with and
    without a lead; inputs on both sides of 4 MB, from which on they are read past the memory-side cache."""
    rng = np.random.default_rng(725 + code)
    b = Builder()
    V = 4 if code in (S.F32, S.I32) else 8
    odt = np.int32 if code == S.I32 else np.float32
    for rows, n, lead in ((1, 1024 * V, 0), (5, 1024 * V, 0), (3, 1024 * V + 1, 1), (4, 1025 * V - 1, 2), (2, 2047 * V + 1, 0), (7, 2048 * V, 0),
                          (3, 4096 * V, 0), (2, 4099 * V + 3, 1), (70, 1030 * V + 2, 0), (260, 1026 * V, 0), (29, 10000 * V + 1, 0)):
        x = b.pool(values(rng, rows * n + lead, code))[lead:].reshape(rows, n)
        if code != S.I32:
            nan = to_dtype(np.array([np.nan], np.float32), code)[0]
            x[1::7, -1] = nan
            x[3::7, 0] = nan
        for name in ("SUM_LAST", "MAX_LAST", "MIN_LAST"):
            b.add(name, b.pool(np.zeros(rows, odt)), [x])
    return b.stream("reduction_long_rows_%d" % code)


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


def row_operation_edges(code):
    """Softmax, masked softmax and layer norm over rows of any length and alignment: a vector and less,
    a vector and one element, the lengths where a row moves from lane groups to a wavefront, to the
    workgroup's registers and beyond them, remainders of one and of all but one element; masks
    repeated every few rows; fp32 parameters under 16-bit rows; NaN, infinities and rows of -inf."""
    rng = np.random.default_rng(720 + code)
    b = Builder()
    V = 4 if code == S.F32 else 8
    dt = np_dtype(code)
    for i, (rows, n) in enumerate(((5, V - 1), (3, V), (70, V + 1), (300, 3 * V - 1), (131, 32 * V + 1), (130, 64 * V - 1), (65, 64 * V + 1),
                                   (19, 128 * V - 3), (17, 128 * V + 1), (9, 256 * V - 1), (9, 256 * V + 1), (5, 512 * V + 3), (3, 1024 * V - 1),
                                   (3, 1024 * V + 1), (3, 2048 * V - 1), (2, 2048 * V + 1), (3, 4096 * V + V + 1), (2, 5632 * V + 1), (2, 65535), (2, 65536))):
        lead = (0, 1, V - 1)[i % 3]
        x = b.pool(values(rng, rows * n + lead, code, 3.0))[lead:].reshape(rows, n)

        def out():
            return b.pool(np.zeros(rows * n + 1, dt))[i % 2:][:rows * n].reshape(rows, n)
        b.add("SOFTMAX_LAST", out(), [x])
        mrow = b.pool(values(rng, n, code))
        b.add("MASKED_SOFTMAX_LAST", out(), [x, np.broadcast_to(mrow, (rows, n))], alpha=0.3)
        if rows % 5 == 0:                                    # a mask of `per` rows, repeated
            per = rows // 5
            m = b.pool(values(rng, per * n + 1, code))[1:].reshape(per, n)
            o = out().reshape(5, per, n)
            b.add("MASKED_SOFTMAX_LAST", o, [x.reshape(5, per, n), np.broadcast_to(m, (5, per, n))], alpha=0.5)
        for pcode in ((code,) if code == S.F32 else (code, S.F32)):
            g, be = b.pool(to_dtype(1 + 0.2 * rng.standard_normal(n + 1), pcode))[1:], b.pool(values(rng, n, pcode))
            b.add("LAYERNORM_LAST", out(), [x, np.broadcast_to(g, (rows, n)), np.broadcast_to(be, (rows, n))], alpha=1e-5)
        if rows >= 3 and code != S.BF16:
            y = b.pool(np.ascontiguousarray(x[:3]))
            y[0, n // 2] = np.nan
            y[1, :] = -np.inf
            y[2, ::2] = -np.inf
            b.add("SOFTMAX_LAST", b.pool(np.zeros((3, n), dt)), [y])
    return b.stream("row_operation_edges_%d" % code)


def every_second_element(code):
    """Slices with a step of two, from the buffer's first element and from its second, that end with the buffer's last
    element: fewer and more than a vector, than a round of the workgroup and than a chunk; alone, with contiguous
    operands of any alignment and with each other; slices of matrices whose rows merge; every operator class."""
    rng = np.random.default_rng(740 + code)
    b = Builder()
    V = 4 if code == S.F32 else 8
    dt = np_dtype(code)
    for i, n in enumerate((1, 2, V - 1, V, V + 1, 2 * V, 255 * V + 3, 1024, 1025, 2047, 4096, 8192, 8193, 16384, 40000 + V, 1 << 20, (1 << 20) + 2049, (1 << 21) + 5)):
        first = i % 2

        def second(k=first):
            return b.pool(values(rng, 2 * n - 1 + k, code))[k::2]
        lead = (0, 1, 3)[i % 3]
        flat = b.pool(values(rng, n + lead, code))[lead:]

        def out():
            return b.pool(np.zeros(n + V, dt))[:n]
        for name in ("SCALE", "RELU", "EXP", "GELU_ERF", "GELU_TANH")[i % 5:][:2]:
            b.add(name, out(), [second()], alpha=0.75)
        b.add(("ADD", "SUB", "MUL", "SUB_EXP", "DIV")[i % 5], out(), [second(), flat])
        b.add(("SUB", "MUL", "DIV", "ADD")[i % 4], out(), [flat, second(1 - first)])
        b.add("MUL", out(), [second(), second(1 - first)])
        b.add("FMA", out(), [second(), flat, second()])
    m = b.pool(values(rng, 30 * 58, code)).reshape(30, 58)                                    # x[:, ::2] * y, merged to one dim
    b.add("MUL", b.pool(np.zeros((30, 29), dt)), [m[:, ::2], b.pool(values(rng, 30 * 29, code)).reshape(30, 29)])
    return b.stream("every_second_element_%d" % code)


def long_softmax_rows(code):
    """Softmax rows of which a workgroup keeps a part in registers and in LDS: either side of every length at
    which it keeps more, fits no more or reads another batch again, at every alignment of rows cut at blocks of memory (x
    and the result at one offset) and at none; infinities at a row's ends."""
    rng = np.random.default_rng(730 + code)
    b = Builder()
    V = 4 if code == S.F32 else 8
    dt = np_dtype(code)
    lengths = [16 * 256, 21 * 256, 22 * 256, 24 * 256, 27 * 256] if code == S.F32 else [8 * 256, 12 * 256, 14 * 256, 15 * 256, 21 * 256, 24 * 256]
    for i, (vectors, more) in enumerate((v, m) for v in lengths for m in (-1, 0, 1, 2 * V + 3)):
        n = vectors * V + more
        if n <= 16384:
            continue
        x_at, o_at = ((0, 0), (1, 1), (V - 1, V - 1), (0, 1))[i % 4]
        x = b.pool(values(rng, 3 * n + x_at, code, 3.0))[x_at:].reshape(3, n)
        if code != S.BF16:
            x[1, 0] = x[1, -1] = -np.inf
            x[2, : n // 2] = -np.inf
        b.add("SOFTMAX_LAST", b.pool(np.zeros(3 * n + o_at, dt))[o_at:].reshape(3, n), [x])
    return b.stream("long_softmax_rows_%d" % code)


def long_softmax_rows_whole_and_not(code):
    """The same lengths, each with less, as many and more elements than its whole vectors hold, each at every alignment: rows of
    whole aligned vectors among them at every length, with as many and with one vector more."""
    rng = np.random.default_rng(760 + code)
    b = Builder()
    V = 4 if code == S.F32 else 8
    dt = np_dtype(code)
    lengths = [16 * 256, 21 * 256, 22 * 256, 24 * 256, 27 * 256] if code == S.F32 else [8 * 256, 12 * 256, 14 * 256, 15 * 256, 21 * 256, 24 * 256]
    for vectors in lengths:
        for more in (-1, 0, 1, V, 2 * V + 3):
            for x_at, o_at in ((0, 0), (1, 1), (V - 1, V - 1), (0, 1)):
                n = vectors * V + more
                if n <= 16384:
                    continue
                x = b.pool(values(rng, 2 * n + x_at, code, 3.0))[x_at:].reshape(2, n)
                if code != S.BF16:
                    x[0, 0] = x[0, -1] = -np.inf
                    x[1, : n // 2] = -np.inf
                b.add("SOFTMAX_LAST", b.pool(np.zeros(2 * n + o_at, dt))[o_at:].reshape(2, n), [x])
    return b.stream("long_softmax_rows_whole_and_not_%d" % code)


def past_the_cache(code):
    """Tasks on both sides of the 16 MB of inputs from which on they are read past the memory-side cache: reductions of short rows,
    whole aligned vectors and not, and operators of some instructions over contiguous tensors, whose last vector is not whole."""
    rng = np.random.default_rng(770 + code)
    b = Builder()
    es = 4 if code in (S.F32, S.I32) else 2
    V = 16 // es
    for size in (15 << 20, 17 << 20):
        x = b.pool(values(rng, size // es + (1 << 12), code))
        for n, lead in ((3 * V, 0), (64 * V, 0), (25 * V + 1, 0), (127 * V, 1)):
            rows = size // es // n + 1
            for name in ("SUM_LAST", "MAX_LAST", "MIN_LAST")[: 2 if n == 3 * V else 1]:
                b.add(name, b.pool(np.zeros(rows, np.int32 if code == S.I32 else np.float32)), [x[lead: lead + rows * n].reshape(rows, n)])
        if code != S.I32:
            one, half = size // es + 3, size // es // 2 + 5
            b.add("EXP", b.pool(np.zeros(one, x.dtype)), [x[:one]])
            for name in ("DIV", "SUB_EXP"):
                b.add(name, b.pool(np.zeros(half, x.dtype)), [x[:half], x[8 * V: 8 * V + half]])
    return b.stream("past_the_cache_%d" % code)


def large_gathers():
    """Gathered tasks of more elements than 1,024 of the gather path's regular chunks hold: a product
    with every other column of a matrix, and a stride-2 slice of 16-bit elements.  (A chunk never run
    leaves zeros.  Not in place: the comparison takes its inputs from what the GPU left.)"""
    rng = np.random.default_rng(730)
    b = Builder()
    R, C = 3000, 3072
    x = b.pool(rng.standard_normal((R, 2 * C), dtype=np.float32))
    y = b.pool(rng.standard_normal((R, C), dtype=np.float32))
    b.add("MUL", b.pool(np.zeros((R, C), np.float32)), [x[:, ::2], y])
    n = (8 << 20) + 5003
    h = b.pool(rng.integers(0, 0x7f00, size=2 * n, dtype=np.uint16))
    b.add("SCALE", b.pool(np.zeros(n, np.uint16)), [h[1::2]], alpha=0.5)
    return b.stream("large_gathers")


def gelu_values(code):
    """Both GELUs over every value of a 16-bit format, or over fp32 values of both signs from 2^-20 to 16
    and the special ones: once contiguous and aligned, once as rows of an odd length."""
    rng = np.random.default_rng(740)
    b = Builder()
    if code == S.F32:
        v = np.ldexp(rng.uniform(0.5, 1.0, 1 << 19), rng.integers(-20, 5, 1 << 19)).astype(np.float32)
        v = np.concatenate([v, -v, np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 3e38, -3e38, 1e-42, -1e-42, 14.3, -14.3, -14.5, -14.6], np.float32)])
    else:
        v = np.arange(65536, dtype=np.uint16).view(np_dtype(code))
    x, y = b.pool(v), b.pool(np.append(v[:1], v[:v.size // 7 * 7]))[1:].reshape(7, -1)
    for name in ("GELU_ERF", "GELU_TANH"):
        b.add(name, b.pool(np.zeros_like(v)), [x])
        b.add(name, b.pool(np.zeros((7, y.shape[1] + 1), v.dtype))[:, 1:], [y])
    return b.stream("gelu_values_%d" % code)


def chains(code, seed):
    """Chains of dependent elementwise tasks over flat buffers of one length (each names the task right
    before it), at lengths round the vector, the chunk and the block of a run, with what ends a run or keeps
    a task out of one: operands that overlap another one in part, other lengths, an operator of another
    kind, a further dependency, a task outside that names a task in the middle.  Exactly rounded
    operations: the buffers at the end are those of sequential execution, byte for byte."""
    rng = np.random.default_rng(1000 * code + seed)
    b = Builder()
    es = 4 if code == S.F32 else 2
    V = 16 // es
    lengths = [1, V - 1, V, 255 * V + 1, 1024, 4096, 4096 + V + 3, 6144, 12288 + 5, 16384, 50001]
    for n in lengths:
        pad = (n + 64) // 64 * 64
        live = b.pool(to_dtype(rng.integers(-3, 4, 6 * pad).astype(np.float32), code))
        const = b.pool(to_dtype(rng.integers(-1, 2, 2 * pad).astype(np.float32), code))
        side = b.pool(to_dtype(np.zeros(4 * pad, np.float32), code))
        at = lambda k: live[k * pad: k * pad + n]
        cur, n_side = 0, 0
        for t in range(70):
            dep = (1, 0, 0) if t else (0, 0, 0)
            x, o = at(cur), int(rng.integers(4))
            kind, other = rng.random(), int(rng.integers(4))
            if kind < 0.13 and o in (cur, other):            # (a task's own operands are the same elements or none in common)
                kind = 1.0
            out = at(o)
            if kind < 0.06:                                  # written one vector further on: overlaps what the run has touched
                out = live[o * pad + V: o * pad + V + n]
                nxt = None
            elif kind < 0.10 and n > 2 * V:                  # a shorter task in the chain
                x, out, nxt = x[: n - V], out[: n - V], o
            elif kind < 0.13:                                # misaligned by an element
                out = live[o * pad + 1: o * pad + 1 + n]
                nxt = None
            else:
                nxt = o
            op = str(rng.choice(["ADD", "SUB", "RELU", "SCALE", "COPY", "MUL", "ADD", "FMA"]))
            c = const[pad * int(rng.integers(2)):][: x.size]
            if op in ("ADD", "SUB", "MUL"):
                if op == "ADD" and rng.random() < 0.2:
                    c = at(other)[: x.size]                  # a second live buffer (or the same one)
                ins = [x, c] if rng.random() < 0.7 else [c, x]
            elif op == "FMA":
                ins = [x, const[:x.size], c]
            else:
                ins = [x]
            if t > 5 and rng.random() < 0.08:
                dep = (1, int(rng.integers(2, 6)), 0)
            b.add(op, out, ins, alpha=0.5 if op == "SCALE" else 0.0, dep=dep)
            if t > 3 and n_side < 4 and rng.random() < 0.05 and nxt is not None:
                # a reader outside the chain, of a task in the middle of a run
                b.add("COPY", side[n_side * pad: n_side * pad + n], [at(nxt)], dep=(1, 0, 0))
                n_side += 1
            cur = nxt if nxt is not None else o
    return b.stream("chains_%d_%d" % (code, seed), batch=128)


def long_chains(code, n, links=150):
    """One chain after the other as a program issues them: x op c into two buffers in turn."""
    rng = np.random.default_rng(n)
    b = Builder()
    pad = (n + 64) // 64 * 64
    for _ in range(4):
        x = b.pool(to_dtype(rng.uniform(-1, 1, n).astype(np.float32), code))
        c = b.pool(to_dtype(rng.uniform(-1, 1, n).astype(np.float32), code))
        t = b.pool(to_dtype(np.zeros(2 * pad, np.float32), code))
        cur = x
        for k in range(links):
            op = ("ADD", "MUL", "RELU", "SCALE", "SUB", "DIV", "COPY")[k % 7]
            out = t[(k & 1) * pad:][:n]
            b.add(op, out, [cur, c] if op in ("ADD", "MUL", "SUB", "DIV") else [cur], alpha=0.99, dep=(1, 0, 0) if k else (0, 0, 0))
            cur = out
    return b.stream("long_chains_%d_%d" % (code, n), batch=128)


def row_chains(code, seed, shapes=None):
    """Chains over rows (scale, mask, maximum, difference, sum, quotient and variations), at row lengths of one vector
    to 65 and a ragged one, masks repeated over leading dims, results of reductions used at once, again
    later, overwritten, stored in 16 bits, or scalars that lay in memory before.  Values are small integers until the
    last step, so that sums are exact in any order."""
    rng = np.random.default_rng(2000 * code + seed)
    b = Builder()
    V = 4 if code == S.F32 else 8
    for n, B, R in shapes or ((V, 3, 5), (2 * V, 2, 64), (3 * V, 1, 130), (8 * V, 5, 33), (13 * V, 2, 40), (32 * V, 4, 32), (33 * V, 1, 9), (64 * V, 2, 17),
                              (65 * V, 2, 9), (5 * V + 1, 2, 11), (8 * V, 8, 1024)):
        size = (B, R, n)
        pool = lambda hi: b.pool(to_dtype(rng.integers(-hi, hi + 1, size).astype(np.float32), code))
        x, t1, t2, e, y = pool(8), pool(1), pool(1), pool(1), pool(1)
        mask = np.broadcast_to(b.pool(to_dtype(rng.integers(-4, 1, (R, n)).astype(np.float32), code)), size)
        vec = np.broadcast_to(b.pool(to_dtype(rng.integers(1, 5, (n,)).astype(np.float32), code)), size)
        rc = int(rng.choice([S.F32, code]))
        scal = lambda c: b.pool(to_dtype(rng.integers(-2, 3, (B, R)).astype(np.float32), c))
        m, l, k = scal(rc), scal(S.F32), scal(S.F32)
        rows = lambda s: np.broadcast_to(s[..., None], size)
        D = dict(dep=(1, 0, 0))
        b.add("SCALE", t1, [x], alpha=2.0)
        b.add("ADD", t2, [t1, mask] if rng.random() < 0.5 else [mask, t1], **D)
        b.add("MAX_LAST", m, [t2], **D)
        b.add("SUB", e, [t2, rows(m)], **D)
        b.add("RELU", t1, [e], **D)
        what = seed % 6
        if what == 1:                                        # a row vector in place of the mask, in place
            b.add("ADD", e, [e, vec], **D)
        elif what == 2:                                      # a scalar per row that no task of the chain wrote
            b.add("MUL", e, [e, rows(k)], **D)
        elif what == 3:                                      # the maximum again, behind another reduction
            b.add("MIN_LAST", l, [e], **D)
            b.add("ADD", e, [e, rows(l)], **D)
            b.add("SUB", e, [e, rows(m)], **D)
        elif what == 4:                                      # written over by the next reduction
            b.add("MIN_LAST", m, [t1], **D)
            b.add("SUB", e, [t2, rows(m)], **D)
        elif what == 5 and n % V == 0:                       # another row length ends it
            half = e.reshape(B, R * n // V, V)
            b.add("MAX_LAST", b.pool(to_dtype(np.zeros((B, R * n // V), np.float32), S.F32)), [half], **D)
            b.add("ADD", e, [e, t2], **D)
        b.add("SUM_LAST", l, [e], **D)
        b.add("SUB" if seed % 2 else "MUL", y, [e, rows(l)], **D)
        b.add("DIV", y, [y, vec], **D)
    return b.stream("row_chains_%d_%d" % (code, seed), batch=[128, 7, 12][seed % 3])


def scalar_chains(code):
    """Chains over rows whose scalars are not in registers any more when a task asks for them: other scalars of
    the rows were read in between, or they are read as another 16-bit format than they were written in."""
    rng = np.random.default_rng(3000 + code)
    b = Builder()
    V = 4 if code == S.F32 else 8
    for n, rows in ((V, 7), (8 * V, 200), (16 * V, 3000), (64 * V, 33)):
        pool = lambda hi, size: b.pool(to_dtype(rng.integers(-hi, hi + 1, size).astype(np.float32), code))
        per_row = lambda s: np.broadcast_to(s[:, None], (rows, n))
        D = dict(dep=(1, 0, 0))
        for m_code in (S.F32, S.F16):
            x, t, y, z = pool(8, (rows, n)), pool(1, (rows, n)), pool(1, (rows, n)), pool(1, (rows, n))
            m, k = (b.pool(to_dtype(rng.integers(1, 3, rows).astype(np.float32), m_code)) for _ in range(2))
            b.add("SCALE", t, [x], alpha=2.0)
            b.add("MAX_LAST", m, [t], **D)
            b.add("SUB", y, [t, per_row(m)], **D)
            b.add("MUL", y, [y, per_row(k)], **D)
            b.add("SUB", y, [y, per_row(m)], **D)
            b.add("MUL", y, [y, per_row(k)], **D)
            b.add("MIN_LAST", m, [y], **D)
            b.add("SUB", z, [y, per_row(m.view(np.uint16) if m_code == S.F16 else m)], **D)
    return b.stream("scalar_chains_%d" % code, batch=8)
