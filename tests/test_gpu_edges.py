"""GPU: every execution path at the sizes where its shape of work changes, against the oracle."""
import pytest

from paper_2604_17861_amd import streams as S
import edge_cases as E
from test_gpu_parity import _run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_reductions_at_their_edges(code):
    stats, _ = _run_and_check(E.reduction_edges(code))
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_reductions_of_shared_out_rows(code):
    stats, _ = _run_and_check(E.reduction_shares(code))
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_reductions_of_long_rows(code):
    stats, _ = _run_and_check(E.reduction_long_rows(code))
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_rows_at_their_edges(code):
    stats, _ = _run_and_check(E.rows_edges(code))
    print(stats, flush=True)


def test_an_operator_swapped_under_tasks_packed_as_rows():
    """Tasks are packed for the operator bound when they are submitted and run with the one bound when
    they are claimed: rows whose new operator has no executor of that kind (a program, another unary
    operator on a converting copy) run element by element.  The swap falls between submission and
    flush, so every task is claimed with the second binding."""
    import numpy as np
    from gpu_helpers import DevicePools, compare_with_oracle
    from helpers import Builder
    from paper_2604_17861_amd import runtime as R
    rng = np.random.default_rng(3)
    P = S.program
    sub = (P(("SUB", 4, 1, 0), ("MOV", 0, 4)), 2)
    # (the last three: one scalar per row under another operator of the class and under a program, int32)
    for op, new, kind in (("COPY", "RELU", "plain"), ("SCALE", (P(("NEG", 0, 0)), 1), "plain"), ("SUB", sub, "plain"),
                          ("SUB", "DIV", "scalar"), ("MUL", sub, "scalar"), ("ADD", "SUB", "int32")):
        print("swap under", op, kind, flush=True)
        b = Builder()
        prog = not isinstance(new, str)
        impl = b.define_program(200, *new) if prog else S.IMPL[new]
        for R_, C_ in ((5, 37), (90, 1001)):
            code = S.I32 if kind == "int32" else S.F32
            x = b.pool(E.values(rng, (R_, C_ + 5), code))[:, 2:C_ + 2]
            y = b.pool(E.values(rng, (R_, C_), code))
            if kind != "plain":
                y = np.broadcast_to(b.pool(E.values(rng, (R_, 1), code)), (R_, C_))
            o = b.pool(np.zeros((R_, C_ + 1), np.float16 if op == "COPY" else np.int32 if kind == "int32" else np.float32))[:, 1:]
            b.add(op, o, [x, y] if op in ("SUB", "MUL", "ADD") else [x], alpha=2.0)
        s = b.stream("swap_under_rows")
        dp = DevicePools(s)
        with R.Runtime(0, idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
            rt.register_table(s.table, s.programs)
            t0 = rt.submit(dp.tasks, 0, len(s), flush=False)
            rt.swap_op(S.OP[op], impl)
            rt.wait()
            comps = rt.completions(t0, len(s))
        assert np.all(comps["status"] == 0) and np.all(comps["op_version"] == 2)
        s.table[S.OP[op]] = impl
        compare_with_oracle(s, dp.download())


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_row_operations_at_their_edges(code):
    stats, _ = _run_and_check(E.row_operation_edges(code))
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_softmax_rows_kept_in_part(code):
    stats, _ = _run_and_check(E.long_softmax_rows(code))
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_slices_with_a_step_of_two(code):
    stats, _ = _run_and_check(E.every_second_element(code))
    print(stats, flush=True)


def test_gathers_larger_than_1024_regular_chunks():
    stats, _ = _run_and_check(E.large_gathers())
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_gelu_rounds_the_64_bit_value(code):
    """A GELU is evaluated in 64 bits whatever its dtype is: every result of a 16-bit input, the sign of a
    zero included, is the rounded value of the oracle's double evaluation.  For fp32 both sides are
    within 2^-45 of the exact value on these inputs, 2^-49 or better on most, so that a result is
    rounded differently about once in 2^20 to 2^24: at most 4 of 2.1 million (an evaluation good to
    2^-39 gives 60)."""
    import numpy as np
    from gpu_helpers import DevicePools, run_stream
    from helpers import run_oracle
    from paper_2604_17861_amd import runtime as R
    s = E.gelu_values(code)
    print("case", s.name, flush=True)
    dp = DevicePools(s)
    with R.Runtime(0, idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
        rt.register_table(s.table, s.programs)
        run_stream(s, rt, dp)
    hp, st = run_oracle(s)
    assert np.all(st == 0)
    differ = total = 0
    for got, want in zip(dp.download(), hp.arrays):
        dt = np.uint32 if code == S.F32 else np.uint16
        fl = {S.F32: np.float32, S.F16: np.float16}.get(code)
        g, w = np.ascontiguousarray(got).view(dt), np.ascontiguousarray(want).view(dt)
        nan = np.isnan(w.view(fl)) if fl else (w & 0x7fff) > 0x7f80
        g_nan = np.isnan(g.view(fl)) if fl else (g & 0x7fff) > 0x7f80
        assert np.array_equal(nan, g_nan)
        differ += int(np.count_nonzero((g != w) & ~nan))
        total += g.size
    print("differ", differ, "of", total, flush=True)
    assert differ <= (4 if code == S.F32 else 0)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_row_operations_in_place(code):
    """Rows written over the rows they are made of: the last vector of a ragged row re-reads elements
    that another lane may have written by then, and must not use them.  The results are those of the
    same tasks with an output of their own (which the test above compares with the oracle)."""
    import numpy as np
    from gpu_helpers import DevicePools, run_stream
    from helpers import Builder
    from paper_2604_17861_amd import runtime as R
    V = 4 if code == S.F32 else 8
    got = []
    for in_place in (False, True):
        rng = np.random.default_rng(750 + code)
        b, outs = Builder(), []
        for rows, n in ((70, V + 1), (300, 3 * V - 1), (131, 32 * V + 1), (65, 64 * V + 1), (17, 128 * V + 1), (9, 256 * V + 1), (9, 257 * V),
                        (5, 512 * V + 3), (3, 1024 * V + 1), (3, 2048 * V + 1), (2, 4096 * V + V + 1), (2, 5632 * V + 1), (64, 64 * V)):
            for name in ("SOFTMAX_LAST", "MASKED_SOFTMAX_LAST", "LAYERNORM_LAST"):
                x = b.pool(E.values(rng, rows * n + 1, code, 3.0))[n % 2:][:rows * n].reshape(rows, n)
                more = [np.broadcast_to(b.pool(E.values(rng, n, code)), (rows, n)) for _ in range({"S": 0, "M": 1, "L": 2}[name[0]])]
                o = x if in_place else b.pool(np.zeros(rows * n + 1, x.dtype))[n % 2:][:rows * n].reshape(rows, n)
                b.add(name, o, [x] + more, alpha=0.25)
                outs.append(b._locate(o) + (rows * n * x.itemsize,))
        s = b.stream("rows_in_place" if in_place else "rows_apart")
        print("case", s.name, code, len(s), flush=True)
        dp = DevicePools(s)
        with R.Runtime(0, idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
            rt.register_table(s.table)
            t0 = run_stream(s, rt, dp)
            assert np.all(rt.completions(t0, len(s))["status"] == 0)
        imgs = dp.download()
        got.append([np.ascontiguousarray(imgs[k]).view(np.uint8).reshape(-1)[off: off + nb] for k, off, nb in outs])
    for i, (a, c) in enumerate(zip(*got)):
        assert np.array_equal(a, c), i


@pytest.mark.parametrize("code", [S.F16, S.BF16])
def test_gelu_of_16bit_inputs_is_the_rounded_fp64_value(code):
    """Every 16-bit pattern, in three orders, through both GELUs: the 16-bit output is the fp32 output (evaluated
    in fp64) rounded once more, bit for bit."""
    import numpy as np
    from gpu_helpers import DevicePools, run_stream
    from helpers import Builder, bf16_bits_to_f32
    from parity_cases import to_dtype
    from paper_2604_17861_amd import runtime as R
    b, pairs = Builder(), []
    for seed in range(3):
        bits = np.random.default_rng(seed).permutation(65536).astype(np.uint16)
        X = b.pool(bits.view(np.float16).copy() if code == S.F16 else bits)
        for name in ("GELU_ERF", "GELU_TANH"):
            o16, o32 = b.pool(np.zeros(65536, X.dtype)), b.pool(np.zeros(65536, np.float32))
            b.add(name, o16, [X])
            b.add(name, o32, [X])
            pairs.append((len(b.bases) - 2, len(b.bases) - 1))
    s = b.stream("gelu_16bit_%d" % code)
    dp = DevicePools(s)
    with R.Runtime(idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
        rt.register_table(s.table)
        run_stream(s, rt, dp)
    got = dp.download()
    for k16, k32 in pairs:
        y16, y32 = got[k16].view(np.uint16), got[k32].view(np.float32)
        if code == S.F16:
            with np.errstate(over="ignore"):
                want = y32.astype(np.float16).view(np.uint16)
        else:
            w = y32.view(np.uint32).astype(np.uint64)
            want = ((w + 0x7FFF + ((w >> 16) & 1)) >> 16).astype(np.uint16)
        nan = np.isnan(y32)
        is_nan = np.isnan(y16.view(np.float16)) if code == S.F16 else np.isnan(bf16_bits_to_f32(y16))
        assert np.array_equal(nan, is_nan)
        bad = np.nonzero((y16 != want) & ~nan)[0]
        assert len(bad) == 0, (code, k16, len(bad), y32[bad[:5]], y16[bad[:5]], want[bad[:5]])


@pytest.mark.parametrize("n", [2048, 8191, 8192, 8193, 12288, 12289, 33000, 65536])
def test_gelu_of_bf16_inputs_round_a_batch(n):
    """Round the batch of 8,192 elements from which on a chunk is evaluated in fp32 first: the result is the fp32
    output (evaluated in fp64) rounded once more, bit for bit, aligned and one element off."""
    import numpy as np
    from gpu_helpers import DevicePools, run_stream
    from helpers import Builder
    from paper_2604_17861_amd import runtime as R
    b, pairs = Builder(), []
    bits = np.random.default_rng(n).permutation(65536).astype(np.uint16)
    bits = np.append(bits[(bits & 0x7fff) <= 0x7f80], bits[:1024])[:n]            # (no NaN, whose bits are free)
    bits[(bits & 0x7fff) > 0x7f80] = 0
    for off in (0, 1):
        X = b.pool(np.append(np.zeros(off, np.uint16), bits))[off:]
        o16, o32 = b.pool(np.zeros(bits.size + off, np.uint16))[off:], b.pool(np.zeros(bits.size, np.float32))
        b.add("GELU_ERF", o16, [X])
        b.add("GELU_ERF", o32, [X])
        pairs.append((len(b.bases) - 2, len(b.bases) - 1, off))
    s = b.stream("gelu_bf16_batch_%d" % n)
    dp = DevicePools(s)
    with R.Runtime(idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
        rt.register_table(s.table)
        run_stream(s, rt, dp)
    got = dp.download()
    for k16, k32, off in pairs:
        w = got[k32].view(np.uint32).astype(np.uint64)
        want = ((w + 0x7FFF + ((w >> 16) & 1)) >> 16).astype(np.uint16)
        assert np.array_equal(got[k16].view(np.uint16)[off:], want)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_long_softmax_rows_at_every_alignment(code):
    """Rows too long for the workgroup's registers, cut at memory's 16-byte blocks where input and output lie alike in
    them and from the row's first element on where they do not; nothing outside the output is written."""
    import numpy as np
    from gpu_helpers import DevicePools, compare_with_oracle, run_stream
    from helpers import Builder
    from paper_2604_17861_amd import runtime as R
    rng = np.random.default_rng(40 + code)
    V, rows, pad = (4 if code == S.F32 else 8), 3, 16
    b, outs = Builder(), []
    for n in (16385, 16384 + V - 1, 20001, 32003):
        for xo, oo in ((0, 0), (1, 1), (V - 1, V - 1), (2, 0), (0, 1)):
            x = b.pool(E.values(rng, rows * n + 2 * pad, code))
            o = b.pool(np.zeros_like(x))
            b.add("SOFTMAX_LAST", o[pad + oo: pad + oo + rows * n].reshape(rows, n), [x[pad + xo: pad + xo + rows * n].reshape(rows, n)])
            outs.append((len(b.bases) - 1, pad + oo, rows * n))
    s = b.stream("long_softmax_%d" % code)
    dp = DevicePools(s)
    with R.Runtime(idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
        rt.register_table(s.table)
        t0 = run_stream(s, rt, dp)
        comps = rt.completions(t0, len(s))
    got = dp.download()
    print(compare_with_oracle(s, got, versions=comps["op_version"]), flush=True)
    for k, first, count in outs:
        words = got[k].view(np.uint32 if code == S.F32 else np.uint16)
        assert not words[:first].any() and not words[first + count:].any()


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_long_softmax_rows_whole_and_not(code):
    """Whole aligned rows on both sides of every length at which more is kept of a row, and the same lengths at other alignments."""
    stats, _ = _run_and_check(E.long_softmax_rows_whole_and_not(code))
    print(stats, flush=True)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_tasks_past_the_cache(code):
    stats, _ = _run_and_check(E.past_the_cache(code))
    print(stats, flush=True)
