"""CPU: the edge streams stay inside their buffers, the oracle takes them, and the host packs each task
into the execution path the stream is there for."""
import numpy as np
import pytest

from paper_2604_17861_amd import runtime as R
from paper_2604_17861_amd import streams as S
import edge_cases as E
from helpers import run_oracle
from parity_cases import stream_extent_violations


def plans(stream):
    """(path, chunks, chunk, dims) of every task, packed with its pools at 256-byte aligned addresses."""
    bases, at = [], 1 << 20
    for p in stream.pools:
        bases.append(at)
        at += (p.nbytes + 511) // 256 * 256
    tasks = stream.materialize(bases)
    impls = stream.impl_for(None)
    return [R.task_plan(tasks, i, int(impls[i])) for i in range(len(stream))]


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_reduction_edges(code):
    s = E.reduction_edges(code)
    assert not stream_extent_violations(s)
    run_oracle(s)
    assert {p[0] for p in plans(s)} == {"RED_CONTIG"}
    # a reduction of a megabyte or less is at least as many chunks as 16 KiB pieces, whole rows each
    for i, (_, chunks, per, _) in enumerate(plans(s)):
        rows, n = (int(v) for v in s.tasks["size"][i][:2])
        assert per == 1 or per * n * S.ELEM_SIZE[code] <= 2 * 16384
        assert chunks == -(-rows // per)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_rows_edges(code):
    s = E.rows_edges(code)
    assert not stream_extent_violations(s)
    run_oracle(s)
    V = 4 if code in (S.F32, S.I32) else 8
    # the chunks cover every element once; a rows task counts vectors of V (8 with a 16-bit operand), the
    # partly filled last one of a row included
    counted_in_vectors = 0
    for (path, chunks, per, _), size, nd, dts in zip(plans(s), s.tasks["size"], s.tasks["ndim"], s.tasks["out"]["dtype"]):
        numel, C = int(np.prod(size[:nd])), int(size[nd - 1])
        W = 8 if V == 8 or dts not in (S.F32, S.I32) else 4
        vectors = numel // C * -(-C // W)
        assert chunks <= 1024 and (chunks == -(-numel // per) or chunks == -(-vectors // per) or C < W or path == "CONTIG")
        counted_in_vectors += chunks == -(-vectors // per)
    assert counted_in_vectors > 0.8 * len(s)


def test_large_gathers():
    s = E.large_gathers()
    assert not stream_extent_violations(s)
    for (path, chunks, per, _), size, nd in zip(plans(s), s.tasks["size"], s.tasks["ndim"]):
        numel = int(np.prod(size[:nd]))
        assert path == "STAGED" and chunks <= 1024 and (chunks - 1) * per < numel <= chunks * per and per > 8192


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_row_operation_edges(code):
    s = E.row_operation_edges(code)
    assert not stream_extent_violations(s)
    run_oracle(s)
    V = 4 if code == S.F32 else 8
    for (path, chunks, per, _), size, nd in zip(plans(s), s.tasks["size"], s.tasks["ndim"]):
        n, rows = int(size[nd - 1]), int(np.prod(size[:nd - 1]))
        assert path in ("ROW_FUSED", "ROW_GENERIC") and (n >= V or path == "ROW_GENERIC")
        assert chunks == -(-rows // per)


def test_what_rows_leaves_to_the_other_paths():
    """Rows shorter than a vector, strided elements, transposed views, more outer dims than three and
    mixed dtypes keep their chunks, which count elements in thousands; rows count vectors."""
    from helpers import Builder
    b = Builder()
    x = b.pool(np.zeros((640, 64), np.float32))
    h = b.pool(np.zeros((640, 64), np.float16))
    o = b.pool(np.zeros((640, 65), np.float32))
    sq = b.pool(np.zeros((640, 640), np.float32))
    six = b.pool(np.zeros((3, 4, 3, 4, 3, 256), np.float32))
    b.add("ADD", o[:, 1:4], [x[:, :3], x[:, 1:4]])
    b.add("RELU", o[:, 1:33], [x[:, ::2]])
    b.add("ADD", o[:, 1:65], [sq.T[:, :64], x])
    b.add("MUL", o[:, 1:33], [h[:, :32], x[:, :32]])
    b.add("COPY", b.pool(np.zeros((2, 3, 2, 3, 3, 129), np.float32))[..., :128], [six[:2, 1:, 1:, 1:, :, :128]])
    b.add("ADD", o[:, 1:33], [x[:, :32], x[:, 32:]])                    # ... and this one is rows
    s = b.stream()
    counts_vectors = []
    for (path, chunks, per, _), size, nd in zip(plans(s), s.tasks["size"], s.tasks["ndim"]):
        numel, C = int(np.prod(size[:nd])), int(size[nd - 1])
        assert path == "GENERIC"
        counts_vectors.append(chunks != -(-numel // per) and chunks == -(-(numel // C * -(-C // 4)) // per))
    assert counts_vectors == [False] * 5 + [True], counts_vectors


def plan_of(op, shape, ins, out, alpha=0.0, dep=(0, 0, 0)):
    """The plan of one task from (address, strides in elements, dtype) of its operands; nothing is read."""
    tasks, pool_of = S.new_tasks(1)
    S.set_head(tasks, 0, S.OP[op], shape, len(ins), alpha=alpha, dep=dep)
    for k, (ptr, st, dt) in enumerate(ins):
        S.set_tensor(tasks, pool_of, 0, k, 0, ptr, st, dt)
    S.set_tensor(tasks, pool_of, 0, 3, 0, *out)
    return R.task_plan(tasks, 0, S.IMPL[op])


@pytest.mark.parametrize("layout", ["contiguous", "unaligned", "gathered", "gathered beside a dense input", "generic", "transposed", "slice"])
@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_no_task_is_more_than_1024_chunks(layout, code):
    """A work unit names its chunk in ten bits: however large a task is and whatever the regular chunk of
    its path, it is at most 1,024 chunks, and they cover it exactly."""
    at = [(k + 1) << 36 for k in range(4)]
    ops = {1: "COPY", 2: "MUL"} if code == S.I32 else {1: "SCALE", 2: "MUL", 3: "FMA"}
    for numel in (1 << 20, (1 << 20) + 4096, 8 << 20, (8 << 20) + 4096, 9 << 20, 12 << 20, 14 << 20, (16 << 20) + 4096, 24 << 20, 32 << 20, 48 << 20, 64 << 20,
                  (64 << 20) + 4096, 256 << 20):
        for arity, op in ops.items():
            n, C = numel, 4096
            dense, out, shape = [1], (at[3], [1], code), [n]
            ins = [(at[k], [1], code) for k in range(arity)]
            if layout == "unaligned":
                ins[0] = (at[0] + 4, [1], code)
            elif layout == "gathered":                       # every input a stride-2 slice
                ins = [(at[k], [2], code) for k in range(arity)]
            elif layout == "gathered beside a dense input":
                ins[0] = (at[0], [2], code)
            elif layout == "generic":
                ins[0], out = (at[0], [3], code), (at[3], [2], code)
            elif layout == "transposed":
                shape, ins, out = [C, n // C], [(at[k], [1, C], code) for k in range(arity)], (at[3], [n // C, 1], code)
            elif layout == "slice":
                shape, ins, out = [n // C, C], [(at[k], [C + 3, 1], code) for k in range(arity)], (at[3], [C + 1, 1], code)
            path, chunks, per, _ = plan_of(op, shape, ins, out)
            what = (layout, op, numel, path, chunks, per)
            assert 1 <= chunks <= 1024, what
            if path in ("CONTIG", "STAGED", "GENERIC") and layout not in ("unaligned", "slice"):
                assert (chunks - 1) * per < n <= chunks * per, what
