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
