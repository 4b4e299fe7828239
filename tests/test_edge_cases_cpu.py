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
    found = [p[0] for p in plans(s)]
    assert found.count("ROWS") > 0.8 * len(s)
    for (path, chunks, per, _), size, nd in zip(plans(s), s.tasks["size"], s.tasks["ndim"]):
        if path == "ROWS":                                # the chunks cover every vector (the narrowest operand's width)
            numel, C = int(np.prod(size[:nd])), int(size[nd - 1])
            assert chunks <= 1024 and chunks * per * 8 >= numel


def test_what_rows_leaves_to_the_other_paths():
    """Rows shorter than a vector, strided elements, transposed views, more outer dims than three,
    programs and mixed dtypes stay where they were."""
    from helpers import Builder
    b = Builder()
    x = b.pool(np.zeros((64, 64), np.float32))
    h = b.pool(np.zeros((64, 64), np.float16))
    o = b.pool(np.zeros((64, 65), np.float32))
    six = b.pool(np.zeros((3, 4, 3, 4, 3, 16), np.float32))
    b.add("ADD", o[:, 1:4], [x[:, :3], x[:, 1:4]])
    b.add("RELU", o[:, 1:33], [x[:, ::2]])
    b.add("ADD", o[:, 1:33], [x.T[:, :32], x[:, 32:]])
    b.add("MUL", o[:, 1:33], [h[:, :32], x[:, :32]])
    b.add("COPY", b.pool(np.zeros((2, 3, 2, 3, 3, 9), np.float32))[..., :8], [six[:2, 1:, 1:, 1:, :, :8]])
    b.add("ADD", o[:, 1:33], [np.broadcast_to(x[:1, :1], (64, 32)), np.broadcast_to(x[:, :1], (64, 32))])
    assert "ROWS" not in [p[0] for p in plans(b.stream())]
