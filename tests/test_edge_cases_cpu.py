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
