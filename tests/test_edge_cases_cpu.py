"""CPU: the edge streams stay inside their buffers, the oracle takes them, and the host packs each task
into the execution path the stream is there for."""
import numpy as np
import pytest

from paper_2604_17861_amd import runtime as R
from paper_2604_17861_amd import streams as S
import edge_cases as E
from helpers import run_oracle
from parity_cases import stream_extent_violations


def aligned_tasks(stream):
    """The stream's descriptors with its pools at 256-byte aligned addresses (nothing lies there)."""
    bases, at = [], 1 << 20
    for p in stream.pools:
        bases.append(at)
        at += (p.nbytes + 511) // 256 * 256
    return stream.materialize(bases)


def plans(stream):
    """(path, chunks, chunk, dims) of every task, packed with its pools at 256-byte aligned addresses."""
    tasks = aligned_tasks(stream)
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
    # a rows task counts pieces of V elements (8 with a 16-bit operand), the partly filled last one of a row
    # included.  Others: an aligned matrix with one scalar per row is ROW2D, and a row shorter than a
    # piece (a cast's, four or five fp32 elements) is gathered or walked.
    taken = {"ROWS": 0, "ROW2D": 0, "STAGED": 0, "GENERIC": 0}
    for (path, chunks, per, dims), size, nd, dts in zip(plans(s), s.tasks["size"], s.tasks["ndim"], s.tasks["out"]["dtype"]):
        numel, C = int(np.prod(size[:nd])), int(size[nd - 1])
        W = 8 if V == 8 or dts not in (S.F32, S.I32) else 4
        taken[path] += 1
        assert path == "ROWS" or (path == "ROW2D" and C % V == 0) or C < W, (path, size, W)
        assert chunks <= 1024 and dims <= 4
        if path == "ROWS":
            vectors = {numel // c * -(-c // W) for c in (C, numel)}              # rows of the last dim, or one flat run
            assert any((chunks - 1) * per < v <= chunks * per for v in vectors)
    assert taken["ROWS"] > 0.85 * len(s) and taken["STAGED"] + taken["GENERIC"] <= 8, taken


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_gelu_values(code):
    s = E.gelu_values(code)
    assert not stream_extent_violations(s)
    assert [p[0] for p in plans(s)] == ["CONTIG", "ROWS"] * 2


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
    paths = []
    for (path, chunks, per, _), size, nd in zip(plans(s), s.tasks["size"], s.tasks["ndim"]):
        n, rows = int(size[nd - 1]), int(np.prod(size[:nd - 1]))
        paths.append((path, n))
        assert chunks == -(-rows // per)
    # shorter than a vector: any strides; whole vectors at aligned addresses: fused; every other one ragged
    t = aligned_tasks(s)
    ptrs = [[int(p) for p in ins[:k]] + [int(out)] for ins, out, k in zip(t["inp"]["ptr"], t["out"]["ptr"], t["n_inputs"])]
    for (path, n), ptr in zip(paths, ptrs):
        want = "ROW_GENERIC" if n < V else "ROW_FUSED" if n % V == 0 and all(p % 16 == 0 for p in ptr) else "ROW_RAGGED"
        assert path == want, (path, want, n, ptr)
    assert {p for p, _ in paths} >= {"ROW_GENERIC", "ROW_RAGGED"}


def test_what_rows_leaves_to_the_other_paths():
    """Rows shorter than a vector, strided elements, transposed views, mixed dtypes and more outer dims
    than three are walked, also where the output is no contiguous tensor."""
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
    assert [p[0] for p in plans(b.stream())] == ["GENERIC"] * 5 + ["ROWS"]


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
            V = 4 if code in (S.F32, S.I32) else 8
            units = {"ROWS": numel // V, "TILE2D": (C // 32) * -(-(n // C) // 32)}.get(path, n)
            assert (chunks - 1) * per < units <= chunks * per, what
            want = {"contiguous": "CONTIG", "unaligned": "ROWS", "slice": "ROWS", "generic": "GENERIC", "transposed": "TILE2D"}.get(layout, "STAGED")
            if code == S.I32 and want in ("TILE2D", "STAGED"):
                want = "GENERIC"
            assert path == want, what


@pytest.mark.parametrize("code", [S.F32, S.F16, S.I32])
def test_small_rows_tasks_stay_within_four_chunks(code):
    """A slice is cut into chunks of vectors, the last vector of a row partly filled: as a dependent task it
    is at most as many chunks as its elements make where those are at most four, the number up to
    which the dispatcher publishes it at once."""
    at = [(k + 1) << 36 for k in range(4)]
    V = 4 if code in (S.F32, S.I32) else 8
    for C in (V, V + 1, 2 * V - 1, 2 * V + 1, 65, 100, 1001):
        for numel in (2000, 9000, 16384, 20000, 32768, 60000, 300000):
            R_ = max(numel // C, 2)
            dense = [(at[k], [C, 1], code) for k in range(2)]
            path, want, per, _ = plan_of("ADD", [R_, C], dense, (at[3], [C, 1], code), dep=(1, 0, 0))
            assert path == "CONTIG"
            path, chunks, per, _ = plan_of("ADD", [R_, C], [(at[0], [C + 3, 1], code), dense[1]], (at[3], [C + 1, 1], code), dep=(1, 0, 0))
            vectors = R_ * -(-C // V)
            assert path == "ROWS" and (chunks - 1) * per < vectors <= chunks * per
            assert (chunks <= 4) if want <= 4 else (chunks > 4), (C, numel, want, chunks)


@pytest.mark.parametrize("op", ["SOFTMAX_LAST", "MASKED_SOFTMAX_LAST", "LAYERNORM_LAST"])
def test_rows_up_to_the_last_addressable_byte(op):
    """The executors of contiguous rows address a row by byte offsets below 0x7ffffff0, the offset that is
    given to the stores that are to do nothing: longer rows are walked."""
    at = [(k + 1) << 40 for k in range(4)]
    most = 0x7ffffff0 // 4                                       # fp32 elements
    for n, want in ((1000, "ROW_FUSED"), (1001, "ROW_RAGGED"), (most - 4, "ROW_FUSED"), (most - 1, "ROW_RAGGED"), (most, "ROW_FUSED"),
                    (most + 1, "ROW_GENERIC"), (most + 2, "ROW_GENERIC"), (most + 3, "ROW_GENERIC")):
        for rows in (1, 3) if n > 2000 else (1, 3, 100000):
            st = {"SOFTMAX_LAST": [[n, 1]], "MASKED_SOFTMAX_LAST": [[n, 1], [0, 1]], "LAYERNORM_LAST": [[n, 1], [0, 1], [0, 1]]}[op]
            path = plan_of(op, [rows, n], [(at[k], s, S.F32) for k, s in enumerate(st)], (at[3], [n, 1], S.F32), alpha=1.0)[0]
            assert path == want, (op, rows, n, path)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_long_softmax_rows_are_whole_and_ragged_at_every_length(code):
    s = E.long_softmax_rows_whole_and_not(code)
    assert not stream_extent_violations(s)
    V, longest = (4, 21 * 256) if code == S.F32 else (8, 15 * 256)       # vectors that registers and LDS hold with fewer batches
    seen = {"ROW_FUSED": set(), "ROW_RAGGED": set()}
    for (path, _, _, _), size in zip(plans(s), s.tasks["size"]):
        seen[path].add(-(-int(size[1]) // V))
    for vectors in seen.values():
        assert min(vectors) <= longest < max(vectors) and {longest, longest + 1} <= vectors
    run_oracle(s)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16, S.I32])
def test_tasks_past_the_cache(code):
    s = E.past_the_cache(code)
    assert not stream_extent_violations(s)
    assert {p[0] for p in plans(s)} == ({"RED_CONTIG"} if code == S.I32 else {"RED_CONTIG", "CONTIG"})
    read = sorted({int(np.prod(t["size"][:t["ndim"]])) * int(t["n_inputs"]) * S.ELEM_SIZE[code] for t in s.tasks})
    assert read[0] < 16 << 20 < read[-1] and read[-1] < 18 << 20
    run_oracle(s)
