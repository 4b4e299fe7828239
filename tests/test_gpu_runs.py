"""GPU: chains of tasks that one workgroup runs chunk by chunk, against sequential execution; how many work units they had."""
import numpy as np
import pytest

from paper_2604_17861_amd import runtime as R
from paper_2604_17861_amd import streams as S
import edge_cases as E

pytestmark = pytest.mark.gpu


def _run(s, capacity=4096):
    """Through the worker and through the oracle, whole buffers byte for byte; the worker's counters."""
    from gpu_helpers import DevicePools, run_stream
    from helpers import run_oracle
    dp = DevicePools(s)
    with R.Runtime(capacity, idle_exit_ms=20000, wait_timeout_ms=20000) as rt:
        rt.register_table(s.table)
        t0 = run_stream(s, rt, dp)
        comps = rt.completions(t0, len(s)) if capacity >= len(s) else None
        rt.stop_worker()
        stats = rt.worker_stats()
    # the units there would be if every task had its own
    stats["lone_units"] = sum(R.task_plan(dp.tasks, i, int(impl))[1] for i, impl in enumerate(s.impl_for(None)))
    assert comps is None or np.all(comps["status"] == 0)
    hp, st = run_oracle(s)
    assert np.all(st == 0)
    for k, (g, o) in enumerate(zip(dp.download(), hp.arrays)):
        g8, o8 = np.asarray(g).view(np.uint8).reshape(-1), np.asarray(o).view(np.uint8).reshape(-1)
        assert np.array_equal(g8, o8), "buffer %d differs at bytes %s" % (k, np.nonzero(g8 != o8)[0][:16])
    return stats


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
@pytest.mark.parametrize("capacity", [64, 4096])
def test_chains_with_what_ends_a_run(code, capacity):
    for seed in range(3):
        s = E.chains(code, seed)
        stats = _run(s, capacity)
        print("chains", code, capacity, seed, len(s), stats["lone_units"], stats["disp_units"], flush=True)
        # (a ring of 64 is published a few tasks at a time, and a run ends where a pass of the dispatcher does)
        assert stats["disp_units"] < stats["lone_units"] // (2 if capacity > 64 else 1)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_chains_over_rows(code):
    for seed in range(6):
        s = E.row_chains(code, seed)
        stats = _run(s)
        print("row chains", code, seed, len(s), stats["lone_units"], stats["disp_units"], flush=True)
        # nine chains of eleven are rows of whole vectors, up to 64: a run's units stand for all its tasks
        assert stats["disp_records"] == len(s) and stats["disp_units"] < stats["lone_units"] // 2


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
@pytest.mark.parametrize("blocks", [384, 768])
def test_chains_over_many_rows(code, blocks):
    """Chunks of two and of four blocks of rows, the last chunk and the last block partly filled."""
    V = 4 if code == S.F32 else 8
    s = E.row_chains(code, 1 + blocks // 384, [(16 * V, 1, blocks * 64 + 37)])
    stats = _run(s)
    print("many rows", code, blocks, len(s), stats["lone_units"], stats["disp_units"], flush=True)
    rows, chunk = blocks * 64 + 37, blocks // 384 * 2 * 64     # 64 rows a block: two blocks a chunk, four from 768 on
    assert stats["disp_units"] == -(-rows // chunk)            # one run


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_scalars_that_left_the_registers(code):
    s = E.scalar_chains(code)
    print("scalar chains", code, len(s), flush=True)
    _run(s)


@pytest.mark.parametrize("code,n", [(S.F32, 1000), (S.F32, 16384), (S.F16, 4097), (S.BF16, 40000)])
def test_long_chains_are_run_together(code, n):
    s = E.long_chains(code, n)
    stats = _run(s)
    print("long chains", code, n, len(s), stats["disp_units"], stats["work_units"], flush=True)
    assert stats["disp_records"] == len(s)
    assert stats["disp_units"] == stats["work_units"] < len(s) // 2
