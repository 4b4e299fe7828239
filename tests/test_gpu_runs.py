"""GPU: chains of elementwise tasks that one workgroup runs chunk by chunk, against sequential execution."""
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
        print("chains", code, capacity, seed, len(s), flush=True)
        _run(s, capacity)


@pytest.mark.parametrize("code", [S.F32, S.F16, S.BF16])
def test_chains_over_rows(code):
    for seed in range(6):
        s = E.row_chains(code, seed)
        print("row chains", code, seed, len(s), flush=True)
        stats = _run(s)
        assert stats["disp_records"] == len(s)


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
