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
