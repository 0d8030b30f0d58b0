"""The gather of the previous block's classes at the sizes where its form
changes: 8 rows a block by 4 or 16 waves, 4 rows by 16 waves, and rows read from
memory (buckets that may hold more than 38,848 tokens at k = 2); 18000 and 36000
tokens at k = 2 take more than 64 KB of LDS a block.  Every block's
graph, pair counts and record against the oracle's chain."""
import pytest

import luffy_gen as G
from tests.test_gpu_history import run_stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_15419_amd as L
    L.load_library()


@pytest.mark.parametrize("T,k", [(700, 1), (9001, 2), (12000, 2), (18000, 2), (20011, 2), (36000, 2), (40003, 2),
                                 (40003, 1)])
def test_gather_forms(T, k):
    stack = G.make_stack("c2", 2, seed=T + k, T=T, d=256, E=64, k=k, n_centres=T // 5, capacity_factor=0.0,
                         token_drift=0.1, gate_drift=0.1)
    st = run_stack(stack, h=0.9, S1=0.8, S2=0.45, check_record=T < 20000)
    assert st[1][0] > 0 and st[1][1] > 0
