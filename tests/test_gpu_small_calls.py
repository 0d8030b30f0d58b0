"""Small calls: the finishing pass and the representative rows in one kernel (at
most 4096 slots), at the edges of its 64- and 1024-position pieces, with chains
that the first round leaves undecided."""
import numpy as np
import pytest

import luffy_gen as G
from tests.layer_runner import assert_condense_equal, assert_output_close, assert_route_equal, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_15419_amd as L
    L.load_library()


@pytest.mark.parametrize("T,k,E,mix", [(1, 1, 1, 0.0), (32, 2, 4, 0.0), (64, 1, 2, 0.2), (65, 1, 1, 0.3), (511, 2, 4, 0.3),
                                       (512, 2, 3, 0.3), (2048, 2, 4, 0.3), (2049, 2, 4, 0.3), (4096, 1, 64, 0.2)])
def test_small_calls(T, k, E, mix):
    """Mixed tokens (of two groups each) link the groups into decision chains."""
    stack = G.make_stack("c2", 1, seed=T + k, T=T, d=256, d_ff=128, E=E, k=k, n_centres=max(1, T // 6),
                         mix_fraction=mix, capacity_factor=0.0, weights=True)
    inp = stack[0]
    print(f"[case] small T={T} k={k} E={E} mix={mix}", flush=True)
    g = run_gpu(inp, h=0.62)
    o = run_oracle(inp, h=0.62)
    assert_route_equal(g, o)
    assert_condense_equal(g, o)
    assert_output_close(g, o, "bf16")


def test_small_call_identical_tokens_and_drops():
    """One group per expert, capacity drops, an expert without tokens."""
    cfg = G.config("c2", T=600, d=256, d_ff=128, E=8, n_centres=1, capacity_factor=0.5)
    inp = G.make_inputs(cfg, seed=3)
    inp.x[:] = inp.x[0]
    g = run_gpu(inp)
    o = run_oracle(inp)
    assert_route_equal(g, o)
    assert_condense_equal(g, o)
    assert np.diff(g["offsets"]).min() == 0
