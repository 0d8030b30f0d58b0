"""Small calls: the undecided positions and the representative rows in one kernel
(at most 4096 slots), at the edges of its 64- and 1024-position pieces, with
chains that the first round leaves undecided."""
import numpy as np
import pytest

import luffy_gen as G
from tests.layer_runner import (assert_condense_equal, assert_output_close, assert_route_equal, fetch, make_layer,
                                run_gpu, run_oracle, upload)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_15419_amd as L
    L.load_library()


@pytest.mark.parametrize("T,k,E,mix", [(1, 1, 1, 0.0), (32, 2, 4, 0.0), (64, 1, 2, 0.2), (65, 1, 1, 0.3), (511, 2, 4, 0.3),
                                       (512, 2, 3, 0.3), (2048, 2, 4, 0.3), (2049, 2, 4, 0.3), (4096, 1, 64, 0.2),
                                       # one block a bucket up to 1024 positions, one per 256 above
                                       (1024, 1, 1, 0.3), (1025, 1, 1, 0.3), (4096, 1, 1, 0.3), (1100, 2, 16, 0.3),
                                       (1100, 1, 64, 0.5)])
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


@pytest.mark.parametrize("T,E", [(900, 1), (3001, 1), (4000, 8)])
def test_small_call_dense(T, E):
    """A bucket of tokens of one direction whose cosines lie around the threshold:
    thousands of undecided positions with full rows."""
    inp = G.make_inputs("c2", seed=2, weights=False, T=T, d=512, E=E, k=1, n_centres=4, capacity_factor=0.0)
    rng = np.random.default_rng(T)
    x = rng.standard_normal((1, 512)) + rng.uniform(0.2, 0.45, (T, 1)) * rng.standard_normal((T, 512))
    inp.x = G.round_bf16(x.astype(np.float32))
    inp.w_g[:] = 0.0
    inp.b_g[:] = -np.arange(E)        # every token goes to expert 0
    g = run_gpu(inp, h=0.9, with_ffn=False)
    lo, hi = 0, int(g["offsets"][1])
    assert hi == T
    # the walk of the oracle on the graph that the cosines give in float64 differs
    # where a cosine lies within float32 rounding of the threshold: the walk's own
    # rule is checked on the call's outputs instead
    rep, deg = g["rep_of_pos"][lo:lo + hi] - lo, g["degree"][lo:lo + hi]
    tok = g["perm_token"][lo:lo + hi]
    u = inp.x[tok].astype(np.float64)
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    c = u @ u.T
    np.fill_diagonal(c, -1.0)
    assert np.abs(deg - (c >= 0.9).sum(1)).max() <= 2
    kept = np.flatnonzero(rep == np.arange(hi))
    assert 1 < kept.size < hi
    assert c[np.ix_(kept, kept)].max() < 0.9 + 1e-6, "two kept positions are similar"
    gone = np.flatnonzero(rep != np.arange(hi))
    assert np.isin(rep[gone], kept).all() and c[gone, rep[gone]].min() >= 0.9 - 1e-6
    # the representative is the first kept neighbour in walk order
    order = np.lexsort((np.arange(hi), -deg))
    rank = np.empty(hi, np.int64)
    rank[order] = np.arange(hi)
    near = np.where(c[np.ix_(gone, kept)] >= 0.9 + 1e-6, rank[kept][None, :], hi)
    assert (rank[rep[gone]] <= near.min(1)).all()


@pytest.mark.parametrize("T,max_bucket", [(900, 100), (3000, 1200), (4096, 1025), (6000, 1000)])
def test_bucket_larger_than_max_bucket(T, max_bucket):
    """A bucket larger than the caller's bound: nothing is decided and every
    position represents itself, in every form of the last kernels."""
    inp = G.make_inputs("c2", seed=2, weights=False, T=T, d=256, E=3, k=1, n_centres=4, capacity_factor=0.0)
    inp.w_g[:] = 0.0
    inp.b_g[:] = -np.arange(3)
    dev = upload(inp)
    layer = make_layer(inp, dev, 0.9)
    assert layer.max_bucket == T
    layer.max_bucket = max_bucket
    print(f"[case] T={T} max_bucket={max_bucket}", flush=True)
    layer.buf.rep_of_pos.fill_(-7)
    layer.route(dev["x"])
    layer.condense(dev["x"])
    g = fetch(layer, with_ffn=False)
    assert g["offsets"].tolist() == [0, T, T, T] and g["rep_offsets"].tolist() == [0, T, T, T]
    assert np.array_equal(g["rep_of_pos"], np.arange(T)) and np.array_equal(g["rep_row"], np.arange(T))
    assert np.array_equal(g["rep_token"], g["perm_token"])
