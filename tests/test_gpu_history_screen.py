"""Historical similarity on fp8 rows (long bf16 rows, large buckets): every
block's graph, pair counts and record must be those of the all-bf16 kernel bit
for bit, whichever way a tile is decided (from its fp8 products, pair by pair,
handed back, or skipped), and the oracle's."""
import copy

import numpy as np
import pytest

import luffy_gen as G
from tests.layer_runner import fetch, make_layer, screen_state, upload
from tests.test_gpu_history import run_stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_15419_amd as L
    L.load_library()


def _chain(stack, h, S1, S2, screen, routed=None, back=None):
    """Blocks of a stack; routed: the inputs they are routed on, if others; back
    receives each block's tiles handed back and tiles in all."""
    import torch
    import paper_2411_15419_amd as L
    prev, out = None, []
    back = [] if back is None else back
    was = L.set_similarity_screen(screen)
    try:
        for inp, first in zip(stack, routed or stack):
            cfg = inp.cfg
            assert L.similarity_screen_applies(cfg.T, cfg.d, cfg.E, cfg.k) == screen
            dev = upload(inp)
            base = make_layer(inp, dev, h)
            layer = L.MoELayer(base.w_gate, base.b_gate, base.w1, base.w2, k=cfg.k, act=cfg.act, threshold=h,
                               capacity_factor=cfg.capacity_factor, T=cfg.T, norms_from_route=routed is None,
                               history=(S1, S2))
            layer.record.zero_()
            layer.route(upload(first)["x"])
            layer.condense(dev["x"], hist_in=prev)
            torch.cuda.synchronize()
            g = fetch(layer, with_ffn=False)
            out.append({**{n: np.array(g[n]) for n in ("offsets", "rep_offsets", "rep_of_pos", "rep_row", "degree")},
                        "stats": layer.hist_stats.cpu().numpy(), "record": layer.record.cpu().numpy()})
            if screen:
                state = screen_state(layer)
                back.append((state["listed"].size, state["total"]))
            prev = layer.record
    finally:
        L.set_similarity_screen(was)
    return out


def _same(a, b):
    for blk, (on, off) in enumerate(zip(a, b)):
        n, r = int(off["offsets"][-1]), int(off["rep_offsets"][-1])
        size = {"rep_of_pos": n, "degree": n, "rep_row": None}
        for name in off:
            m = size.get(name)
            assert np.array_equal(on[name][:m], off[name][:m]), (blk, name)
        assert 0 < r <= n


# back: tiles handed back in the first and in each later block (none, some or
# nearly all); skips: the last block skips tiles
@pytest.mark.parametrize("T,E,k,d,h,S1,S2,centres,mix,drift,back,skips", [
    (3000, 4, 2, 2112, 0.9, 0.8, 0.2, 300, 0.05, 0.1, ("none", "none"), False),   # rows padded to 2176 values; ragged buckets
    (2049, 4, 1, 2048, 0.9, 0.8, 0.2, 200, 0.5, 0.3, ("none", "none"), False),    # mixtures, no pair within the band
    (2049, 4, 1, 2048, 0.9, 0.72, 0.2, 200, 0.03, 0.3, ("none", "none", "some"), True),   # a few pairs of a tile at S1: one by one
    (2600, 2, 1, 2048, 0.45, 0.8, 0.2, 60, 1.0, 0.3, ("all", "all"), False),      # too many of them: tiles handed back
    (12000, 1, 1, 2048, 0.45, 0.8, 0.2, 60, 1.0, 0.3, ("all", "all"), False),     # four tiles a block, later ones without their product
    (2048, 4, 2, 4096, 0.97, 0.97, 0.97, 256, 0.1, 0.0, ("some", "none"), True),  # equal thresholds
    (1536, 3, 2, 2048, 0.9, 2.0, -2.0, 64, 0.1, 0.1, ("none", "none"), False),    # nothing is decided
    (1536, 3, 2, 2048, 0.9, -2.0, 2.0, 64, 0.1, 0.1, ("none", "none"), True),     # every shared pair is decided
    (1100, 2, 1, 2048, 0.9, np.inf, -np.inf, 64, 0.1, 0.1, ("none", "none"), False),
    (1025, 2, 1, 2048, 0.9, 0.8, 0.3, 16, 0.0, 0.0, ("none", "none"), True),      # identical blocks: every tile skipped
])
def test_forms(T, E, k, d, h, S1, S2, centres, mix, drift, back, skips):
    stack = G.make_stack("c2", 3, seed=T + d, T=T, d=d, E=E, k=k, n_centres=centres, mix_fraction=mix,
                         capacity_factor=0.0, token_drift=drift, gate_drift=drift / 4)
    print(f"[case] T={T} E={E} k={k} d={d} h={h} S1={S1} S2={S2} mix={mix} drift={drift}", flush=True)
    tiles = []
    on = _chain(stack, h, S1, S2, True, back=tiles)
    _same(on, _chain(stack, h, S1, S2, False))
    how = ["none" if n == 0 else "all" if n > 0.9 * total else "some" for n, total in tiles]
    assert how == [back[0], back[1], back[-1]], tiles
    assert on[0]["stats"][3] == 0 and (on[2]["stats"][3] > 0) == skips


@pytest.mark.parametrize("row", ["zero", "large", "small", "overflow", "underflow", "inf", "nan"])
def test_odd_rows(row):
    """Rows of zeros, of large and small norms, of finite values whose squares
    over- or underflow, and with an infinity or a NaN."""
    value = {"zero": 0.0, "large": 2.0 ** 40, "small": 2.0 ** -40, "overflow": 2.0 ** 100, "underflow": 2.0 ** -100}
    stack = G.make_stack("c2", 2, seed=3, T=1500, d=2048, E=4, k=2, n_centres=100, mix_fraction=0.1,
                         capacity_factor=0.0, token_drift=0.1, gate_drift=0.0)
    routed = copy.deepcopy(stack)
    for inp in stack:
        for t in (5, 300, 1499):
            if row in value:
                inp.x[t] *= value[row]
            else:
                inp.x[t, 17] = np.inf if row == "inf" else np.nan
    print(f"[case] row={row}", flush=True)
    tiles = []
    _same(_chain(stack, 0.9, 0.8, 0.3, True, routed, tiles), _chain(stack, 0.9, 0.8, 0.3, False, routed))
    # no bound holds for rows whose squares over- or underflow: their tiles go back
    assert [0 < n < total for n, total in tiles] == [row in ("overflow", "underflow")] * 2, tiles


def test_oracle():
    stack = G.make_stack("c2", 3, seed=9, T=1500, d=2048, E=4, n_centres=150, mix_fraction=0.1,
                         token_drift=0.2, gate_drift=0.05)
    st = run_stack(stack, h=0.9, S1=0.8, S2=0.3)
    assert st[1][0] > 0 and st[1][1] > 0
