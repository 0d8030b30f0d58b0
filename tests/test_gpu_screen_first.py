"""The similarity screen's two phases and its pair-by-pair decisions: a screened
luffy_condense must give the outputs of the all-bf16 call bit for bit, whichever
way a tile is decided (after the first values of the rows, after all of them,
pair by pair on fp8 or bf16 rows, or handed back)."""
import numpy as np
import pytest

import luffy_gen as G
from tests.layer_runner import fetch, make_layer, screen_state, upload
from tests.test_gpu_screen import _assert_same, _near_threshold_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_15419_amd as L
    L.load_library()


def _run(inp, screen, h, dev):
    """The call's outputs, and with the screen on what it left in its workspace."""
    import paper_2411_15419_amd as L
    was = L.set_similarity_screen(screen)
    try:
        assert L.similarity_screen_applies(inp.cfg.T, inp.cfg.d, inp.cfg.E, inp.cfg.k) == screen
        layer = make_layer(inp, dev, h)
        layer.route(dev["x"])
        layer.condense(dev["x"])
        out = fetch(layer, with_ffn=False)
        return (out, screen_state(layer)) if screen else out
    finally:
        L.set_similarity_screen(was)


def _first_values(d, h):
    """Values of the first phase: the fewest (of whole 128) that leave unrelated
    pairs below h minus what rows keep beyond them, or all of them."""
    for da in range(128, d // 2 + 1, 128):
        f = da / d
        if h - (1.0 - f) >= 0.02 + 0.05 * f ** 0.5 + 6.0 * (f / d) ** 0.5:
            return da
    return d


def _wave_pairs(out, state, d, h):
    """Per tile the most pairs that the first values of the rows leave in a wave's
    part (128 x 64) of it, from the call's own fp8 rows and bounds."""
    import torch
    da = _first_values(d, h)
    x = state["x8"][:, :da].view(torch.float8_e4m3fn).float() / 256.0
    q = state["rowq"]
    most = []
    for lo, hi in zip(out["offsets"][:-1], out["offsets"][1:]):
        tok = torch.from_numpy(out["perm_token"][lo:hi].astype(np.int64)).cuda()
        for a in range(0, hi - lo, 256):
            for b in range(a, hi - lo, 256):
                P, Q = tok[a:a + 256], tok[b:b + 256]
                rho = float(torch.maximum(q[P, 1].max(), q[Q, 1].max()))
                thr = h - (2 * rho + rho * rho + 4e-3) - float(q[P, 2].max() * q[Q, 2].max())
                hit = x[P] @ x[Q].t() >= thr
                if a == b:
                    hit = torch.triu(hit, 1)
                full = torch.zeros(256, 256, device="cuda")
                full[:hit.shape[0], :hit.shape[1]] = hit
                most.append(float(full.view(2, 128, 4, 64).sum((1, 3)).max()))
    return np.array(most)


def _some(n, total):
    return "none" if n == 0 else "all" if n == total else "some"


@pytest.mark.parametrize("T,E,k,d,h,n_centres,goes_on,back", [
    (2600, 2, 1, 2048, 0.9, 2000, "none", "none"),     # few pairs: every tile decided pair by pair
    (3000, 4, 2, 2112, 0.9, 300, "some", "none"),      # rows padded to 2176 values; ragged buckets
    (2600, 2, 1, 2048, 0.9, 4, "all", "none"),         # dense groups: every tile goes on to phase 2
    (2600, 2, 1, 2048, 0.9, 60, "all", "none"),        # about 180 pairs a wave
    (4096, 4, 2, 2048, 0.45, 512, None, "none"),       # a threshold whose first phase would be most of the row: one phase
    (2048, 4, 2, 4096, 0.97, 256, "some", "some"),     # the band reaches some groups' cosines
    (2049, 4, 1, 8192, 0.9, 300, "some", "none"),      # one row past a tile
    (9000, 1, 1, 2048, 0.9, 400, "some", "none"),      # two or three tiles a block, some of which go on
    (17000, 1, 1, 2048, 0.9, 100, "all", "none"),      # nine tiles a block, all of which go on: whole tiles, then a new try
])
def test_phases(T, E, k, d, h, n_centres, goes_on, back):
    """goes_on: tiles with more than 32 pairs left in a wave after the first values
    (one-phase calls: None); back: tiles handed back."""
    inp = G.make_inputs("c3", seed=d + n_centres, weights=False, T=T, E=E, k=k, d=d, n_centres=n_centres)
    inp.x[7] = 0.0                   # a zero row joins nothing
    inp.x[11] *= 2.0 ** 40
    inp.x[13] *= 2.0 ** -40
    print(f"[case] T={T} E={E} k={k} d={d} h={h} centres={n_centres}", flush=True)
    dev = upload(inp)
    on, state = _run(inp, True, h, dev)
    _assert_same(on, _run(inp, False, h, dev))
    assert on["degree"].max() > 0
    assert _some(state["listed"].size, state["total"]) == back
    if goes_on is None:
        assert _first_values(d, h) == d
    else:
        assert _first_values(d, h) < d
        assert _some((_wave_pairs(on, state, d, h) > 32).sum(), state["total"]) == goes_on


@pytest.mark.parametrize("near,back", [(24, "some"), (200, "some"), (1200, "all")])
def test_close_pairs_one_by_one(near, back):
    """A few, some and many tokens whose cosines with each other cover the
    threshold, among tight groups: pairs left within the band get their bf16
    dot product, and tiles with too many of them are handed back."""
    T, d, h = 2400, 2048, 0.9
    inp = _near_threshold_inputs(T, d, h, 5)
    rng = np.random.default_rng(near)
    # keep `near` of the first half's tokens, the others i.i.d.
    x = inp.x.copy()
    x[near:T // 2] = rng.standard_normal((T // 2 - near, d)).astype(np.float32)
    inp.x = G.round_bf16(x)[rng.permutation(T)]
    print(f"[case] near={near}", flush=True)
    dev = upload(inp)
    on, state = _run(inp, True, h, dev)
    _assert_same(on, _run(inp, False, h, dev))
    assert _some(state["listed"].size, state["total"]) == back


@pytest.mark.parametrize("tail", ["full", "zero"])
@pytest.mark.parametrize("row", ["zero", "large", "small", "overflow", "underflow", "inf", "nan"])
def test_odd_rows(row, tail):
    """Rows of zeros, of large and small norms, of finite values whose squares
    over- or underflow (no bound holds for them), and with an infinity or a NaN,
    among ordinary rows; with `tail` zero every row is zero past the values of
    the first phase (512 of 2048 at h = 0.9)."""
    import copy
    import paper_2411_15419_amd as L
    value = {"zero": 0.0, "large": 2.0 ** 40, "small": 2.0 ** -40, "overflow": 2.0 ** 100, "underflow": 2.0 ** -100}
    inp = G.make_inputs("c3", seed=1, weights=False, T=1100, E=1, k=1, d=2048, n_centres=200)
    if tail == "zero":
        inp.x[:, 512:] = 0.0
    odd = copy.deepcopy(inp)
    for t in (5, 700):
        if row in value:
            odd.x[t] *= value[row]
        else:
            odd.x[t, 17] = np.inf if row == "inf" else np.nan
    print(f"[case] row={row} tail={tail}", flush=True)
    clean, dev = upload(inp), upload(odd)
    got = []
    for screen in (True, False):
        was = L.set_similarity_screen(screen)
        try:
            layer = make_layer(odd, dev, 0.9, norms_from_route=False)
            layer.route(clean["x"])
            layer.condense(dev["x"])
            got.append(fetch(layer, with_ffn=False))
        finally:
            L.set_similarity_screen(was)
    _assert_same(*got)
    assert got[0]["degree"].max() > 0


def _launches(kernel, call):
    import torch
    import paper_2411_15419_amd as L
    L.profile_kernel(kernel)
    try:
        call()
        torch.cuda.synchronize()
        return L.profile_read()[1]
    finally:
        L.profile_kernel(None)


@pytest.mark.parametrize("h,S1,S2,screened", [
    (0.9, 0.8, 0.2, True), (0.13, 0.8, 0.2, True), (0.9, 0.8, -0.2, True), (0.9, np.inf, -np.inf, True),
    (0.12, 0.8, 0.2, False), (0.9, 0.8, 0.1, False), (0.9, -0.1, 0.2, False), (0.9, 0.8, 0.0, False),
])
def test_thresholds_among_unrelated_cosines(h, S1, S2, screened):
    """Calls with a threshold among the cosines of unrelated tokens (within 0.06 +
    3 / sqrt(2048) = 0.126 of 0) keep the bf16 kernels; outputs do not depend on
    it.  Plain calls go by h alone."""
    import paper_2411_15419_amd as L
    inp = G.make_inputs("c3", seed=2, weights=False, T=1500, E=2, k=1, d=2048, n_centres=300)
    dev = upload(inp)
    plain = make_layer(inp, dev, h)
    hist = L.MoELayer(plain.w_gate, plain.b_gate, plain.w1, plain.w2, k=1, act=inp.cfg.act, threshold=h,
                      capacity_factor=inp.cfg.capacity_factor, T=1500, history=(S1, S2))
    print(f"[case] h={h} S1={S1} S2={S2}", flush=True)
    out = {}
    for on in (True, False):
        was = L.set_similarity_screen(on)
        try:
            for name, layer in (("plain", plain), ("hist", hist)):
                layer.route(dev["x"])
                if name == "hist":
                    layer.record.zero_()
                n = _launches("gram_recheck", lambda: layer.condense(dev["x"]))
                want = on and (h >= 0.126 if name == "plain" else screened)
                assert n == want, (name, on, n)
                g = fetch(layer, with_ffn=False)
                if name == "hist":
                    g["record"] = layer.record.cpu().numpy()
                out[name, on] = g
        finally:
            L.set_similarity_screen(was)
    for name in ("plain", "hist"):
        _assert_same(out[name, True], out[name, False])
    assert np.array_equal(out["hist", True]["record"], out["hist", False]["record"])
