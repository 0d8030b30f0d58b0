"""The float32 MFMA kernels at the edges of their tiles: the grouped FFN's two
tile shapes, the 64 x 64 similarity tiles and the gate's 16-token blocks,
against the oracle.  float32 sums of K products of independent terms are
within a few sqrt(K) * 2^-24 of the exact sum (below 1e-5 for K <= 8192)."""
import numpy as np
import pytest

import luffy_gen as G
from oracle import luffy_oracle as O
from tests.layer_runner import (TOL, assert_condense_equal, assert_output_close, assert_route_equal, fetch,
                                rel_err_rows, run_gpu, run_oracle)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_15419_amd as L
    L.load_library()


EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 0, 200]
# (512, 8192): the first product has enough 64 x 64 tiles for two a CU, the
# second splits K over the waves in 32 x 32 tiles; (64, 64): two K chunks for
# four waves; (192, 4160): chunk counts that four does not divide
@pytest.mark.parametrize("d,d_ff,act,offset", [(64, 64, "gelu", 0), (192, 4160, "silu", 0), (512, 8192, "gelu", 0),
                                               (256, 1024, "silu", 1), (512, 8192, "gelu", 1)])
def test_expert_ffn_f32_tiles(d, d_ff, act, offset):
    """Expert sizes around both tile edges, rows through a row index; with
    `offset` every operand starts 4 bytes past a 16-byte boundary."""
    import torch
    import paper_2411_15419_amd as L
    print(f"[case] expert_ffn f32 d={d} d_ff={d_ff} act={act} offset={offset}", flush=True)
    E, R = len(EDGES), sum(EDGES)
    rng = np.random.default_rng(d + d_ff)
    x = rng.standard_normal((R + 9, d)).astype(np.float32)
    idx = rng.permutation(R + 9)[:R].astype(np.int32)
    w1 = (0.05 * rng.standard_normal((E, d_ff, d))).astype(np.float32)
    w2 = (0.05 * rng.standard_normal((E, d, d_ff))).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(EDGES)]).astype(np.int32)

    def dev(a):
        buf = torch.zeros(a.size + offset, dtype=torch.float32, device="cuda")
        buf[offset:] = torch.from_numpy(a.reshape(-1)).cuda()
        return buf[offset:].view(a.shape)

    y = dev(np.full((R + 3, d), np.nan, np.float32))
    ws = torch.empty(L.expert_ffn_workspace_size(R, E, d_ff, L.LUFFY_F32), dtype=torch.uint8, device="cuda")
    L.luffy_expert_ffn(dev(x), torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda(), dev(w1), dev(w2), act, R,
                       y, ws)
    got = y.double().cpu().numpy()
    assert np.isnan(got[R:]).all(), "rows past the last representative were written"
    err, _ = rel_err_rows(got[:R], O.expert_ffn(x[idx].astype(np.float64), off, w1, w2, act))
    assert err.max() <= TOL["f32"], f"max row rel err {err.max():.3g}"


@pytest.mark.parametrize("T,E,k,d", [(1, 2, 1, 64), (17, 3, 2, 64), (130, 1, 1, 192), (1000, 33, 2, 128),
                                     (8200, 64, 2, 64), (32800, 20, 1, 64)])
def test_layer_f32_sizes(T, E, k, d):
    """Whole float32 layers whose buckets cross the 64-row similarity tiles
    and whose token counts cross the gate's 16-, 32- and 64-token blocks."""
    inp = G.make_inputs("c1", seed=T, T=T, E=E, k=k, d=d, d_ff=128, n_centres=max(1, T // 6))
    print(f"[case] layer f32 T={T} E={E} k={k} d={d}", flush=True)
    g = run_gpu(inp)
    o = run_oracle(inp)
    assert_route_equal(g, o)
    assert_condense_equal(g, o)
    assert_output_close(g, o, "f32")


@pytest.mark.parametrize("T,E,k,d", [(130, 2, 1, 192), (1000, 5, 2, 128), (8200, 16, 1, 64)])
def test_layer_f32_unaligned(T, E, k, d):
    """Tokens, gate and expert weights that start 4, 8 and 12 bytes past a 16-byte
    boundary: the gate's vector loads and the similarity tiles' 16-byte DMA."""
    import torch
    import paper_2411_15419_amd as L
    inp = G.make_inputs("c1", seed=T + 1, T=T, E=E, k=k, d=d, d_ff=128, n_centres=max(1, T // 6))
    print(f"[case] layer f32 unaligned T={T} E={E} k={k} d={d}", flush=True)

    def dev(a, offset):
        buf = torch.zeros(a.size + offset, dtype=torch.float32, device="cuda")
        buf[offset:] = torch.from_numpy(a.astype(np.float32).reshape(-1)).cuda()
        return buf[offset:].view(a.shape)

    o = run_oracle(inp)
    for offset in (1, 2, 3):
        x = dev(inp.x, offset)
        layer = L.MoELayer(dev(inp.w_g, offset), dev(inp.b_g, 1), dev(inp.w1, offset), dev(inp.w2, offset), k=k,
                           act=inp.cfg.act, threshold=inp.cfg.h, capacity_factor=inp.cfg.capacity_factor, T=T)
        layer(x)
        g = fetch(layer)
        assert_route_equal(g, o)
        assert_condense_equal(g, o)
        assert_output_close(g, o, "f32")


def test_expert_ffn_f32_rows_past_4_gib():
    """x of more than 4 GiB (no limit is set on it): rows at offsets that 32 bits
    do not hold, on the tile shape that reads rows at 32-bit offsets (512 tiles
    and more)."""
    import torch
    import paper_2411_15419_amd as L
    d, d_ff, R, T = 1024, 4096, 500, (1 << 20) + 4096
    print(f"[case] expert_ffn f32 T={T} d={d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(0)
    x = torch.zeros(T, d, device="cuda")
    idx = torch.randint(0, 1 << 20, (R,), generator=gen, device="cuda")
    idx[::7] = torch.arange(T - idx[::7].numel(), T, device="cuda")
    x[idx] = torch.randn(R, d, generator=gen, device="cuda")
    w1 = 0.02 * torch.randn(1, d_ff, d, generator=gen, device="cuda")
    w2 = 0.02 * torch.randn(1, d, d_ff, generator=gen, device="cuda")
    y = torch.empty(R, d, device="cuda")
    ws = torch.empty(L.expert_ffn_workspace_size(R, 1, d_ff, L.LUFFY_F32), dtype=torch.uint8, device="cuda")
    L.luffy_expert_ffn(x, idx.int(), torch.tensor([0, R], dtype=torch.int32, device="cuda"), w1, w2, "silu", R, y, ws)
    z = x[idx].double() @ w1[0].double().t()
    ref = (z * torch.sigmoid(z)) @ w2[0].double().t()
    err, _ = rel_err_rows(y.double().cpu().numpy(), ref.cpu().numpy())
    assert err.max() <= TOL["f32"], f"max row rel err {err.max():.3g}"
