"""16-bit dK/dV kernel at the edges of its plan: fewer keys than one wave,
two, three and four waves a workgroup, a window one token past a 64-token
tile, chunks whose last waves own no key, windows whose LDS plan fits a CU once
(four waves on grids this small), widths that are and are not multiples of 4, both wrap
masks; bf16 and fp16, both layouts, against the fp64 oracle.

The bars are those of one attention call in 16-bit storage (max abs 2e-2,
relative L2 5e-3) and hold for fp16 a fortiori."""

import numpy as np
import pytest

import terra_synth as ts
from oracle import Geometry, attn_bwd, attn_fwd, route, unroute

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2608_15211_amd")

pytestmark = pytest.mark.gpu

# (heads, hd, window, grid, mask)
CASES = [
    (2, 32, (3, 5), (9, 17), 1),         # 15 tokens: half of one wave
    (2, 32, (8, 8), (16, 24), 3),        # two waves
    (1, 32, (5, 13), (11, 26), 3),       # 65 tokens: one past a tile; three waves
    (3, 64, (9, 11), (20, 25), 1),       # 99 tokens, odd widths
    (2, 64, (17, 16), (34, 37), 1),      # 272 tokens: the last chunk owns 16 keys
    (1, 64, (24, 24), (30, 41), 3),      # 576 tokens, ragged both ways
    (2, 128, (8, 8), (16, 19), 1),       # two waves at 128 channels
    (1, 128, (23, 29), (25, 33), 1),     # 667 tokens, odd width
    (1, 128, (32, 32), (40, 48), 1),     # 1024 tokens
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("heads,hd,win,grid,mask", CASES)
def test_backward_edges(heads, hd, win, grid, mask, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wh, ww = win
    cfg = ts.small_config("tiles", dtype, 2 if wh * ww < 100 else 1, grid[0], grid[1], heads, hd, wh, ww,
                          wh // 2, ww // 2, mask)
    g = Geometry(**cfg.geom_kwargs())
    inp = ts.make_inputs(cfg, seed=3)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float16
    x = {n: torch.from_numpy(inp[n]).cuda().to(tdt) for n in ("q", "k", "v", "dout")}
    table = torch.from_numpy(inp["table"]).cuda()
    o, lse = P.terra_winattn_fwd_nhwc(x["q"], x["k"], x["v"], table, cfg)
    got = P.terra_winattn_bwd_nhwc(x["q"], x["k"], x["v"], o, x["dout"], lse, table, cfg)
    w = {n: P.terra_window_route(t, cfg) for n, t in x.items()}
    ow, lw = P.terra_winattn_fwd(w["q"], w["k"], w["v"], table, cfg)
    gotw = P.terra_winattn_bwd(w["q"], w["k"], w["v"], ow, w["dout"], lw, table, cfg)
    torch.cuda.synchronize()
    r = {n: route(inp[n], g) for n in ("q", "k", "v", "dout")}
    ref = attn_bwd(r["q"], r["k"], r["v"], r["dout"], inp["table"], g)
    ro, _ = attn_fwd(r["q"], r["k"], r["v"], inp["table"], g)
    host = lambda t: t.float().cpu().numpy().astype(np.float64)  # noqa: E731
    pairs = [("O", host(o), unroute(ro, g))]
    for n, a, b, c in zip(("dQ", "dK", "dV", "dT"), got, gotw, ref):
        pairs.append((n, host(a), c if n == "dT" else unroute(c, g)))
        pairs.append((n + " window-major", host(b), c))
    for n, a, b in pairs:
        b = np.asarray(b).reshape(a.shape)
        assert np.abs(a - b).max() <= 2e-2, n
        assert np.linalg.norm(a - b) <= 5e-3 * np.linalg.norm(b), n
