"""The eight-wave dQ kernel (16-bit types, 128 channels, windows of more than
512 tokens, more work than one round of the general kernel) and the eight-wave
forward and dK/dV that such grids take, in all their forms: quads of one
window row or single pairs, folded or single bias bins, both wrap masks,
ragged windows and odd widths, window-major and NHWC, D from O_lo or from the
kernel's own sweep; against the fp64 oracle.

The bars are those of one attention call in 16-bit storage (max abs 2e-2,
relative L2 5e-3) and hold for fp16 a fortiori."""

import numpy as np
import pytest

import terra_synth as ts
from oracle import Geometry, attn_bwd, attn_fwd, route, unroute

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2608_15211_amd")

# (heads, window, grid, mask)
CASES = [
    (9, (32, 32), (64, 64), 1),          # quads, folded bins
    (9, (32, 32), (64, 64), 3),          # pairs, folded bins
    (11, (21, 31), (45, 62), 3),         # pairs, single bins, a short last row of windows
    (12, (24, 32), (50, 70), 1),         # ragged both ways, last column's width no multiple of 4
]


def config(heads, win, grid, mask, dtype):
    return ts.small_config("dq_waves", dtype, 1, grid[0], grid[1], heads, 128, win[0], win[1], win[0] // 2,
                           win[1] // 2, mask)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("heads,win,grid,mask", CASES)
def test_eight_wave_backward(heads, win, grid, mask, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = config(heads, win, grid, mask, dtype)
    g = Geometry(**cfg.geom_kwargs())
    inp = ts.make_inputs(cfg, seed=4)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float16
    x = {n: torch.from_numpy(inp[n]).cuda().to(tdt) for n in ("q", "k", "v", "dout")}
    table = torch.from_numpy(inp["table"]).cuda()
    r = {n: route(inp[n], g) for n in ("q", "k", "v", "dout")}
    ref = attn_bwd(r["q"], r["k"], r["v"], r["dout"], inp["table"], g)
    ro, _ = attn_fwd(r["q"], r["k"], r["v"], inp["table"], g)
    ref = dict(zip(("O", "dQ", "dK", "dV", "dT"), (ro,) + tuple(ref)))
    for layout in ("nhwc", "win"):
        fwd, bwd = (P.terra_winattn_fwd, P.terra_winattn_bwd) if layout == "win" else \
            (P.terra_winattn_fwd_nhwc, P.terra_winattn_bwd_nhwc)
        t = x if layout == "nhwc" else {n: P.terra_window_route(a, cfg) for n, a in x.items()}
        for lo in (None, torch.empty_like(t["q"])):
            o, lse = fwd(t["q"], t["k"], t["v"], table, cfg, o_lo=lo)
            got = bwd(t["q"], t["k"], t["v"], o, t["dout"], lse, table, cfg, o_lo=lo)
            for n, a in zip(("O", "dQ", "dK", "dV", "dT"), (o,) + tuple(got)):
                b = ref[n] if n == "dT" or layout == "win" else unroute(ref[n], g)
                a = a.float().cpu().numpy().astype(np.float64)
                b = np.asarray(b).reshape(a.shape)
                what = "%s %s %s" % (n, layout, "sweep" if lo is None else "O_lo")
                assert np.abs(a - b).max() <= 2e-2, what
                assert np.linalg.norm(a - b) <= 5e-3 * np.linalg.norm(b), what
