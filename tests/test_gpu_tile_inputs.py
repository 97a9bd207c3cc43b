"""What the 16-bit attention kernels' staged tiles must not change: an
infinity in a window's last token reaches the outputs it belongs to as an
infinity, whatever the rows that pad the window's last tile hold, and tensors
that start at any element of a larger buffer give the results of aligned
ones."""

import pytest

import terra_synth as ts

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2608_15211_amd")

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16}
# (heads, hd, window, grid): windows whose token count is no multiple of 64
PADDED = [
    (2, 32, (3, 5), (9, 17)),
    (2, 64, (5, 13), (11, 26)),
    (1, 128, (5, 13), (11, 26)),
    (1, 64, (17, 16), (34, 37)),
    (11, 128, (21, 31), (42, 62)),       # the eight-wave dQ kernel: 4 windows x 11 heads x 3 chunks
]


def _inputs(dtype, heads, hd, win, grid):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = ts.small_config("tile_inputs", dtype, 1, grid[0], grid[1], heads, hd, win[0], win[1], win[0] // 2,
                          win[1] // 2, 0)
    inp = ts.make_inputs(cfg, seed=5)
    x = {n: torch.from_numpy(inp[n]).cuda().to(DTYPES[dtype]) for n in ("q", "k", "v", "dout")}
    return cfg, x, torch.from_numpy(inp["table"]).cuda()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("heads,hd,win,grid", PADDED)
def test_infinity_in_the_last_token(heads, hd, win, grid, dtype):
    cfg, x, table = _inputs(dtype, heads, hd, win, grid)
    o, lse = P.terra_winattn_fwd_nhwc(x["q"], x["k"], x["v"], table, cfg)
    dv = P.terra_winattn_bwd_nhwc(x["q"], x["k"], x["v"], o, x["dout"], lse, table, cfg)[2]
    # the last token of window (0, 0), a channel of the last head
    wh, ww = win
    c = heads * hd - 3
    u, v = (wh - 1 + wh // 2) % grid[0], (ww - 1 + ww // 2) % grid[1]
    rows = (torch.arange(wh) + wh // 2) % grid[0]
    cols = (torch.arange(ww) + ww // 2) % grid[1]
    inf = {n: x[n].clone() for n in ("v", "dout")}
    for t in inf.values():
        t[0, u, v, c] = float("inf")
    oi, _ = P.terra_winattn_fwd_nhwc(x["q"], x["k"], inf["v"], table, cfg)
    dvi = P.terra_winattn_bwd_nhwc(x["q"], x["k"], x["v"], o, inf["dout"], lse, table, cfg)[2]
    pairs = [("dV", dvi, dv)]
    if not (dtype == "bf16" and hd <= 64 and wh * ww <= 128):      # the window-resident forward
        pairs.append(("O", oi, o))
    for name, got, finite in pairs:
        want = finite.clone()
        want[0, rows[:, None].cuda(), cols.cuda(), c] = float("inf")    # every weight of the window is positive
        assert bool((got == want).all()), name


# (heads, hd, window, grid)
VIEWS = [
    (2, 32, (3, 5), (9, 17)),
    (3, 32, (12, 12), (24, 31)),
    (2, 64, (17, 16), (34, 37)),
    (2, 128, (8, 8), (16, 19)),
    (1, 128, (23, 29), (25, 33)),
]


@pytest.mark.parametrize("layout", ["nhwc", "win"])
@pytest.mark.parametrize("start", [1, 2, 4])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("heads,hd,win,grid", VIEWS)
def test_views_at_any_element(heads, hd, win, grid, dtype, start, layout):
    cfg, x, table = _inputs(dtype, heads, hd, win, grid)
    fwd, bwd = (P.terra_winattn_fwd, P.terra_winattn_bwd) if layout == "win" else \
        (P.terra_winattn_fwd_nhwc, P.terra_winattn_bwd_nhwc)
    if layout == "win":
        x = {n: P.terra_window_route(t, cfg) for n, t in x.items()}
    like = x["q"]
    use_lo = P.terra_winattn_uses_o_lo(cfg, like.dtype)

    def results(new):
        def view(t=None):
            v = new(like.numel()).view(like.shape)
            return v if t is None else v.copy_(t)
        q, k, v, dout = (view(x[n]) for n in ("q", "k", "v", "dout"))
        lo = view() if use_lo else None
        o, lse = fwd(q, k, v, table, cfg, out=view(), o_lo=lo)
        grads = bwd(q, k, v, o, dout, lse, table, cfg, out=(view(), view(), view(), torch.empty_like(table)), o_lo=lo)
        return (o, lse) + tuple(grads) + ((lo,) if use_lo else ())

    base = results(lambda n: torch.empty(n, dtype=like.dtype, device="cuda"))
    moved = results(lambda n: torch.empty(n + start, dtype=like.dtype, device="cuda")[start:])
    for i, (a, b) in enumerate(zip(base, moved)):
        assert torch.equal(a, b), i
