"""The GPU tests' cases reach the kernel forms that they are there for, by the
library's own rules (256 compute units where there is no GPU)."""

import ctypes
import os

import pytest

P = pytest.importorskip("paper_2608_15211_amd")
pytest.importorskip("torch")

import test_gpu_block_waves as block_waves  # noqa: E402
import test_gpu_dq_waves as dq_waves  # noqa: E402

pytestmark = pytest.mark.skipif(not os.path.exists(P.LIB_PATH), reason="libterra_swin.so not built")

FWD, DQ, DKDV = 0, 1, 2


def attn_waves(cfg, dtype, which):
    code = {"f32": P.TERRA_F32, "bf16": P.TERRA_BF16, "f16": P.TERRA_F16}[dtype]
    n = P.lib().terra_internal_attn_waves(ctypes.byref(P._geom(cfg)), code, which)
    assert n >= 0
    return n


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("heads,win,grid,mask", dq_waves.CASES)
def test_eight_wave_cases(heads, win, grid, mask, dtype):
    cfg = dq_waves.config(heads, win, grid, mask, dtype)
    assert [attn_waves(cfg, dtype, w) for w in (FWD, DQ, DKDV)] == [8, 8, 8]


# Both sides of the eight-wave dQ kernel's line: measured whole backwards, us,
# general kernel then eight waves (bf16, 128 channels).
LINE = [
    (8, (32, 32), (64, 64), 4),          # 157.1, 170.0
    (12, (32, 32), (64, 64), 8),         # 223.8, 177.0
    (3, (21, 31), (64, 96), 4),          # 159.7, 196.9: 9 of 16 windows are full
    (4, (21, 31), (64, 96), 8),          # 219.8, 199.3
    (2, (21, 31), (64, 200), 4),         # 169.2, 199.9
    (6, (24, 32), (60, 80), 8),          # 146.0, 129.2
    (3, (32, 32), (80, 80), 4),          # 146.2, 158.4
    (4, (32, 32), (80, 80), 8),          # 168.7, 161.8
    (12, (28, 28), (56, 56), 4),         # 25 of 32 waves busy
]


@pytest.mark.parametrize("heads,win,grid,waves", LINE)
def test_eight_wave_line(heads, win, grid, waves):
    assert attn_waves(dq_waves.config(heads, win, grid, 1, "bf16"), "bf16", DQ) == waves


def block_plans(T, C):
    """(waves, slices) of each of the block's products."""
    L = P.lib()
    product = {"qkv": (3 * C, C, 1), "proj": (C, C, 1), "fc1": (4 * C, C, 1), "fc2": (C, 4 * C, 8),
               "dln1": (C, 3 * C, 8)}
    wgrad = {"w_qkv": (3 * C, C), "w_proj": (C, C), "w_fc1": (4 * C, C), "w_fc2": (C, 4 * C)}
    out = {n: L.terra_internal_product_plan(T, *a) for n, a in product.items()}
    out.update({n: L.terra_internal_wgrad_plan(T, *a) for n, a in wgrad.items()})
    return {n: divmod(v, 100) for n, v in out.items()}


@pytest.mark.parametrize("cfg,eight", block_waves.CASES, ids=[c.name for c, _ in block_waves.CASES])
def test_eight_wave_products(cfg, eight):
    k = cfg.geom_kwargs()
    plans = block_plans(k["B"] * k["H"] * k["W"], k["C"])
    assert {n for n, (nw, _) in plans.items() if nw == 8} == set(eight)


def test_rest_of_rows_is_ragged():
    k = block_waves.CASES[-1][0].geom_kwargs()
    T, C = k["B"] * k["H"] * k["W"], k["C"]
    rows, cols = -(-T // 256), -(-C // 256)
    whole = rows * cols // 256 * 256 // cols
    assert 0 < whole < rows and T % 128 != 0 and C % 256 == 128


@pytest.mark.parametrize("C", [128, 384, 768, 1408, 1920])
def test_no_empty_contraction_slice(C):
    """Slices hold whole 64-deep stages; the last one must hold some too."""
    for T in list(range(1, 400, 13)) + list(range(400, 40000, 211)) + [2056, 138240]:
        for n, (_, slices) in block_plans(T, C).items():
            depth = T if n.startswith("w_") else {"fc2": 4 * C, "dln1": 3 * C}.get(n, C)
            stages = -(-depth // 64)
            assert (slices - 1) * -(-stages // slices) < stages, (T, n, slices)
