"""The block's eight-wave products with ragged edges: token counts and widths
that leave partial 256 x 256 tiles (bounds-checked epilogues, operand rows and
columns outside the matrix, partial rows of the dh column sums), a rest of
rows past whole rounds, weight gradients over few and many tokens, dW_qkv in
thirds; against the fp64 oracle with the block's bars."""

import pytest

import terra_synth as ts
from test_gpu_block import P, _check, _gpu  # noqa: F401  (the fixture skips without a GPU)

# Config and the products that take eight waves.
CASES = [
    (ts.small_config("waves_c384", "bf16", 1, 49, 110, 12, 32, 7, 10, 3, 5), ("fc1",)),
    (ts.small_config("waves_c1152", "bf16", 1, 79, 91, 9, 128, 8, 8, 4, 4),
     ("qkv", "proj", "fc1", "fc2", "dln1", "w_fc1", "w_fc2")),
    (ts.small_config("waves_c1920", "bf16", 1, 14, 15, 60, 32, 7, 5, 3, 2), ("w_fc1", "w_fc2", "w_qkv")),
    # fc2 and dln1: 42 of 43 row tiles in whole rounds of eight waves, the rest in four
    (ts.small_config("waves_c1408", "bf16", 1, 83, 131, 11, 128, 8, 8, 4, 4),
     ("qkv", "fc1", "w_fc1", "w_fc2", "w_qkv")),
]


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [c for c, _ in CASES], ids=[c.name for c, _ in CASES])
def test_block_eight_waves(cfg):
    _check(cfg, seed=3)
