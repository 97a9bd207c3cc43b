"""The block at the edges of its product plans: fewer tokens than one tile,
contraction slices with a short last one, a width whose three-part operand
takes 128-row tiles only, and token counts that leave ragged tiles; against
the fp64 oracle with the block's bars."""

import pytest

import terra_synth as ts
from test_gpu_block import P, _check, _gpu  # noqa: F401  (the fixture skips without a GPU)

pytestmark = pytest.mark.gpu

CASES = [
    ts.small_config("forms_35", "bf16", 1, 5, 7, 4, 32, 5, 7, 2, 3),
    ts.small_config("forms_c384", "bf16", 1, 37, 41, 3, 128, 8, 8, 4, 4),
    ts.small_config("forms_c256", "bf16", 2, 33, 41, 8, 32, 8, 16, 4, 8),
    ts.small_config("forms_c1152", "bf16", 1, 13, 20, 9, 128, 13, 10, 0, 0),
    ts.small_config("forms_t4100", "bf16", 1, 41, 100, 4, 32, 4, 4, 2, 2),
]


@pytest.mark.parametrize("cfg", CASES, ids=[c.name for c in CASES])
def test_block_forms(cfg):
    _check(cfg, seed=2)
