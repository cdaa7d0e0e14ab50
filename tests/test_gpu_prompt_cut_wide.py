"""Prompts cut along K (tile_rules.hpp: prompt_k_ranges) of layers that are not taken in one launch (prompt_step.hip): wider than 1024 columns,
or more than 4096 feed-forward ones, on either side of the row limits."""
import pytest

from tests import test_gpu_prompt_cut as cut

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,ffn,lens", [
    (1152, 18, 1152, [17]),                  # uneven ranges: the 64-row tile, K is no multiple of 256
    (1152, 9, 2432, [40, 1, 23]),            # 64 rows
    (1088, 17, 4352, [33]),                  # hidden an odd multiple of 64
    (768, 12, 4224, [64, 1]),                # 65: the output projection below the floor
    (1280, 10, 2688, [100, 28]),             # 128
    (512, 8, 4608, [129]),                   # two row tiles
    (1152, 18, 4608, [200, 57]),             # 257: not cut this way
])
@pytest.mark.parametrize("left", [False, True])
def test_prompt(hidden, heads, ffn, lens, left):
    cut.test_prompt(hidden, heads, ffn, lens, left)
