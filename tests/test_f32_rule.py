"""The number of wavefronts of a workgroup of the fp32 attention, for a device of 256 CUs: eight where the chip has a CU for
every item and the longest item has 32 key blocks or more.  No GPU is needed."""
import pytest

import paper_2505_18809_amd as vorta
from helpers import f32_wavefronts


def plan_of(grid, heads, tile=(3, 3, 3), window=(3, 3, 3), **kw):
    return vorta.vorta_plan_create(grid, heads, 64, "fp32", tile, window, **kw)


@pytest.mark.parametrize("grid,routes,want", [
    ((1, 16, 31), (0,), 4), ((1, 7, 71), (0,), 8),              # 496 keys, 31 blocks; 497
    ((2, 16, 31), (2,), 4), ((2, 16, 32), (2,), 8),             # 496 core-set rows; 512
    ((4, 16, 31), (1,), 4),                                     # windows of at most 729 of 1,984 keys: more items than CUs
    ((6, 12, 12), (1,), 4), ((8, 9, 9), (1,), 8),               # windows of 486 keys; of 648
    ((7, 15, 17), (0, 2), 8), ((7, 15, 17), (0, 0, 0), 4),      # 169 items, 336
    ((4, 8, 8), (0, 1, 2), 4), ((16, 16, 16), (0,), 8), ((16, 16, 16), (0, 2), 4)])
def test_eight_wavefronts_for_long_items_with_a_cu_each(grid, routes, want):
    tile = (2, 3, 3) if grid == (6, 12, 12) else (3, 3, 3)
    plan = plan_of(grid, len(routes), tile, keep_num=1, keep_den=2, bucket=(2, 1, 1))
    assert f32_wavefronts(plan, routes) == want


def test_text_rows_of_window_heads_meet_every_key():
    plan = plan_of((4, 9, 15), 1, (2, 3, 3), (1, 1, 1), n_text=16)
    assert f32_wavefronts(plan, (1,)) == 8                      # windows of 34 keys, text rows over 556
    assert f32_wavefronts(plan_of((4, 9, 15), 1, (2, 3, 3), (1, 1, 1)), (1,)) == 4
    assert f32_wavefronts(plan, (1,), units=16) == 4
