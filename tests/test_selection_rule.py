"""The rule by which the one-pass selection gives each tensor of a bucket a wavefront of its own, for a device of 256 CUs.
No GPU is needed."""
import pytest

import paper_2505_18809_amd as vorta
from helpers import select_form


def plan_of(bucket, heads, dtype="bf16", d=128, rope=False, grid=None, n_text=0):
    """Two buckets along each axis unless a grid is given: 8 (bucket, head) pairs for every head on route 2."""
    dims = ((44, 42, 42) if d == 128 else (16, 24, 24)) if rope else (0, 0, 0)
    return vorta.vorta_plan_create(grid or tuple(2 * b for b in bucket), heads, d, dtype, (4, 4, 4), (3, 3, 3), bucket=bucket,
                                   keep_num=2, keep_den=3, rope_dims=dims, n_text=n_text)


@pytest.mark.parametrize("bucket,dtype,d,rope,most", [
    ((2, 3, 2), "bf16", 128, False, 336), ((2, 3, 2), "bf16", 128, True, 336), ((4, 2, 2), "bf16", 128, True, 336),
    ((3, 3, 3), "bf16", 128, False, 336), ((2, 3, 2), "fp32", 64, True, 336), ((4, 2, 2), "fp32", 64, True, 336),
    ((2, 3, 2), "fp32", 128, False, 336), ((4, 2, 2), "fp32", 128, False, 336),
    # rotated rows in more than four passes, which look the rotation up pass by pass: rows of 32 chunks among them
    ((3, 3, 3), "bf16", 128, True, 576), ((3, 3, 3), "fp32", 64, True, 576),
    ((2, 3, 2), "fp32", 128, True, 576), ((4, 2, 2), "fp32", 128, True, 576)])
def test_a_wavefront_for_each_tensor_up_to_so_many_pairs(bucket, dtype, d, rope, most):
    for pairs, apart in ((8, 1), (most, 1), (most + 8, 0), (1024, 0)):
        plan = plan_of(bucket, pairs // 8, dtype, d, rope)
        assert plan.n_buckets == 8
        assert select_form(plan, (2,) * (pairs // 8))["apart"] == apart, pairs
    plan = plan_of(bucket, most // 8, dtype, d, rope)
    assert select_form(plan, (2,) * (most // 8), units=128)["apart"] == 0


@pytest.mark.parametrize("grid,bucket,routes,rope,alone,layer", [
    ((8, 16, 16), (2, 3, 2), (0, 8, 1), True, 1, 1),          # 400 workgroups, 8 heads turned
    ((8, 16, 16), (2, 3, 2), (4, 20, 1), True, 1, 0),         # 24 heads: each turning workgroup is the longest of the launch
    ((12, 16, 16), (2, 3, 2), (0, 6, 1), True, 1, 1), ((12, 16, 16), (2, 3, 2), (1, 22, 1), True, 1, 0),
    ((12, 16, 16), (3, 3, 3), (1, 22, 1), True, 1, 1),        # the buckets take longer than 23 heads
    ((12, 16, 16), (2, 3, 2), (1, 22, 1), False, 1, 1),       # nothing is turned
    ((16, 16, 16), (4, 2, 2), (0, 2, 1), True, 1, 1), ((16, 16, 16), (4, 2, 2), (2, 10, 1), True, 1, 0),
    ((16, 24, 24), (3, 3, 3), (0, 8, 1), True, 1, 0),         # 1,440 workgroups
    ((4, 8, 8), (2, 3, 2), (0, 39, 1), True, 1, 1)])
def test_turned_rows_in_the_same_launch_count(grid, bucket, routes, rope, alone, layer):
    heads = sum(routes)
    plan = plan_of(bucket, heads, rope=rope, grid=grid)
    r = (0,) * routes[0] + (1,) * routes[1] + (2,) * routes[2]
    one, whole = select_form(plan, r), select_form(plan, r, layer=True)
    assert (one["apart"], whole["apart"]) == (alone, layer)
    rows = grid[0] * grid[1] * grid[2]
    assert one["turn_blocks"] == 0 and whole["turn_blocks"] == (2 * rows // 16 if rope else 0)


def test_text_rows_count_and_core_set_heads_alone_turn_nothing():
    few, many = (plan_of((2, 3, 2), 1, n_text=n) for n in (77, 20000))
    assert select_form(few, (2,))["apart"] == 1 and select_form(few, (2,))["text_blocks"] == 5
    assert select_form(many, (2,))["apart"] == 0
    assert select_form(plan_of((2, 3, 2), 3, rope=True), (2, 2, 2), layer=True) == {"apart": 1, "bucket_blocks": 2, "text_blocks": 0, "turn_blocks": 0}


def test_buckets_that_no_instance_holds_have_no_form():
    assert select_form(plan_of((3, 3, 3), 2, "fp32", 128), (2, 2)) is False
    assert select_form(plan_of((4, 3, 3), 2), (2, 2)) is False
