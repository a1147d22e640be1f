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


def test_buckets_that_no_instance_holds_have_no_form():
    assert select_form(plan_of((3, 3, 3), 2, "fp32", 128), (2, 2)) is False
    assert select_form(plan_of((4, 3, 3), 2), (2, 2)) is False
