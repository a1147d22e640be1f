"""Glue shared by the tests: config -> oracle spec, tensor -> fp64 array."""
import ctypes

import numpy as np
import torch

import paper_2505_18809_amd as vorta
from oracle import vorta_oracle as vo
from synth_inputs import LayerConfig


def spec_of(cfg: LayerConfig, **over) -> vo.LayerSpec:
    kw = dict(grid=cfg.grid, tile=cfg.tile, window=cfg.window, bucket=cfg.bucket,
              keep_num=cfg.keep_num, keep_den=cfg.keep_den, n_text=cfg.n_text,
              rope_dims=cfg.rope_dims, rope_theta=cfg.rope_theta)
    kw.update(over)
    return vo.LayerSpec(**kw)


def f64(t) -> np.ndarray:
    """Widen a (possibly bf16, possibly device) tensor to an fp64 NumPy array."""
    if isinstance(t, torch.Tensor):
        return t.detach().to("cpu", torch.float64).numpy()
    return np.asarray(t, dtype=np.float64)


def smooth_field(rng, grid, d, noise=0.5):
    """A small correlated field for oracle tests (not the benchmark recipe):
    cumulative-sum smoothing keeps neighbours similar without any library."""
    F, H, W = grid
    x = rng.standard_normal((F, H, W, d))
    x = x + np.roll(x, 1, 0) + np.roll(x, 1, 1) + np.roll(x, 1, 2)
    x = x / x.std() + noise * rng.standard_normal((F, H, W, d))
    return x.reshape(F * H * W, d)


# Forms of a bf16 attention launch (an internal hook of the library): 0 = the library's own choice; split kernel
# with two or four key shares; pipelined kernels; pipelined with the window rows on the split kernel, and with all
# of them in 128-row items.
SPLIT2, SPLIT4, PIPE, PIPE_SPLIT_WIN, PIPE_WIN_128 = 2, 4, 3, 5, 6


def force_form(plan, form, halves=-1):
    """All attention launches of the plan take this form; halves: items issued as half-row items, -1 = the rule's."""
    assert vorta.load_library().vorta_test_force_form(plan.handle, ctypes.c_int32(form), ctypes.c_int32(halves)) == 0
    return plan


def attention_form(plan, routes, mix=False, units=256):
    """What the library chooses for a layer call with these routes on a device of `units` CUs."""
    r = np.ascontiguousarray(routes, dtype=np.uint8)
    out = np.zeros(9, dtype=np.int32)
    assert vorta.load_library().vorta_test_form(plan.handle, r.ctypes.data_as(ctypes.c_void_p), ctypes.c_int32(mix),
                                                ctypes.c_int32(units), out.ctypes.data_as(ctypes.c_void_p)) == 0
    return dict(zip(("split_all", "shares", "split_win", "together", "n_long", "half_long", "n_big", "half_big", "win_128"), map(int, out)))


def round_shift(plan, routes, window_only=False, units=256):
    """The item that a split launch of two key shares begins with, of a layer call or of its window rows alone."""
    r = np.ascontiguousarray(routes, dtype=np.uint8)
    out = ctypes.c_int32()
    assert vorta.load_library().vorta_test_round_shift(plan.handle, r.ctypes.data_as(ctypes.c_void_p), ctypes.c_int32(window_only),
                                                       ctypes.c_int32(units), ctypes.byref(out)) == 0
    return out.value


def window_list(plan, which):
    """The window items of a list, 16 numbers each: first place, rows, the numbers of the keys, zeros."""
    lib, n = vorta.load_library(), ctypes.c_int32()
    assert lib.vorta_test_window_list(plan.handle, ctypes.c_int32(which), None, ctypes.byref(n)) == 0
    out = np.empty((n.value, 16), dtype=np.int32)
    assert lib.vorta_test_window_list(plan.handle, ctypes.c_int32(which), out.ctypes.data_as(ctypes.c_void_p), ctypes.byref(n)) == 0
    return out


def select_form(plan, routes, layer=False, units=256):
    """How the one-pass selection is cut, called alone or in a layer call; False where the plan's buckets are selected and
    pooled in separate passes."""
    r = np.ascontiguousarray(routes, dtype=np.uint8)
    out = np.zeros(4, dtype=np.int32)
    assert vorta.load_library().vorta_test_select_form(plan.handle, r.ctypes.data_as(ctypes.c_void_p), ctypes.c_int32(layer),
                                                       ctypes.c_int32(units), out.ctypes.data_as(ctypes.c_void_p)) == 0
    return dict(zip(("apart", "bucket_blocks", "text_blocks", "turn_blocks"), map(int, out))) if out[1] else False


def f32_wavefronts(plan, routes, units=256):
    """Wavefronts of a workgroup of the fp32 attention launch of a layer call."""
    r = np.ascontiguousarray(routes, dtype=np.uint8)
    out = ctypes.c_int32()
    assert vorta.load_library().vorta_test_f32_wavefronts(plan.handle, r.ctypes.data_as(ctypes.c_void_p), ctypes.c_int32(units),
                                                          ctypes.byref(out)) == 0
    return out.value
