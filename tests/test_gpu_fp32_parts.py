"""fp32 convolutions whose products run on the bf16 matrix instructions in three parts per operand: as exact as fp32
arithmetic against float64, over the whole exponent range in which the third part is representable; and the kernel that
takes 64 x 64 tiles per wave at the edges of its tiles, taps, K slices and wave counts."""
import time

import numpy as np
import pytest
import torch

import paper_2504_08795_amd as D
import workloads as wl
from gpu_helpers import GpuNet

pytestmark = pytest.mark.gpu
N = wl.nets


def _conv(cin, h, w, cout, k, s, p, scale_x=1.0, scale_w=1.0, plan_cus=0, seed=3):
    rng = np.random.default_rng(seed)
    L = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=0, in_from=-1)]
    wt = (rng.normal(0, np.sqrt(2.0 / (cin * k * k)), (cout, cin, k, k)) * scale_w).astype(np.float32)
    x = (rng.normal(0, 1, (cin, h, w)) * scale_x).astype(np.float32)
    b = (rng.normal(0, 0.3, cout) * scale_x * scale_w).astype(np.float32)
    with GpuNet(L, [(wt, b)], (cin, h, w), "fp32", plan_cus=plan_cus) as g:
        got = g.forward(x).astype(np.float64)
        plan = D.daris_get_launch_plan(g.task, 0)
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(wt).double(), torch.from_numpy(b).double(),
                                      stride=s, padding=p).numpy().ravel()
    return float(np.linalg.norm(got - want) / np.linalg.norm(want)), plan


@pytest.mark.parametrize("scale_x,scale_w", [(1.0, 1.0), (1e30, 1e-3), (1e-20, 1e-8), (3e4, 1e33)])
@pytest.mark.parametrize("cin,h,w,cout,k", [(512, 7, 7, 512, 3), (128, 28, 28, 128, 3), (24, 13, 13, 40, 1), (4, 9, 9, 8, 3)])
def test_three_part_products_are_fp32_products(cin, h, w, cout, k, scale_x, scale_w):
    err, _ = _conv(cin, h, w, cout, k, 1, k // 2, scale_x, scale_w)
    assert err <= 5e-7, err       # sqrt(4608) * 2^-25 = 2e-6 is what plain fp32 sums may show; the fp32 instruction: 4.3e-7


@pytest.mark.parametrize("scale_x,scale_w", [(1e-33, 1.0), (1e-35, 1.0), (1e-37, 1.0), (1e-36, 1e3)])
@pytest.mark.parametrize("cin,h,w,cout,k", [(512, 7, 7, 512, 3), (128, 28, 28, 128, 3), (24, 13, 13, 40, 1), (4, 9, 9, 8, 3), (256, 56, 56, 256, 3), (3, 31, 29, 40, 3)])
def test_small_pixels_keep_their_bits(cin, h, w, cout, k, scale_x, scale_w):
    """Pixels whose third part is below the smallest bf16 number: their sums are taken with fp32 products."""
    err, _ = _conv(cin, h, w, cout, k, 1, k // 2, scale_x, scale_w)
    assert err <= 5e-7, err


# (cin, h, w, cout, k, stride, pad, plan_cus, pixels per wave tile)
@pytest.mark.parametrize("case", [(64, 5, 40, 32, 3, 1, 1, 8, 32), (128, 5, 40, 64, 3, 1, 1, 128, 16), (64, 10, 40, 64, 3, 1, 1, 8, 64), (3, 36, 74, 32, 3, 2, 0, 8, 32), (3, 36, 74, 64, 3, 2, 0, 8, 32)],
                         ids=lambda c: "x".join(map(str, c)))
def test_pixels_that_nobody_stores_have_no_say_in_the_range_of_a_tile(case):
    """Small pixels, and 1 where in the last tile only windows past the output reach: the first pixels of the last row (3x3 with
    padding), or a last row and column that no window of stride 2 covers."""
    cin, h, w, cout, k, s, p, cus, rows = case
    rng = np.random.default_rng(23)
    x = (rng.normal(0, 1, (cin, h, w)) * 1e-36).astype(np.float32)
    if p:
        x[:, h - 1], x[:, h - 1, :8] = 0.0, 1.0      # (waves whose taps lie in the last row or below have sums of 0, which are in range)
    else:
        x[:, h - 1], x[:, :, w - 1] = 1.0, 1.0
    wt = rng.normal(0, np.sqrt(2.0 / (cin * k * k)), (cout, cin, k, k)).astype(np.float32)
    L = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=0, in_from=-1)]
    with GpuNet(L, [(wt, np.zeros(cout, np.float32))], (cin, h, w), "fp32", plan_cus=cus) as g:
        got = g.forward(x).astype(np.float64).reshape(cout, -1)
        plan = D.daris_get_launch_plan(g.task, 0)
    assert plan["rows"] == rows and plan["gather"] == (D.GATHER_TAPS if p else D.GATHER_IMAGE)      # the case runs the kernel it names
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(wt).double(), stride=s, padding=p).numpy().reshape(cout, -1)
    first = got.shape[1] // rows * rows if p else 0      # of the last tile; without padding every window misses the ones
    assert first < got.shape[1] and np.abs(want[:, first:]).max() < 1e-34
    assert np.linalg.norm(got[:, first:] - want[:, first:]) <= 5e-7 * np.linalg.norm(want[:, first:])


@pytest.mark.parametrize("scale_w", [1e-33, 1e-36])
def test_small_weights_keep_what_bf16_resolves(scale_w):
    """A weight is kept in its three parts: off by at most 2^-134, hence a sum by 2^-134 / (weights' standard deviation) of itself
    (K terms of either kind add up alike)."""
    cin, k = 128, 3
    err, _ = _conv(cin, 28, 28, 128, k, 1, 1, 1.0, scale_w)
    assert err <= 5e-7 + 2.0 ** -134 / (scale_w * np.sqrt(2.0 / (cin * k * k))), err


# (cin, h, w, cout, k, stride, pad, plan_cus): what it is about
BLOCK_CASES = [
    (64, 56, 56, 64, 3, 1, 1, 32),     # M = 3136 = 49 tiles of 64: 49 workgroups of 4 waves
    (32, 41, 43, 64, 3, 1, 1, 32),     # ragged last tile (1763 = 27 * 64 + 35), K = 288
    (64, 48, 47, 128, 3, 2, 1, 8),     # stride 2, many tiles for few CUs: 2 waves
    (256, 23, 29, 64, 1, 1, 0, 8),     # 1x1: one tap, K = 256, the smallest; last tile of 27 pixels
    (16, 33, 33, 192, 5, 1, 2, 32),    # 5x5 with 25 taps, one chunk per tap, three channel tiles
    (48, 21, 20, 64, 3, 1, 0, 8),      # no padding, three chunks per tap
    (512, 28, 28, 512, 3, 1, 1, 128),  # 104 workgroups of 8 waves
    (512, 28, 28, 512, 3, 1, 1, 48),   # K split over workgroups as well
    (64, 3, 200, 64, 3, 1, 1, 8),      # wide and flat: every row touches the border
]


@pytest.mark.parametrize("case", BLOCK_CASES, ids=lambda c: "x".join(map(str, c)))
def test_block_tiles(case):
    cin, h, w, cout, k, s, p, cus = case
    err, plan = _conv(cin, h, w, cout, k, s, p, plan_cus=cus)
    assert plan["rows"] == 64 and plan["tn"] == 2 and (plan["M"] + 63) // 64 * plan["NTn"] >= cus * 3 // 4      # the case runs the kernel it names
    assert err <= 5e-7, err


# (cin, h, w, cout): 3x3 windows with stride 1 and padding 1 on maps as wide as a tile, one pixel less or more, and one or two pixels wide
# or high; three channel blocks of 16; waves with no group of taps to walk
@pytest.mark.parametrize("cin,h,w,cout", [(32, 700, 1, 64), (32, 350, 2, 64), (32, 1, 700, 64), (48, 2, 333, 128), (32, 9, 63, 64), (32, 9, 64, 64), (32, 9, 65, 64),
                                          (48, 23, 29, 192)])
def test_three_taps_from_one_fetch_of_rows(cin, h, w, cout):
    """Single pixels at corners, row ends and tile ends: nothing reaches a pixel on the other side of the image's edge."""
    rng = np.random.default_rng(19)
    x = np.zeros((cin, h * w), np.float32)
    at = sorted({0, w - 1, w * (h // 2), w * (h // 2) + w - 1, h * w - w, h * w - 1, min(63, h * w - 1), min(64, h * w - 1)})
    for i, m in enumerate(at):
        x[(7 * i) % cin, m] = 1.0 + i
    x = x.reshape(cin, h, w)
    wt = rng.normal(0, 1, (cout, cin, 3, 3)).astype(np.float32)
    L = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, stride=1, pad=1, act=0, in_from=-1)]
    with GpuNet(L, [(wt, None)], (cin, h, w), "fp32", plan_cus=8) as g:
        got = g.forward(x).astype(np.float64).reshape(cout, h, w)
        plan = D.daris_get_launch_plan(g.task, 0)
        assert plan["rows"] == 64 and plan["gather"] == D.GATHER_TAPS      # the case runs the kernel it names
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(wt).double(), padding=1).numpy()[0]
    bound = torch.nn.functional.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(wt).double().abs(), padding=1).numpy()[0]
    assert (np.abs(got - want) <= 2.0 ** -22 * bound).all()      # products to 2^-23 each, at most a few of them in a sum


@pytest.mark.parametrize("case", [(64, 112, 112, 64, 7, 1, 3, 128), (64, 56, 56, 64, 6, 1, 3, 32), (16, 64, 64, 64, 9, 1, 4, 32), (256, 56, 56, 256, 1, 1, 1, 128)],
                         ids=lambda c: "x".join(map(str, c)))
def test_large_layers_that_block_tiles_cannot_take(case):
    """More filter taps than a word has bits, padding as wide as the window: enough tiles of 64 pixels, but another kernel."""
    cin, h, w, cout, k, s, p, cus = case
    err, plan = _conv(cin, h, w, cout, k, s, p, plan_cus=cus)
    assert (plan["M"] + 63) // 64 * plan["NTn"] >= cus * 3 // 4 and plan["rows"] != 64
    assert err <= 5e-7, err


# (cin, h, w, cout, k, stride, pad, plan_cus), pixels per wave tile, K split over workgroups, gather: every kernel that walks a tile again
SECOND_WALK_CASES = [
    ((3, 31, 29, 40, 3, 2, 1, 128), 32, 0, D.GATHER_INPUT),      # the network input as the caller gives it
    ((3, 31, 29, 40, 3, 1, 1, 128), 32, 0, D.GATHER_IMAGE),      # ... in patches
    ((20, 13, 13, 40, 1, 1, 0, 128), 32, 0, D.GATHER_GENERAL),   # pixels straight into registers
    ((128, 29, 27, 128, 3, 2, 1, 16), 32, 0, D.GATHER_ROWS),     # whole rows, eight waves
    ((16, 41, 43, 64, 1, 1, 0, 128), 32, 0, D.GATHER_ROWS),      # ... two, a single chunk between them
    ((4096, 5, 5, 32, 1, 1, 0, 256), 32, 1, D.GATHER_ROWS),      # ... K split over workgroups
    ((512, 9, 9, 32, 3, 2, 1, 256), 32, 1, D.GATHER_ROWS),
    ((512, 7, 7, 512, 1, 1, 0, 128), 16, 0, D.GATHER_ROWS),
    ((256, 14, 14, 512, 3, 2, 1, 128), 16, 0, D.GATHER_ROWS),
    ((256, 23, 29, 64, 1, 1, 0, 8), 64, 0, D.GATHER_ROWS),
    ((64, 48, 47, 128, 3, 2, 1, 8), 64, 0, D.GATHER_ROWS),
    ((128, 14, 14, 128, 3, 1, 1, 16), 32, 0, D.GATHER_TAPS),
    ((512, 5, 5, 32, 3, 1, 1, 256), 32, 1, D.GATHER_TAPS),
    ((128, 9, 7, 32, 3, 1, 1, 256), 16, 0, D.GATHER_TAPS),
    ((512, 7, 7, 512, 3, 1, 1, 128), 16, 0, D.GATHER_TAPS),
    ((64, 41, 43, 64, 3, 1, 1, 32), 64, 0, D.GATHER_TAPS),
]


def _runs(plan, rows, split, gather):
    return plan["rows"] == rows and (plan["splitk"] > 1) == bool(split) and plan["gather"] == gather


@pytest.mark.parametrize("case,rows,split,gather", SECOND_WALK_CASES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_small_pixels_keep_their_bits_in_every_kernel(case, rows, split, gather):
    cin, h, w, cout, k, s, p, cus = case
    err, plan = _conv(cin, h, w, cout, k, s, p, 1e-35, 1.0, plan_cus=cus)
    assert _runs(plan, rows, split, gather), plan      # the case runs the kernel it names
    assert err <= 5e-7, err


@pytest.mark.parametrize("case,rows,split,gather", SECOND_WALK_CASES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_infinities_and_nan_pass_as_in_fp32_arithmetic(case, rows, split, gather):
    cin, h, w, cout, k, s, p, cus = case
    rng = np.random.default_rng(11)
    x = rng.normal(0, 1, (cin, h, w)).astype(np.float32)
    wt = rng.normal(0, np.sqrt(2.0 / (cin * k * k)), (cout, cin, k, k)).astype(np.float32)
    wt[0, 0, 0, 0] = np.inf
    b = rng.normal(0, 0.3, cout).astype(np.float32)
    x[0, 0, 0], x[1, h - 1, w - 1], x[cin - 1, h // 2, w // 2] = np.inf, -np.inf, np.nan
    x[0, h // 2, 0] = 3.4e38       # its upper half alone is finite, rounded to bf16 it would not be
    wt[1:, 0] *= 0.1               # ... and the products stay finite
    L = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=0, in_from=-1)]
    with GpuNet(L, [(wt, b)], (cin, h, w), "fp32", plan_cus=cus) as g:
        got = g.forward(x).astype(np.float64).reshape(cout, -1)[1:]
        assert _runs(D.daris_get_launch_plan(g.task, 0), rows, split, gather)
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(wt).double(), torch.from_numpy(b).double(),
                                      stride=s, padding=p).numpy().reshape(cout, -1)[1:]      # (channel 0: 0 * inf at the border)
    big = np.abs(want) > 1e30
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.isinf(want).any() and np.isnan(want).any()
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    for part in (np.isfinite(want) & ~big, np.isfinite(want) & big):
        assert np.linalg.norm(got[part] - want[part]) <= 5e-7 * max(np.linalg.norm(want[part]), 1e-30)


# two convolutions on one tensor in one launch: (cin, h, w, cout, stride, plan_cus), pixels per wave tile
@pytest.mark.parametrize("what", ["small", "infinite"])
@pytest.mark.parametrize("case,rows", [((64, 28, 28, 64, 2, 16), 32), ((256, 14, 14, 512, 2, 128), 16)], ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_second_walk_in_joint_launches(case, rows, what):
    """A 3x3 convolution and a 1x1 one on the same tensor, and a depthwise 1x1 window over the first, one layer after the other as the
    network's output, so that each of the two is seen by itself."""
    cin, h, w, cout, s, cus = case
    rng = np.random.default_rng(14)
    x = rng.normal(0, 1, (cin, h, w)).astype(np.float32)
    if what == "small":
        x *= np.float32(1e-35)
    else:
        x[0, 0, 0], x[1, h // 2, w // 2], x[cin - 1, h - 2, w - 2] = np.inf, -np.inf, np.nan
    pair = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, stride=s, pad=1, act=0, in_from=-1),
            N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, stride=s, pad=0, act=0, in_from=-1)]
    wts = [(rng.normal(0, np.sqrt(2.0 / (cin * L.k * L.k)), (cout, cin, L.k, L.k)).astype(np.float32), np.zeros(cout, np.float32)) for L in pair]
    same = (np.ones((cout, 1, 1, 1), np.float32), np.zeros(cout, np.float32))
    for i in (0, 1):
        layers = pair + [N.Layer(op=N.OP_CONV, c_in=cout, c_out=cout, k=1, stride=1, pad=0, groups=cout, act=0, in_from=i)]
        with GpuNet(layers, wts + [same], x.shape, "fp32", plan_cus=cus) as g:
            got = g.forward(x).astype(np.float64)
            plan = [D.daris_get_launch_plan(g.task, n) for n in (0, 1)]
        assert plan[0]["pair_with"] == 1 and all(_runs(q, rows, 0, D.GATHER_ROWS) for q in plan), plan
        want = torch.nn.functional.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(wts[i][0]).double(), stride=s, padding=pair[i].pad).numpy().ravel()
        fin = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
        assert what == "small" or (np.isinf(want).any() and np.isnan(want).any())
        assert np.linalg.norm(got[fin] - want[fin]) <= 5e-7 * np.linalg.norm(want[fin])


def test_infinities_and_nan_through_a_fused_depthwise_layer():
    """Expansion, depthwise and projection with the depthwise layer inside the projection's launch; all weights positive, so
    that an infinite pixel stays one."""
    rng = np.random.default_rng(12)
    layers = [N.Layer(op=N.OP_CONV, c_in=3, c_out=32, k=1, stride=1, pad=0, act=0, in_from=-1),
              N.Layer(op=N.OP_CONV, c_in=32, c_out=32, k=3, stride=1, pad=1, groups=32, act=0, in_from=0),
              N.Layer(op=N.OP_CONV, c_in=32, c_out=16, k=1, stride=1, pad=0, act=0, in_from=1)]
    wts = [((rng.random((L.c_out, L.c_in // L.groups, L.k, L.k)) * 0.1 + 0.01).astype(np.float32), rng.normal(0, 0.3, L.c_out).astype(np.float32)) for L in layers]
    x = rng.normal(0, 1, (3, 56, 57)).astype(np.float32)
    x[0, 5, 6], x[1, 30, 56], x[2, 55, 20] = np.inf, -np.inf, np.nan
    with GpuNet(layers, wts, x.shape, "fp32") as g:
        assert D.daris_get_launch_plan(g.task, 1)["pair_with"] == 2      # the case runs the kernel it names
        got = g.forward(x).astype(np.float64).reshape(16, -1)
    want = torch.from_numpy(x).double()[None]
    for L, (w, b) in zip(layers, wts):
        want = torch.nn.functional.conv2d(want, torch.from_numpy(w).double(), torch.from_numpy(b).double(), stride=L.stride, padding=L.pad, groups=L.groups)
    want = want.numpy().reshape(16, -1)
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.isinf(want).any() and np.isnan(want).any()
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.linalg.norm(got[fin] - want[fin]) <= 2e-6 * np.linalg.norm(want[fin])      # three layers of at most 32 terms in fp32


@pytest.mark.parametrize("cin,hw,cout,k,gather", [(512, 28, 512, 3, D.GATHER_TAPS), (2048, 28, 512, 1, D.GATHER_ROWS)])
def test_the_time_of_a_layer_is_bounded_whatever_its_input(cin, hw, cout, k, gather):
    """Stages are not preempted, so no frame may take a layer far longer than others do.  A frame through one layer whose
    sums all have to be taken again with fp32 products takes 2.4 times as long (the layer's matrix instructions: 1 + 8/3 times as
    long, plus what a frame costs besides); the bound leaves room for noise."""
    rng = np.random.default_rng(13)
    L = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=1, pad=k // 2, act=0, in_from=-1)]
    wt = rng.normal(0, 0.02, (cout, cin, k, k)).astype(np.float32), np.zeros(cout, np.float32)
    best = {}
    with GpuNet(L, [wt], (cin, hw, hw), "fp32") as g:
        assert D.daris_get_launch_plan(g.task, 0)["gather"] == gather
        y = torch.zeros(g.n_out, device="cuda")
        for what, v in (("ordinary", 1.0), ("infinite", float("inf")), ("nan", float("nan"))):
            x = torch.randn((cin, hw, hw), device="cuda") * v
            torch.cuda.synchronize()
            for _ in range(10):
                t0 = time.perf_counter()
                D.daris_forward(g.task, x, y, g.parts[0])
                best[what] = min(best.get(what, 1.0), time.perf_counter() - t0)
    assert best["infinite"] < 4 * best["ordinary"] and best["nan"] < 4 * best["ordinary"], best
