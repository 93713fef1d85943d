"""GPU parity of every kernel against the CPU oracle, one or two layers at a time, through the C ABI.
Shapes span several tiles, ragged M / N / K tails, split-K, both strides and both arithmetic types."""
import numpy as np
import pytest

import workloads as wl
import paper_2504_08795_amd as D
from gpu_helpers import GpuNet, oracle_logits, rel_err

pytestmark = pytest.mark.gpu
N = wl.nets
RNG = np.random.default_rng(99)

# per-layer bars, far inside the whole-network tolerances: fp32 accumulation over K <= 4608 terms versus a double sum
# (~sqrt(K) * 2^-24 relative to the row norm), bf16 one final rounding (2^-9) on top
LAYER_TOL = {"fp32": 2e-5, "bf16": 6e-3}


def rand_w(L, scale=None):
    cg = L.c_in // L.groups
    if L.op == N.OP_CONV:
        w = RNG.normal(0, np.sqrt(2.0 / (cg * L.k * L.k)), (L.c_out, cg, L.k, L.k))
    else:
        w = RNG.normal(0, np.sqrt(2.0 / L.c_in), (L.c_out, L.c_in))
    return w.astype(np.float32), RNG.normal(0, 0.3, L.c_out).astype(np.float32)


def run_case(layers, shp, dtype, tol=None):
    weights = [rand_w(L) if L.op in (N.OP_CONV, N.OP_FC) else (None, None) for L in layers]
    x = RNG.normal(0, 1, shp).astype(np.float32)
    want = oracle_logits(layers, weights, x, dtype)
    with GpuNet(layers, weights, shp, dtype) as net:
        got = net.forward(x)
    e_max, e_l2 = rel_err(got, want)
    tol = tol or LAYER_TOL[dtype]
    assert e_max <= tol and e_l2 <= tol, (e_max, e_l2)
    return got, want


CONV_CASES = [
    # (cin, h, w, cout, k, s, p, act)  -- comment: what it stresses
    (3, 32, 32, 16, 3, 1, 1, 1),      # Tiny c1: padded 3-channel input, N = 16 < tile
    (16, 32, 32, 32, 3, 1, 1, 1),     # Tiny c2
    (32, 16, 16, 64, 3, 1, 1, 1),     # Tiny c4
    (3, 64, 64, 64, 7, 2, 3, 1),      # stem 7x7 s2 (quarter-size image)
    (64, 28, 28, 64, 3, 1, 1, 1),     # layer1-like, M = 784
    (64, 29, 27, 128, 3, 2, 1, 1),    # stride 2, odd sizes, ragged M
    (64, 28, 28, 128, 1, 2, 0, 0),    # 1x1 s2 downsample, no activation
    (128, 14, 14, 256, 3, 1, 1, 1),   # M = 196 -> split-K
    (512, 7, 7, 512, 3, 1, 1, 1),     # M = 49, K = 4608 -> deep split-K
    (256, 7, 7, 1024, 1, 1, 0, 1),    # 1x1 wide N
    (24, 13, 13, 40, 1, 1, 0, 2),     # ragged everything, ReLU6
    (40, 9, 11, 24, 3, 1, 1, 0),      # K = 360: K tail inside a tile
    (8, 5, 5, 8, 3, 1, 1, 1),         # smaller than any tile
    (32, 56, 56, 64, 3, 1, 1, 1),     # M = 3136: many M tiles
    (16, 112, 112, 96, 1, 1, 0, 2),   # MobileNet expand: M = 12544, largest tile variant
    (1, 7, 7, 4, 3, 1, 1, 0),         # degenerate: one input channel, four outputs
    (4, 3, 3, 8, 3, 1, 0, 1),         # output is a single pixel (M = 1)
    (8, 1, 1, 12, 1, 1, 0, 0),        # 1x1 image, 1x1 kernel: a plain mat-vec
    (4, 9, 9, 4, 3, 3, 0, 0),         # stride equal to the kernel size: no window overlap
    (8, 6, 6, 8, 3, 1, 2, 1),         # padding larger than half the kernel: whole windows of zeros at the border
    (256, 14, 14, 200, 3, 1, 1, 1),   # 16-pixel tiles (M = 196: ragged last tile), N = 200: 13 blocks of 16, the last one ragged
    (512, 7, 7, 520, 3, 1, 1, 2),     # 16-pixel tiles, M = 49, 33 channel blocks, K = 4608, ReLU6
    (64, 224, 224, 64, 3, 1, 1, 1),   # the largest layer of any configuration (VGG-16 conv1_2): M = 50176
    (3, 224, 224, 64, 3, 1, 1, 1),    # VGG-16 conv1_1: K = 27, M = 50176
]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", CONV_CASES, ids=lambda c: "x".join(map(str, c)))
def test_conv(case, dtype):
    cin, h, w, cout, k, s, p, act = case
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=act, in_from=-1)]
    run_case(layers, (cin, h, w), dtype)


# 3x3 windows with stride 1 and padding 1 on maps one pixel wide or high, as wide as a tile and one less or more: 16-pixel tiles, 32-pixel
# tiles with and without K split over workgroups; groups of three taps that fill the waves evenly, unevenly and not all of them
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,h,w,cout", [(128, 1, 401, 64), (128, 390, 1, 64), (128, 13, 15, 64), (128, 13, 16, 64), (192, 13, 33, 40), (512, 3, 5, 64), (512, 1, 17, 520),
                                          (576, 16, 2, 96), (640, 1, 1, 512), (64, 1, 3201, 64), (64, 3137, 1, 64), (96, 103, 31, 64), (64, 99, 32, 64), (64, 98, 33, 32)])
def test_three_taps_from_one_fetch_of_rows(cin, h, w, cout, dtype):
    """Single pixels at corners, row ends and tile ends: nothing reaches a pixel on the other side of the image's edge."""
    x = np.zeros((cin, h * w), np.float32)
    for i, m in enumerate(sorted({0, w - 1, w * (h // 2), w * (h // 2) + w - 1, h * w - w, h * w - 1, min(31, h * w - 1), min(32, h * w - 1)})):
        x[(7 * i) % cin, m] = 1.0 + i
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, stride=1, pad=1, act=0, in_from=-1)]
    weights = [(rand_w(layers[0])[0], np.zeros(cout, np.float32))]
    want = oracle_logits(layers, weights, x.reshape(cin, h, w), dtype)
    with GpuNet(layers, weights, (cin, h, w), dtype) as net:
        got = net.forward(x.reshape(cin, h, w))
        plan = D.daris_get_launch_plan(net.task, 0)
        assert plan["rows"] in (16, 32) and plan["gather"] == D.GATHER_TAPS      # the case runs the kernel it names
    e_max, e_l2 = rel_err(got, want)
    assert e_max <= LAYER_TOL[dtype] and e_l2 <= LAYER_TOL[dtype] and (np.asarray(got)[np.asarray(want) == 0] == 0).all(), (e_max, e_l2)


@pytest.mark.parametrize("dtype,c", [("fp32", 256), ("bf16", 512)])
def test_tensors_of_more_than_2_GiB(dtype, c):
    """1500 x 1500 pixels of 1024 bytes: written, read as a residual operand, by a 1x1 and by a 3x3 window; compared at the upper
    and lower edge and around the byte 2^31."""
    h = w = 1500
    layers = [N.Layer(op=N.OP_CONV, c_in=1, c_out=32, k=1, stride=1, pad=0, act=1, in_from=-1),
              N.Layer(op=N.OP_CONV, c_in=32, c_out=c, k=1, stride=1, pad=0, act=0, in_from=0),
              N.Layer(op=N.OP_CONV, c_in=c, c_out=c, k=1, stride=1, pad=0, act=1, in_from=1, res_from=1),
              N.Layer(op=N.OP_CONV, c_in=c, c_out=16, k=3, stride=1, pad=1, act=0, in_from=2)]
    weights = [rand_w(L) for L in layers]
    x = RNG.normal(0, 1, (1, h, w)).astype(np.float32)
    with GpuNet(layers, weights, x.shape, dtype) as net:
        got = np.asarray(net.forward(x)).reshape(16, h, w)
        plans = [D.daris_get_launch_plan(net.task, i) for i in (1, 2, 3)]
    assert [q["gather"] for q in plans] == [D.GATHER_ROWS, D.GATHER_ROWS, D.GATHER_TAPS]
    middle = (1 << 31) // (1024 * w)
    for a, b in ((0, 2), (middle - 1, middle + 2), (h - 2, h)):      # rows [a, b) of the output want one more on either side inside the image
        a0, b0 = max(a - 1, 0), min(b + 1, h)
        want = np.asarray(oracle_logits(layers, weights, x[:, a0:b0], dtype)).reshape(16, b0 - a0, w)[:, a - a0:b - a0]
        e_max, e_l2 = rel_err(got[:, a:b], want)
        tol = {"fp32": 4 * LAYER_TOL["fp32"], "bf16": 2e-2}[dtype]   # four layers' sums; their bf16 roundings
        assert e_max <= tol and e_l2 <= tol, (a, e_max, e_l2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,h,w,cout,rows", [
    (192, 28, 28, 32, 16),    # a fifth of the partition's CUs with 32-pixel tiles
    (64, 14, 14, 384, 16),    # a short K, two thirds of the CUs
    (96, 13, 15, 576, 16),    # the same, ragged, 126 of 128 CUs
    (64, 17, 17, 384, 16),    # ... 120 of 128
    (64, 18, 18, 384, 32),    # ... and 132: one workgroup a CU no longer
    (128, 3, 3, 20, 32),      # a short K, a single channel tile
    (160, 7, 7, 960, 16),     # wide
    (256, 14, 14, 1024, 32),  # a longer K, more than half of the CUs
])
def test_small_tiles_where_large_ones_leave_cus_idle(cin, h, w, cout, rows, dtype):
    """1x1 convolutions on either side of the line between 16- and 32-pixel tiles, with a residual operand."""
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, stride=1, pad=0, act=1, in_from=-1),
              N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, stride=1, pad=0, act=1, in_from=-1, res_from=0)]
    weights = [rand_w(L) for L in layers]
    x = RNG.normal(0, 1, (cin, h, w)).astype(np.float32)
    with GpuNet(layers, weights, (cin, h, w), dtype, flags=D.NO_PAIR) as net:
        got = net.forward(x)
        assert D.daris_get_launch_plan(net.task, 1)["rows"] == (rows if dtype == "fp32" or cin >= 128 else 32)    # (bf16: two waves have four steps between them at least)
    e_max, e_l2 = rel_err(got, oracle_logits(layers, weights, x, dtype))
    tol = {"fp32": 2e-5, "bf16": 1.2e-2}[dtype]  # two layers' sums; two bf16 roundings and a margin
    assert e_max <= tol and e_l2 <= tol, (e_max, e_l2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,h,w,cout,k,s,p,patched", [
    (3, 45, 61, 64, 7, 2, 3, ("fp32", "bf16")),      # last tiles partly outside, input rows of an odd length
    (1, 16, 16, 32, 3, 1, 1, ("fp32",)),             # whole tiles, one channel plane; no more blocks of 32 x 32 than CUs
    (1, 16, 48, 32, 3, 1, 1, ("fp32", "bf16")),
    (2, 9, 200, 40, 1, 1, 0, ("fp32", "bf16")),      # a single tap, channels that end inside a block
    (4, 37, 33, 96, 5, 2, 2, ("fp32", "bf16")),      # three channel blocks, no pad channel
    (3, 30, 31, 24, 3, 3, 1, ()),                    # more places than the patch has: gathered tap by tap
    (3, 61, 47, 64, 3, 3, 0, ("fp32", "bf16")),      # stride 3
    (3, 17, 19, 128, 11, 1, 5, ("fp32", "bf16")),    # 121 taps
    (3, 66, 70, 64, 11, 4, 2, ()),                   # gathered tap by tap
])
def test_network_input_in_patches(cin, h, w, cout, k, s, p, patched, dtype):
    """The first convolution reads the caller's layout; also with pixels so small that fp32 takes its tiles a second time (2^-110: every
    sum is below 2^-103 of 1).  The error bars are relative to the largest sum, and so hold at both scales.  Planned for 8 CUs, where there
    are more tiles than CUs, and for 256, where one round of the gather is enough (but for small windows with stride 1 in fp32)."""
    L = N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=0, in_from=-1)
    weights = [(rand_w(L)[0], np.zeros(cout, np.float32))]
    x = RNG.normal(0, 1, (cin, h, w)).astype(np.float32)
    want = np.asarray(oracle_logits([L], weights, x, dtype), np.float64)
    for cus, patches in ((8, dtype in patched), (256, dtype == "fp32" and dtype in patched and s == 1 and 3 <= k <= 5)):
        with GpuNet([L], weights, (cin, h, w), dtype, plan_cus=cus) as net:
            assert D.daris_get_launch_plan(net.task, 0)["gather"] == (D.GATHER_IMAGE if patches else D.GATHER_INPUT), cus
            for scale in (1.0, 2.0 ** -110):
                xs = (x * np.float32(scale)).astype(np.float32)
                e_max, e_l2 = rel_err(np.asarray(net.forward(xs), np.float64) / scale, want)
                assert e_max <= LAYER_TOL[dtype] and e_l2 <= LAYER_TOL[dtype], (cus, scale, e_max, e_l2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,hw,cout,s", [(64, 28, 128, 2), (64, 14, 64, 1), (256, 7, 512, 2)])
def test_conv_residual_block(cin, hw, cout, s, dtype):
    """downsample 1x1 (or identity) + 3x3 + 3x3 with residual add before ReLU: the basic-block epilogue."""
    layers = []
    if s != 1 or cin != cout:
        layers.append(N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, stride=s, pad=0, act=0, in_from=-1))
        skip, base = 0, 1
    else:
        layers.append(N.Layer(op=N.OP_MAXPOOL, c_in=cin, c_out=cin, k=1, stride=1, pad=0, in_from=-1))   # identity copy as tensor 0
        skip, base = 0, 1
    layers.append(N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, stride=s, pad=1, act=1, in_from=-1))
    layers.append(N.Layer(op=N.OP_CONV, c_in=cout, c_out=cout, k=3, stride=1, pad=1, act=1, in_from=base, res_from=skip))
    run_case(layers, (cin, hw, hw), dtype, tol={"fp32": 5e-5, "bf16": 1.2e-2}[dtype])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cin,h,w,mid,cout,s,ds_first", [
    (64, 28, 28, 32, 128, 2, True),     # ResNet-50 shape of block: shortcut 1x1 s2 and 1x1 s1 read the same tensor, different output sizes
    (64, 28, 28, 32, 128, 2, False),    # the same with the shortcut listed after the first convolution
    (40, 13, 11, 24, 72, 1, True),      # ragged sizes: padding workgroups between the two problems of the launch
    (256, 14, 14, 64, 512, 2, True),    # heavier problem split over K (its reduction follows the joint launch)
    (32, 9, 9, 96, 96, 1, False),       # channel block counts 3 and 3: the wide-tile variant does not apply to either
])
def test_conv_pair_in_bottleneck_block(cin, h, w, mid, cout, s, ds_first, dtype):
    """Two convolutions reading one tensor (issued as one launch) inside a bottleneck block with a strided middle layer."""
    ds = N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, stride=s, pad=0, act=0, in_from=-1)
    c1 = N.Layer(op=N.OP_CONV, c_in=cin, c_out=mid, k=1, stride=1, pad=0, act=1, in_from=-1)
    layers = [ds, c1] if ds_first else [c1, ds]
    i_ds, i_c1 = (0, 1) if ds_first else (1, 0)
    layers.append(N.Layer(op=N.OP_CONV, c_in=mid, c_out=mid, k=3, stride=s, pad=1, act=1, in_from=i_c1))
    layers.append(N.Layer(op=N.OP_CONV, c_in=mid, c_out=cout, k=1, stride=1, pad=0, act=1, in_from=2, res_from=i_ds))
    run_case(layers, (cin, h, w), dtype, tol={"fp32": 5e-5, "bf16": 1.5e-2}[dtype])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w,s", [(32, 112, 112, 1), (96, 57, 55, 2), (144, 28, 28, 1), (960, 7, 7, 1), (24, 9, 9, 2)])
def test_depthwise(c, h, w, s, dtype):
    layers = [N.Layer(op=N.OP_CONV, c_in=c, c_out=c, k=3, stride=s, pad=1, groups=c, act=2, in_from=-1)]
    run_case(layers, (c, h, w), dtype)


# (block input channels, hidden channels, h, w, depthwise stride, output channels, residual)
DW_PROJECT_CASES = [
    (16, 32, 112, 112, 1, 16, True),    # MobileNetV2's first block: K = 32, one chunk per wave, 392 pixel tiles
    (16, 96, 113, 111, 2, 24, False),   # stride 2 on odd sizes: 57 x 56 outputs, ragged last tile
    (24, 144, 56, 56, 1, 24, True),     # 144 channels: whole 64-byte rows in fp32 only (bf16 keeps the separate launch)
    (16, 64, 56, 56, 1, 64, False),     # 64 output channels: one tile of two channel blocks in bf16 (fused), two tiles in fp32 (not)
    (32, 192, 28, 28, 2, 64, False),    # the rest: too few pixel tiles or several channel blocks, the depthwise launch stays
    (64, 384, 14, 14, 1, 64, True),
    (160, 960, 7, 7, 1, 320, False),
    (40, 64, 9, 9, 1, 40, True),
]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", DW_PROJECT_CASES, ids=lambda c: "x".join(map(str, c)))
def test_depthwise_computed_inside_the_projection(case, dtype):
    """An inverted residual block's depthwise 3x3 convolution computed inside the launch of the 1x1 convolution that reads it:
    against the oracle, and against the same block with the depthwise layer in a launch of its own (bit for bit when the
    1x1 convolution keeps its plan, since the fused producer accumulates in the same order)."""
    cin, hid, h, w, s, cout, res = case
    if res:
        assert s == 1 and cin == cout
    layers = [N.Layer(op=N.OP_CONV, c_in=3, c_out=cin, k=3, stride=1, pad=1, act=0, in_from=-1),
              N.Layer(op=N.OP_CONV, c_in=cin, c_out=hid, k=1, stride=1, pad=0, act=2, in_from=0),
              N.Layer(op=N.OP_CONV, c_in=hid, c_out=hid, k=3, stride=s, pad=1, groups=hid, act=2, in_from=1),
              N.Layer(op=N.OP_CONV, c_in=hid, c_out=cout, k=1, stride=1, pad=0, act=0, in_from=2, res_from=0 if res else -1)]
    weights = [rand_w(L) for L in layers]
    x = RNG.normal(0, 1, (3, h, w)).astype(np.float32)
    want = oracle_logits(layers, weights, x, dtype)
    outs, plans = [], []
    for flags in (0, D.NO_FUSED_DW):
        with GpuNet(layers, weights, (3, h, w), dtype, flags=flags) as net:
            outs.append(net.forward(x))
            plans.append([D.daris_get_launch_plan(net.task, l) for l in range(4)])
    # fused where the hidden tensor's pixels are whole 64-byte rows and the 1x1 convolution has at least 96 pixel tiles and one
    # channel tile of a staged kernel variant
    o = plans[1][3]
    want_fused = (hid * (4 if dtype == "fp32" else 2)) % 64 == 0 and o["MT"] >= 96 and o["NTn"] == 1 and (dtype == "bf16" or o["tn"] == 1)
    assert (plans[0][2]["pair_with"] == 3) == want_fused and plans[1][2]["pair_with"] == -1    # the case runs the path it names
    assert want_fused == {"fp32": case in DW_PROJECT_CASES[:3], "bf16": case in DW_PROJECT_CASES[:2] + DW_PROJECT_CASES[3:4]}[dtype]
    tol = {"fp32": 5e-5, "bf16": 1.5e-2}[dtype]
    for got in outs:
        e_max, e_l2 = rel_err(got, want)
        assert e_max <= tol and e_l2 <= tol, (e_max, e_l2)
    if all(plans[0][3][k] == plans[1][3][k] for k in ("kernel_id", "splitk", "sz", "sw", "rows")):
        np.testing.assert_array_equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w,k,s,p", [(64, 112, 112, 3, 2, 1), (32, 32, 32, 2, 2, 0), (3, 9, 7, 3, 2, 1), (16, 15, 15, 2, 2, 0)])
def test_maxpool(c, h, w, k, s, p, dtype):
    layers = [N.Layer(op=N.OP_MAXPOOL, c_in=c, c_out=c, k=k, stride=s, pad=p, in_from=-1)]
    weights = [(None, None)]
    x = (-np.abs(RNG.normal(0, 1, (c, h, w))) - 0.5).astype(np.float32)       # all negative: padding must not win
    want = oracle_logits(layers, weights, x, dtype)
    with GpuNet(layers, weights, (c, h, w), dtype) as net:
        got = net.forward(x)
    np.testing.assert_array_equal(got, want)                                  # selection only: bit exact


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w", [(512, 7, 7), (1280, 7, 7), (20, 3, 5)])
def test_gavgpool(c, h, w, dtype):
    layers = [N.Layer(op=N.OP_GAVGPOOL, c_in=c, c_out=c, in_from=-1)]
    run_case(layers, (c, h, w), dtype, tol={"fp32": 1e-6, "bf16": 4e-3}[dtype])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,h,w,n,act", [(64, 8, 8, 10, 0), (512, 1, 1, 1000, 0), (32, 7, 7, 4096, 1), (3, 5, 5, 7, 0)])
def test_fc(c, h, w, n, act, dtype):
    layers = [N.Layer(op=N.OP_FC, c_in=c * h * w, c_out=n, act=act, in_from=-1)]
    run_case(layers, (c, h, w), dtype)


# (dtype, c, h, w, n): vectors of 16 bytes a row, and what is left after the loop of one (fp32) or two (bf16) loads per lane
FC_STREAM_CASES = [("bf16", 40, 23, 29, 2521),   # 3335 = 26 * 128 + 7, 134.5 MB
                   ("bf16", 8, 2137, 1, 3930),   # 2137 = 16 * 128 + 89: the rest takes two passes
                   ("bf16", 16, 32, 36, 7300),   # 2304 = 18 * 128: nothing is left
                   ("fp32", 8, 2051, 1, 2050),   # 4102 = 64 * 64 + 6
                   ("fp32", 64, 16, 12, 2733)]   # 3072 = 48 * 64


@pytest.mark.parametrize("case", FC_STREAM_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fc_matrices_read_past_the_last_cache(case):
    """Matrices of 128 MiB and more with rows of more than 2048 vectors: the streaming loop and its remainder."""
    dtype, c, h, w, n = case
    es = 2 if dtype == "bf16" else 4
    assert n * c * h * w * es >= 128 << 20 and c * h * w * es // 16 > 2048      # the case runs the loop it names
    layers = [N.Layer(op=N.OP_FC, c_in=c * h * w, c_out=n, act=0, in_from=-1)]
    run_case(layers, (c, h, w), dtype, tol=2e-5)      # the logits stay in fp32: sqrt(K) * 2^-24 = 1e-5 in either type


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_fc_chain_with_padded_vector(dtype):
    """FC -> FC where the intermediate vector length (10) is not a multiple of the 16-byte vector."""
    layers = [N.Layer(op=N.OP_FC, c_in=16 * 4 * 4, c_out=10, act=1, in_from=-1), N.Layer(op=N.OP_FC, c_in=10, c_out=6, in_from=0)]
    run_case(layers, (16, 4, 4), dtype, tol={"fp32": 2e-5, "bf16": 1e-2}[dtype])


def test_identity_passthrough_is_exact():
    """ingest + 1x1 max-pool + egress moves every value unchanged (layout conversions only)."""
    layers = [N.Layer(op=N.OP_MAXPOOL, c_in=5, c_out=5, k=1, stride=1, pad=0, in_from=-1)]
    x = RNG.normal(0, 1, (5, 6, 7)).astype(np.float32)
    with GpuNet(layers, [(None, None)], (5, 6, 7), "fp32") as net:
        np.testing.assert_array_equal(net.forward(x), x.reshape(-1))


def test_joint_launch_whose_earlier_member_has_a_residual_operand():
    """L2 (3x3, + L0's output as residual) and L3 (1x1) both read L1 and share a launch that is issued at L3.  L0's output
    is read last by L2, so its buffer falls free exactly when L3's output is placed: it must not be reused before the
    joint launch (and L2's split-K reduction) have read it."""
    def c(i, r=-1, k=3, cin=32):
        return N.Layer(op=N.OP_CONV, c_in=cin, c_out=32, k=k, stride=1, pad=k // 2, act=1, in_from=i, res_from=r)
    layers = [c(-1, cin=3), c(0), c(1, 0), c(1, -1, 1), c(3, 2), N.Layer(op=N.OP_GAVGPOOL, c_in=32, c_out=32, in_from=4),
              N.Layer(op=N.OP_FC, c_in=32, c_out=10, in_from=5)]
    for dtype in ("fp32", "bf16"):
        run_case(layers, (3, 12, 12), dtype, tol={"fp32": 2e-5, "bf16": 2e-2}[dtype])
