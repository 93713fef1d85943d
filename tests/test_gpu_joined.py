"""Layers that are computed in the launch of another one, against the oracle and, bit for bit, against launches of their own (a stage cut between the
two layers parts them)."""
import numpy as np
import pytest
import torch

import paper_2504_08795_amd as D
import workloads as wl
from gpu_helpers import TOL, GpuNet, oracle_logits, rel_err

pytestmark = pytest.mark.gpu
N = wl.nets


def _joined_and_parted(layers, weights, shp, dtype, xs, n_cu=128, plan_cus=0):
    """The network in one stage and with every legal cut in use, on each of the inputs: [(joined, parted)], and the plans of the joined one."""
    outs = []
    with GpuNet(layers, weights, shp, dtype, n_cu=n_cu, plan_cus=plan_cus) as g:
        plans = [D.daris_get_launch_plan(g.task, l) for l in range(len(layers))]
        joined = [g.forward(x) for x in xs]
    with GpuNet(layers, weights, shp, dtype, k=len(layers), n_cu=n_cu, plan_cus=plan_cus) as g:       # a chain: every cut is legal
        for x, j in zip(xs, joined):
            outs.append((j, g.forward(x)))
    return outs, plans


# c_in, h, w, c_out, k, stride, pad: the edges of a workgroup's 4 x 7 pooled pixels, outputs of odd and even sizes, and frames larger than one round
# (in fp32 planned for as many CUs as there are workgroups at least)
STEMS = [(3, 224, 224, 64, 7, 2, 3), (3, 189, 253, 64, 7, 2, 3), (3, 130, 131, 64, 7, 2, 3), (4, 61, 83, 128, 5, 1, 2), (1, 70, 90, 192, 3, 1, 1), (3, 97, 61, 60, 3, 1, 0)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("stem", STEMS)
def test_first_convolution_and_its_pooling(stem, dtype):
    cin, h, w, cout, k, s, p = stem
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=1, in_from=-1, has_bn=False),
              N.Layer(op=N.OP_MAXPOOL, c_in=cout, c_out=cout, k=3, stride=2, pad=1, in_from=0)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    bad = x.copy()
    bad[0, h // 2, w // 3], bad[0, 1, w - 2] = np.nan, np.inf
    outs, plans = _joined_and_parted(layers, weights, (cin, h, w), dtype, [x, bad], plan_cus=128 if dtype == "bf16" else 256 if h * w > 6000 else 128)
    assert plans[0]["pair_with"] == 1 and "image_pool" in D.daris_kernel_name(plans[1]["kernel_id"]), plans
    np.testing.assert_array_equal(*outs[0])
    np.testing.assert_array_equal(*outs[1])
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


# c_in, h, w, c_out, stride of the depthwise layer, plan CUs: one to five chunks of K, a band of all rows, bands of one row, a last band of fewer rows, tiles that end
# inside a row, maps of one pixel and as wide as LDS has room for
EXPANSIONS = [(160, 7, 7, 960, 1, 128), (96, 14, 14, 576, 2, 128), (64, 14, 14, 384, 1, 128), (32, 28, 28, 192, 2, 128), (32, 28, 28, 192, 1, 96), (128, 13, 17, 48, 2, 32),
              (64, 1, 1, 16, 1, 128), (32, 40, 106, 32, 1, 256), (96, 5, 100, 16, 2, 8), (160, 21, 9, 32, 1, 64)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", EXPANSIONS)
def test_expansion_and_its_depthwise_layer(shape, dtype):
    cin, h, w, cout, s, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, act=2, in_from=-1, has_bn=False),
              N.Layer(op=N.OP_CONV, c_in=cout, c_out=cout, k=3, stride=s, pad=1, groups=cout, act=2, in_from=0, has_bn=False)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    bad = x.copy()
    bad[0, h // 2, w // 3], bad[cin - 1, 0, w - 1] = np.nan, np.inf
    outs, plans = _joined_and_parted(layers, weights, (cin, h, w), dtype, [x, bad], plan_cus=cus)
    assert "expand_dw" in D.daris_kernel_name(plans[1]["kernel_id"]) and plans[0]["out_slot"] == -1, plans
    np.testing.assert_array_equal(*outs[0])
    np.testing.assert_array_equal(*outs[1])
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


def test_expansion_of_small_numbers_keeps_its_precision():
    """Pixels of 1e-37, whose third parts fall below the smallest bf16 number: the joined launch walks such tiles in plain fp32 as well."""
    layers = [N.Layer(op=N.OP_CONV, c_in=96, c_out=64, k=1, act=0, in_from=-1, has_bn=False),
              N.Layer(op=N.OP_CONV, c_in=64, c_out=64, k=3, pad=1, groups=64, act=0, in_from=0, has_bn=False)]
    weights = [(w, np.zeros_like(b)) for w, b in wl.make_weights(layers, 3)]
    x = wl.make_inputs((96, 14, 14), 3, 1, "normal")[0]
    with GpuNet(layers, weights, (96, 14, 14), "fp32") as g:
        assert "expand_dw" in D.daris_kernel_name(D.daris_get_launch_plan(g.task, 1)["kernel_id"])
        one, small = g.forward(x), g.forward(x * np.float32(2.0 ** -122))
    # sums of 96 terms near 2^-122 have no denormal results; what is lost are bits of single products below 2^-149, 2^-27 of a sum's terms
    np.testing.assert_allclose(small * np.float64(2.0 ** 122), one, rtol=0, atol=2e-6 * np.abs(one).max())


# h, w, channels of the first 1x1, of the second (0: none), input of the first as residual, plan CUs: whole and ragged last tiles, one of a single pixel, images narrower than
# a tile, other channels (which stay by themselves)
CHAINS = [(56, 56, 256, 64, True, 128), (56, 56, 256, 0, True, 128), (48, 65, 256, 64, False, 128), (13, 17, 256, 40, True, 8), (193, 1, 256, 64, False, 8), (3, 75, 256, 36, True, 8),
          (15, 15, 256, 0, False, 8), (15, 15, 160, 64, True, 8)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", CHAINS)
def test_bottleneck_in_one_launch(shape, dtype):
    """A convolution in front makes the residual's channels.  NO_JOIN parts all of it, a stage cut the 3x3 from the first 1x1 or that from the second: bit for bit the same."""
    h, w, n3, n1, res, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=32, c_out=n3, k=1, act=1, in_from=-1, has_bn=False), N.Layer(op=N.OP_CONV, c_in=n3, c_out=64, k=1, act=1, in_from=0, has_bn=False),
              N.Layer(op=N.OP_CONV, c_in=64, c_out=64, k=3, pad=1, act=1, in_from=1, has_bn=False),
              N.Layer(op=N.OP_CONV, c_in=64, c_out=n3, k=1, act=1, in_from=2, res_from=0 if res else -1, has_bn=False)]
    if n1:
        layers.append(N.Layer(op=N.OP_CONV, c_in=n3, c_out=n1, k=1, act=2, in_from=3, has_bn=False))
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((32, h, w), 3, 1, "normal")[0]
    bad = x.copy()
    bad[0, h // 2, w // 3], bad[31, 0, w - 1] = np.nan, np.inf
    outs = []
    for flags, k in ((0, 1), (0, 2), (D.NO_JOIN, 1)):
        with GpuNet(layers, weights, (32, h, w), dtype, flags=flags, k=k, plan_cus=cus) as g:
            assert (D.daris_get_launch_plan(g.task, 2)["out_slot"] == -1) == (flags == 0 and n3 == 256 and 3 not in D.daris_get_stage_cuts(g.task))
            outs.append([g.forward(x), g.forward(bad)])
    for other in outs[1:]:
        np.testing.assert_array_equal(outs[0][0], other[0])
        np.testing.assert_array_equal(outs[0][1], other[1])
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


# c_in, h, w, c_out of the convolution, its window, FC outputs, plan CUs; one to four tiles of 16 or 32 pixels, the last one full or of one pixel; more channels than a lane has
# loads in flight for, and not a multiple of a wave's
AVERAGES = [(64, 7, 7, 512, 3, 1000, 128), (320, 7, 7, 1280, 1, 37, 128), (64, 7, 7, 2048, 1, 10, 128), (32, 1, 1, 64, 1, 5, 128), (32, 4, 8, 96, 1, 16, 8), (64, 3, 11, 4000, 1, 9, 256),
            (64, 10, 10, 512, 1, 21, 128), (128, 8, 8, 24, 3, 1000, 64), (32, 8, 16, 40, 3, 3, 8)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", AVERAGES)
def test_convolution_global_average_and_fc(shape, dtype):
    cin, h, w, cout, k, n_out, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, pad=k // 2, act=1, in_from=-1, has_bn=False),
              N.Layer(op=N.OP_GAVGPOOL, c_in=cout, c_out=cout, in_from=0), N.Layer(op=N.OP_FC, c_in=cout, c_out=n_out, in_from=1)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    outs, plans = _joined_and_parted(layers, weights, (cin, h, w), dtype, [x, x[::-1].copy()], plan_cus=cus)
    assert plans[0]["pair_with"] == 2 and not plans[0]["pair_lead"] and plans[1]["kernel_id"] == plans[0]["kernel_id"], plans
    for o in outs:
        np.testing.assert_array_equal(*o)                     # the pooling layer alone in its stage makes the averages from the same sums
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)
    with GpuNet(layers, weights, (cin, h, w), dtype, flags=D.NO_JOIN, plan_cus=cus) as g:   # pooling in a launch of its own: the same sums in another order
        assert D.daris_kernel_name(D.daris_get_launch_plan(g.task, 1)["kernel_id"]) == "gavgpool"
        e_max, e_l2 = rel_err(outs[0][0], g.forward(x))
    assert e_max <= (2e-6 if dtype == "fp32" else 2 ** -7), e_max


def test_infinite_averages_stay_infinite():
    layers = [N.Layer(op=N.OP_CONV, c_in=32, c_out=100, k=1, act=1, in_from=-1, has_bn=False), N.Layer(op=N.OP_GAVGPOOL, c_in=100, c_out=100, in_from=0),
              N.Layer(op=N.OP_FC, c_in=100, c_out=8, in_from=1)]
    weights = [(np.abs(w), np.abs(b)) for w, b in wl.make_weights(layers, 3)[:1]] + [(None, None)] + [(np.abs(w) + 1, b) for w, b in wl.make_weights(layers, 3)[2:]]
    x = np.ones((32, 5, 5), np.float32)
    x[0, 2, 2] = np.inf
    with GpuNet(layers, weights, x.shape, "fp32") as g:
        assert D.daris_get_launch_plan(g.task, 0)["pair_with"] == 2
        x_d, y_d = torch.from_numpy(x).cuda(), torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        D.daris_forward(g.task, x_d, y_d, g.parts[0])
        assert torch.isposinf(y_d).all(), y_d


# c_in, h, w, c_out, plan CUs: tiles of 16 pixels and two blocks of channels whose second block of pixels is whole, ragged, of one pixel or empty, images narrower than
# a block, a single row; eight waves (the second layer of the last in bf16, K = 1152: four, which keep two blocks of channels)
TALL = [(256, 14, 14, 256, 128), (256, 7, 7, 512, 64), (512, 7, 7, 512, 64), (256, 1, 49, 256, 32), (256, 1, 33, 256, 32), (256, 16, 15, 128, 64)]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", TALL)
def test_two_blocks_of_pixels_or_of_channels(shape, dtype):
    """The same sums, bit for bit, whichever blocks share a wave, with infinities and NaN as well."""
    cin, h, w, cout, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, pad=1, act=1, in_from=-1, has_bn=False),
              N.Layer(op=N.OP_CONV, c_in=cout, c_out=cout, k=3, pad=1, act=1, in_from=0, res_from=0, has_bn=False)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    bad = x.copy()
    bad[0, h // 2, w // 3], bad[cin - 1, 0, w - 1] = np.nan, np.inf
    outs = []
    for flags in (0, D.NO_TALL_TILES):
        with GpuNet(layers, weights, (cin, h, w), dtype, flags=flags, plan_cus=cus) as g:
            assert "conv_wave16_taps" in D.daris_kernel_name(D.daris_get_launch_plan(g.task, 0)["kernel_id"]) and D.daris_get_launch_plan(g.task, 0)["tn"] == 2, D.daris_get_launch_plan(g.task, 0)
            outs.append([g.forward(x), g.forward(bad)])
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)


# c_in, h, w, c_out, plan CUs: workgroups of eight, four and two waves, whole and ragged last tiles, a single pair of rows, rows of two pixels and of fewer than a tile's,
# channels that end inside a block
BLOCK_POOLS = [(64, 20, 22, 64, 8), (64, 16, 24, 64, 8), (32, 28, 30, 64, 8), (32, 38, 48, 64, 8), (64, 2, 200, 100, 8), (48, 70, 6, 64, 8), (64, 200, 2, 64, 8), (128, 56, 56, 256, 128),
               (64, 112, 110, 128, 128)]


@pytest.mark.parametrize("shape", BLOCK_POOLS)
def test_large_convolution_and_its_pooling(shape):
    cin, h, w, cout, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, pad=1, act=1, in_from=-1, has_bn=False), N.Layer(op=N.OP_MAXPOOL, c_in=cout, c_out=cout, k=2, stride=2, in_from=0)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    bad, small = x.copy(), x * np.float32(2.0 ** -115)
    bad[0, h // 2, w // 3], bad[cin - 1, 0, w - 1] = np.nan, np.inf
    outs, plans = _joined_and_parted(layers, weights, (cin, h, w), "fp32", [x, bad, small], plan_cus=cus)
    assert plans[0]["rows"] == 64, plans
    with GpuNet(layers, weights, (cin, h, w), "fp32", plan_cus=cus) as g:
        ms, kid, _ = D.daris_profile_layers(g.task, g.parts[0], 2, 2)
        assert ms[0] == 0 and D.daris_kernel_name(kid[1]) == "conv_wave64_pool_f32", (ms, kid)
    np.testing.assert_array_equal(*outs[0])
    np.testing.assert_array_equal(*outs[1])
    np.testing.assert_array_equal(*outs[2])                         # (all sums of every tile are so small that all of it is walked again)
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, "fp32"))
    assert e_max <= TOL["fp32"] and e_l2 <= TOL["fp32"], (e_max, e_l2)


# c_in, h, w, c_out, plan CUs: 9, 12, 13, 15 and 18 groups of taps on eight waves, in 32-pixel tiles of one and two blocks, 64-pixel and 16-pixel ones; K split across
# workgroups whose last share is the smallest
SHARES = [(96, 5, 5, 96, 128), (64, 13, 17, 64, 8), (64, 56, 56, 64, 128), (208, 7, 9, 32, 8), (80, 13, 17, 64, 8), (96, 13, 17, 64, 8), (64, 48, 64, 64, 64), (96, 20, 21, 64, 8), (416, 7, 7, 256, 64), (512, 5, 5, 512, 240)]


@pytest.mark.parametrize("shape", SHARES)
def test_uneven_shares_of_k(shape):
    cin, h, w, cout, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=3, pad=1, act=1, in_from=-1, has_bn=False)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    with GpuNet(layers, weights, (cin, h, w), "fp32", plan_cus=cus) as g:
        assert "taps" in D.daris_kernel_name(D.daris_get_launch_plan(g.task, 0)["kernel_id"])
        e_max, e_l2 = rel_err(g.forward(x), oracle_logits(layers, weights, x, "fp32"))
    assert e_max <= 2e-6 and e_l2 <= 1e-6, (e_max, e_l2)            # a group too many or too few is an error of the order of a sum


@pytest.mark.parametrize("first,then", [(1, 4), (4, 1)])
def test_stages_chosen_behind_the_io_pool(first, then):
    """The argument blocks of a pool are those of the launches that run: a cut that parts or joins the first layers gives the pool new ones."""
    layers = [N.Layer(op=N.OP_CONV, c_in=3, c_out=64, k=7, stride=2, pad=3, act=1, in_from=-1, has_bn=False), N.Layer(op=N.OP_MAXPOOL, c_in=64, c_out=64, k=3, stride=2, pad=1, in_from=0),
              N.Layer(op=N.OP_GAVGPOOL, c_in=64, c_out=64, in_from=1), N.Layer(op=N.OP_FC, c_in=64, c_out=10, in_from=2)]
    x = torch.from_numpy(wl.make_inputs((3, 96, 100), 3, 3, "normal")).cuda()
    with GpuNet(layers, wl.make_weights(layers, 3), (3, 96, 100), "fp32", k=first, plan_cus=64) as g:
        want, got = torch.zeros((3, 10), device="cuda"), torch.zeros((3, 10), device="cuda")
        D.daris_task_set_io(g.task, x, 3, got, 3)
        D.daris_split_stages(g.task, then)
        joined = "image_pool" in D.daris_kernel_name(D.daris_get_launch_plan(g.task, 1)["kernel_id"])
        assert joined == (1 not in D.daris_get_stage_cuts(g.task)) == (then == 1)
        D.daris_commit()
        D.daris_run_closed_loop([3])
        for i in range(3):
            D.daris_forward(g.task, x[i], want[i], g.parts[0])
        torch.cuda.synchronize()
    assert want.abs().min() > 0
    np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())


# dtype, c_in, h, w, c_out, stride, plan CUs, whether a second 1x1 of 64 channels shares the launch: tiles of 16 and 32 pixels, one and two blocks of channels, two to eight waves,
# whole and ragged last tiles, K that leaves a wave a chunk less or none, K split across workgroups
WINDOWS = [("bf16", 224, 6, 19, 24, 2, 8, False), ("bf16", 512, 13, 8, 24, 2, 8, False), ("bf16", 2048, 11, 8, 96, 2, 32, False), ("bf16", 160, 13, 24, 24, 2, 8, False), ("bf16", 512, 22, 18, 64, 1, 64, False),
           ("bf16", 2048, 26, 34, 64, 1, 128, False), ("bf16", 128, 31, 17, 96, 1, 8, False), ("bf16", 256, 14, 21, 96, 2, 8, False), ("bf16", 256, 37, 37, 256, 1, 8, False), ("bf16", 512, 25, 27, 64, 2, 8, False),
           ("fp32", 96, 5, 28, 24, 2, 8, False), ("fp32", 256, 25, 29, 24, 2, 32, False), ("fp32", 512, 2, 29, 24, 2, 8, False), ("fp32", 128, 33, 14, 256, 2, 32, False), ("fp32", 256, 14, 28, 64, 1, 64, False),
           ("fp32", 2048, 17, 17, 256, 2, 64, False), ("fp32", 96, 23, 19, 96, 1, 8, False), ("fp32", 1024, 7, 19, 96, 1, 8, False), ("fp32", 256, 11, 27, 64, 2, 8, False), ("fp32", 160, 34, 26, 1000, 1, 8, False),
           ("fp32", 224, 17, 26, 256, 2, 8, False), ("fp32", 512, 23, 31, 256, 2, 32, False),
           ("bf16", 224, 3, 29, 24, 2, 32, True), ("bf16", 512, 7, 10, 96, 1, 32, True), ("bf16", 2048, 2, 29, 96, 2, 32, True), ("bf16", 224, 18, 22, 96, 2, 64, True), ("bf16", 1024, 19, 13, 96, 1, 64, True),
           ("bf16", 2048, 21, 37, 64, 1, 128, True), ("bf16", 224, 17, 6, 96, 2, 8, True), ("bf16", 512, 6, 5, 256, 2, 8, True), ("bf16", 160, 30, 14, 1000, 2, 8, True), ("bf16", 512, 3, 13, 512, 2, 8, True),
           ("fp32", 224, 6, 9, 64, 2, 32, True), ("fp32", 256, 2, 19, 64, 2, 32, True), ("fp32", 512, 5, 2, 64, 1, 8, True), ("fp32", 96, 7, 9, 96, 2, 8, True), ("fp32", 1024, 15, 26, 24, 1, 64, True),
           ("fp32", 96, 26, 8, 96, 1, 8, True), ("fp32", 160, 39, 7, 24, 2, 8, True), ("fp32", 512, 39, 8, 24, 2, 32, True), ("fp32", 32, 18, 25, 64, 1, 8, True), ("fp32", 224, 9, 3, 512, 1, 8, True),
           ("fp32", 1024, 19, 19, 1000, 1, 240, True), ("fp32", 2048, 24, 25, 1000, 2, 32, True)]


@pytest.mark.parametrize("case", WINDOWS, ids=lambda c: "-".join(map(str, c)))
def test_windows_of_one_by_one_without_padding_and_with(case):
    """With padding the general kernels run; inside, the same plan has the same sums, bit for bit."""
    dtype, cin, h, w, cout, s, cus, two = case
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    outs, plans = [], []
    for padded in (False, True):
        last = dict(k=1, act=1, in_from=-1, has_bn=False)
        layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, stride=s, pad=s if padded else 0, **last)]
        if two:
            layers.append(N.Layer(op=N.OP_CONV, c_in=cin, c_out=64, pad=1 if padded else 0, **last))
        with GpuNet(layers, wl.make_weights(layers, 3), (cin, h, w), dtype, plan_cus=cus) as g:
            plans.append([{q: p[q] for q in ("rows", "tn", "nw", "S", "sz", "sw", "splitk", "gather", "pair_with")} for p in (D.daris_get_launch_plan(g.task, l) for l in range(len(layers)))])
            outs.append(g.forward(x).reshape(wl.layer_shapes(layers, (cin, h, w))[-1]))
    assert plans[0] == plans[1] and plans[0][0]["gather"] == D.GATHER_ROWS and (plans[0][0]["pair_with"] == 1) == two
    inside = outs[1][:, 1:1 + outs[0].shape[1], 1:1 + outs[0].shape[2]]       # (stride 2 has two pixels of padding)
    np.testing.assert_array_equal(outs[0], inside)
    assert np.abs(outs[0]).max() > 0


# c_in, h, w, c_out, k, stride, pad, plan CUs, the kernel: 64-pixel tiles with and without three taps per fetch, 32-pixel and 16-pixel ones (two blocks of pixels), whole rows, 1x1, any channels, the
# network input in patches and gathered, K split across workgroups
SECOND_WALKS = [(64, 40, 44, 64, 3, 1, 1, 8, "conv_wave64_taps"), (64, 40, 44, 64, 3, 2, 1, 8, "conv_wave64_f32"), (64, 28, 28, 64, 3, 1, 1, 64, "conv_wave_taps"), (256, 14, 14, 256, 3, 1, 1, 128, "conv_wave16_taps"),
                (64, 28, 28, 96, 3, 2, 1, 64, "conv_wave16_f32"), (64, 57, 57, 96, 3, 2, 1, 32, "conv_wave_f32"), (256, 20, 20, 96, 1, 1, 0, 32, "conv_wave"), (24, 30, 30, 64, 3, 1, 1, 64, "conv_wave_f32"), (3, 64, 70, 64, 7, 2, 3, 32, "conv_wave_image"),
                (3, 20, 20, 32, 7, 2, 3, 128, "conv_wave_f32"), (512, 6, 6, 512, 3, 1, 1, 240, "conv_wave_taps")]


@pytest.mark.parametrize("case", SECOND_WALKS, ids=lambda c: "-".join(map(str, c)))
def test_what_is_not_finite_changes_only_the_sums_that_it_is_part_of(case):
    """A tile with a NaN or an infinity is walked a second time; its other sums stay, bit for bit, what they are without."""
    cin, h, w, cout, k, s, p, cus, kernel = case
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=p, act=0, in_from=-1, has_bn=False)]
    weights = wl.make_weights(layers, 3)
    x = wl.make_inputs((cin, h, w), 3, 1, "normal")[0]
    with GpuNet(layers, weights, (cin, h, w), "fp32", plan_cus=cus) as g:
        plan = D.daris_get_launch_plan(g.task, 0)
        assert D.daris_kernel_name(plan["kernel_id"]).startswith(kernel) and (plan["splitk"] > 1) == (cus == 240), plan
        ho, wo = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
        clean = g.forward(x).reshape(cout, ho, wo)
        for bad in (np.nan, np.inf, -np.inf):
            y, z = x.copy(), (h // 2, w // 3)
            y[cin // 2, z[0], z[1]] = bad
            got = g.forward(y).reshape(cout, ho, wo)
            rows, cols = (np.abs(np.arange(n) * s - p + (k - 1) / 2 - at) <= (k - 1) / 2 for n, at in ((ho, z[0]), (wo, z[1])))
            hit = np.broadcast_to(rows[:, None] & cols[None, :], got.shape)
            np.testing.assert_array_equal(got[~hit], clean[~hit])
            assert hit.any() and not np.isfinite(got[hit]).any()
            if not np.isnan(bad):
                taps = weights[0][0][:, cin // 2]                                # each sum has the infinity times one weight
                want = np.stack([bad * taps[:, z[0] + p - s * i, z[1] + p - s * j] for i in np.flatnonzero(rows) for j in np.flatnonzero(cols)], 1)
                np.testing.assert_array_equal(got[:, rows][:, :, cols].reshape(cout, -1), want)


@pytest.mark.parametrize("net,hw,cus", [("resnet18", (96, 100), 64), ("resnet50", (112, 112), 32), ("mobilenet_v2", (96, 128), 128), ("vgg16", (64, 64), 32)])
def test_networks_with_infinities_do_not_depend_on_the_stages(net, hw, cus):
    layers, (c, _, _) = wl.build_net(net)
    if net == "vgg16":
        layers = layers[:-3]
    x = wl.make_inputs((c,) + hw, 3, 1, "normal")[0]
    x[0, hw[0] // 2, hw[1] // 3], x[1, 3, hw[1] - 2], x[2, hw[0] - 1, 0] = np.nan, np.inf, -np.inf
    weights, outs = wl.make_weights(layers, 3), []
    legal = 1 + sum(1 for l in range(len(layers) - 1) if all(q.in_from >= l and not 0 <= q.res_from < l for q in layers[l + 1:]))
    for k in (1, 3, legal):
        with GpuNet(layers, weights, (c,) + hw, "fp32", k=k, plan_cus=cus) as g:
            outs.append(g.forward(x))
    for o in outs[1:]:
        np.testing.assert_array_equal(outs[0], o)
