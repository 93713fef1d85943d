"""What the launches of joined layers assume, checked without a device."""
import re

import pytest

import paper_2504_08795_amd as D
import workloads as wl
from lib_helpers import Session
from paper_2504_08795_amd import build
from test_host_logic import _code_object_kernels
from test_host_networks import _resized

HOST = D.VIRTUAL_TIME | D.NO_DEVICE
N = wl.nets

# code object: {kernel: (bytes of its argument block, how many instances)}
JOINED_KERNELS = {"daris_joined_kernels": {"conv_image_pool_kernel": (160, 2), "conv_expand_dw_kernel": (160, 10), "fc_pooled_kernel": (64, 2), "conv_chain_kernel": (248, 2), "conv_block_pool_kernel": (160, 3)},
                  "daris_tall_kernels": {"conv_taps16_tall_kernel": (160, 2)},
                  "daris_pointwise_kernels": {"conv_point_kernel": (160, 22), "conv_point_pair_kernel": (324, 22)}}


@pytest.mark.parametrize("co", sorted(JOINED_KERNELS))
def test_joined_kernels_match_the_argument_structures(co):
    want, seen = JOINED_KERNELS[co], {}
    for name, has in _code_object_kernels(co):
        base = [k for k in want if re.search(r"\d+" + k + r"(I|E)", name)]
        assert len(base) == 1, name
        assert has["kernarg_segment_size"] == want[base[0]][0], name
        assert has["private_segment_fixed_size"] == 0 and has["group_segment_fixed_size"] <= (81920 if "chain" in name else 65536), (name, has)
        seen[base[0]] = seen.get(base[0], 0) + 1
    assert seen == {k: n for k, (_, n) in want.items()}
    assert set(build.JOINED_SOURCES.values()) == set(JOINED_KERNELS)


def _plans(layers, shp, dtype, k=1, cus=128):
    with Session(HOST):
        D.daris_set_plan_cus(cus)
        D.daris_create_partition(64)
        dnn, keep = D.make_dnn(layers, None, shp, dtype)
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        if k > 1:
            D.daris_split_stages(t, k)
        return [D.daris_get_launch_plan(t, l) for l in range(len(layers))]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("net", ["resnet18", "resnet50"])
def test_first_pooling_layer_joins_the_convolution(net, dtype):
    layers, shp = wl.build_net(net)
    p = _plans(layers, shp, dtype)
    assert p[0]["pair_with"] == 1 and not p[0]["pair_lead"] and p[0]["out_slot"] == p[1]["in_slot"] == -1 and p[1]["pair_with"] == -1
    assert "image_pool" in D.daris_kernel_name(p[1]["kernel_id"])
    legal = 1 + sum(1 for l in range(len(layers) - 1) if all(q.in_from >= l and not 0 <= q.res_from < l for q in layers[l + 1:]))
    p = _plans(layers, shp, dtype, k=legal)                             # a cut between the two
    assert p[0]["pair_with"] == -1 and p[0]["out_slot"] == p[1]["in_slot"] >= 0 and D.daris_kernel_name(p[1]["kernel_id"]) == "maxpool"
    other = [N.Layer(op=N.OP_CONV, c_in=3, c_out=64, k=7, stride=2, pad=3, in_from=-1), N.Layer(op=N.OP_MAXPOOL, c_in=64, c_out=64, k=3, stride=2, pad=1, in_from=0),
             N.Layer(op=N.OP_CONV, c_in=64, c_out=64, k=3, stride=2, pad=1, in_from=1), N.Layer(op=N.OP_CONV, c_in=64, c_out=64, k=1, in_from=0)]
    assert _plans(other, shp, dtype)[0]["pair_with"] == -1              # somebody else reads the convolution


# h, w, plan CUs, joined in fp32: workgroups of 4 x 7 pooled pixels to a CU (bf16 always joins)
STEMS = [(224, 224, 128, True), (224, 224, 112, False), (224, 224, 96, False), (224, 224, 64, False), (224, 224, 56, False), (178, 123, 72, True), (130, 215, 80, False), (307, 299, 248, True),
         (188, 304, 152, True), (274, 183, 128, True), (274, 183, 120, False), (96, 96, 32, True)]


@pytest.mark.parametrize("h,w,cus,want", STEMS)
def test_first_pooling_layer_joins_while_a_cu_has_few_workgroups(h, w, cus, want):
    layers = wl.build_net("resnet18")[0][:2]
    for dtype in ("fp32", "bf16"):
        p = _plans(layers, (3, h, w), dtype, cus=cus)
        assert ("image_pool" in D.daris_kernel_name(p[1]["kernel_id"])) == (want or dtype == "bf16"), (dtype, p[1])


@pytest.mark.parametrize("net", ["resnet18", "resnet50", "mobilenet_v2"])
def test_global_average_without_a_launch(net):
    layers, shp = wl.build_net(net)
    for dtype in ("fp32", "bf16"):
        p = _plans(layers, shp, dtype)
        n = len(layers)
        assert p[n - 3]["pair_with"] == n - 1 and p[n - 2]["pair_with"] == -1 and p[n - 2]["kernel_id"] == p[n - 3]["kernel_id"]
        assert len({p[n - 3]["in_slot"], p[n - 3]["out_slot"], p[n - 2]["out_slot"]} - {-1}) == 3   # the sums live until the FC layer has read them
        legal = 1 + sum(1 for l in range(n - 1) if all(q.in_from >= l and not 0 <= q.res_from < l for q in layers[l + 1:]))
        assert D.daris_kernel_name(_plans(layers, shp, dtype, k=legal)[n - 2]["kernel_id"]) == "gavgpool"    # alone in its stage


def test_bottlenecks_of_64_channels_share_a_launch():
    for dtype, cus in (("bf16", 128), ("fp32", 128)):
        layers, shp = wl.build_net("resnet50")
        p = _plans(layers, shp, dtype, cus=cus)
        first = [l for l in range(len(layers)) if p[l]["out_slot"] == -1 and l > 0 and l + 1 < len(layers)]
        assert len(first) == 3 and all(layers[l].k == 3 for l in first) and first[1] - first[0] == first[2] - first[1] == 3, first
        for l in first:
            assert p[l + 1]["in_slot"] == -1
            live = [p[l]["in_slot"], p[l + 1]["out_slot"], p[l + 1]["res_slot"]] + ([p[l + 2]["out_slot"]] if l != first[2] else [])  # (the last one's successor shares its launch with a shortcut)
            assert -1 not in live and len(set(live)) == len(live), live                            # what the launch reads and writes lies in places of its own
    chain = [N.Layer(op=N.OP_CONV, c_in=64, c_out=64, k=3, pad=1, in_from=-1), N.Layer(op=N.OP_CONV, c_in=64, c_out=256, k=1, in_from=0), N.Layer(op=N.OP_CONV, c_in=256, c_out=64, k=1, in_from=1)]
    for k, joined in ((1, True), (2, True), (3, False)):                                           # two stages: the cut that balances them lies behind the first layer or the second
        p = _plans(chain, (64, 56, 56), "bf16", k=k)
        with Session(HOST):
            D.daris_create_partition(64)
            dnn, keep = D.make_dnn(chain, None, (64, 56, 56), "bf16")
            t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
            D.daris_split_stages(t, k)
            cuts = D.daris_get_stage_cuts(t)
        assert (p[0]["out_slot"] == -1) == (1 not in cuts) and (joined or 1 in cuts), (p, cuts)


def test_joins_do_not_cost_a_network_the_static_scratch():
    """Joint launches keep what they read until they are issued, which takes VGG-16 a third buffer: 16.0 MiB instead of 15.1 at 160 x 193 pixels, where the scratch holds 16."""
    for side, buffers in (((160, 160), 3), ((160, 193), 2), ((194, 160), 2), ((224, 224), 3)):   # small enough either way, only without joins, and neither
        layers, shp = _resized("vgg16", *side)
        assert len({v for p in _plans(layers, shp, "fp32") for v in (p["out_slot"], p["in_slot"])} - {-1}) == buffers, side


# (c_in, h, w, channels, stride of the depthwise layer, plan CUs), joined in (fp32, bf16): what a CU has to compute decides
EXPANSIONS = [((32, 28, 28, 192, 1, 128), (True, True)), ((96, 14, 14, 576, 1, 128), (True, True)), ((160, 7, 7, 960, 1, 128), (True, True)), ((160, 10, 10, 960, 1, 128), (True, True)),
              ((160, 10, 10, 960, 1, 120), (False, True)), ((96, 14, 14, 576, 1, 64), (True, True)), ((32, 28, 28, 192, 1, 64), (True, False)), ((64, 15, 20, 384, 1, 40), (False, False)),
              ((96, 15, 20, 576, 1, 40), (False, False)), ((160, 29, 55, 960, 1, 40), (False, False))]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape,want", EXPANSIONS)
def test_expansions_join_their_depthwise_layer_while_the_launch_is_short(shape, want, dtype):
    cin, h, w, cout, s, cus = shape
    layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=1, act=2, in_from=-1), N.Layer(op=N.OP_CONV, c_in=cout, c_out=cout, k=3, stride=s, pad=1, groups=cout, act=2, in_from=0)]
    p = _plans(layers, (cin, h, w), dtype, cus=cus)
    joined = "expand_dw" in D.daris_kernel_name(p[1]["kernel_id"])
    assert joined == want[dtype == "bf16"] == (p[0]["out_slot"] == -1)
    if not joined:                                                      # the convolution by itself, with the plan that it has without a depthwise layer behind it
        own = _plans(layers[:1], (cin, h, w), dtype, cus=cus)[0]
        assert all(p[0][k] == own[k] for k in ("kernel_id", "rows", "tn", "nw", "sw")), (p[0], own)


def _shared(net, dtype, flags):
    """How many (launch pairs, layers joined to another's launch, buffers) a network has under the flags."""
    layers, shp = wl.build_net(net)
    with Session(HOST | flags):
        D.daris_create_partition(64)
        dnn, keep = D.make_dnn(layers, None, shp, dtype)
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        p = [D.daris_get_launch_plan(t, l) for l in range(len(layers))]
    pairs = sum(1 for l, q in enumerate(p) if q["pair_lead"] and layers[l - 1].groups == 1)
    kernel = [D.daris_kernel_name(q["kernel_id"]) for q in p]
    joined = sum(1 for l, q in enumerate(p) if ("pool" in kernel[l] or "expand_dw" in kernel[l]) and kernel[l] not in ("maxpool", "gavgpool"))
    joined += sum(1 for l, L in enumerate(layers) if L.op == N.OP_GAVGPOOL and kernel[l] != "gavgpool")
    joined += sum(1 for l in range(len(layers) - 1) if layers[l + 1].op == layers[l].op == N.OP_CONV and p[l]["out_slot"] == -1 and layers[l + 1].groups == layers[l].groups == 1)
    return pairs, joined, len({v for q in p for v in (q["out_slot"], q["in_slot"])} - {-1})


@pytest.mark.parametrize("net,dtype", [("resnet18", "fp32"), ("resnet50", "bf16"), ("vgg16", "fp32"), ("mobilenet_v2", "fp32")])
def test_flags_part_what_they_name_and_nothing_else(net, dtype):
    pairs, joined, buffers = _shared(net, dtype, 0)
    assert (pairs > 0) == net.startswith("resnet") and (joined > 0) == (net != "vgg16")   # (of pooling behind 64-pixel tiles plans show the third buffer)
    assert _shared(net, dtype, D.NO_PAIR)[1:] == (joined, buffers) and _shared(net, dtype, D.NO_PAIR)[0] == 0
    assert _shared(net, dtype, D.NO_JOIN)[:2] == (pairs, 0) and (net != "vgg16" or buffers == 3 and _shared(net, dtype, D.NO_JOIN)[2] == 2)
    assert _shared(net, dtype, D.NO_FUSED_DW)[:2] == (pairs, 1 if net == "mobilenet_v2" else joined)   # (the global average)
    assert _shared(net, dtype, D.NO_TALL_TILES) == (pairs, joined, buffers)
