"""Whole networks planned, cut into stages, joined or parted and encoded as launches, and the launches walked on the CPU: what each reads lies where the layer in
front left it, what it writes fits the buffer, and every tile of it is computed once.  The planner and the encoders are compiled into a small executable
(`tests/host_plans/networks.cpp`), no GPU needed."""
import os
import subprocess

import numpy as np
import pytest

import workloads as wl

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_08795_amd", "csrc")
N = wl.nets


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("networks") / "networks")
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-w", "-I/opt/rocm/include", "-o", exe, os.path.join(HERE, "host_plans", "networks.cpp")] +
                          [os.path.join(CSRC, f) for f in ("net_plan.cpp", "launch.cpp", "net_encode.cpp")])

    def run(cases):
        """cases: (dtype, (c, h, w), plan CUs, stages, layers); [(case, [(layer, kernel, workgroups)])]."""
        lines = []
        for dtype, shp, cus, k, layers in cases:
            lines.append(" ".join(map(str, (int(dtype == "bf16"),) + tuple(shp) + (cus, k, len(layers)))))
            lines += [f"{L.op} {L.c_in} {L.c_out} {L.k} {L.stride} {L.pad} {L.groups} {L.act} {L.in_from} {L.res_from}" for L in layers]
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        out = r.stdout.splitlines()
        assert len(out) == len(cases)
        for case, ln in zip(cases, out):
            assert ln.startswith("ok"), (case[:4], ln, [(L.op, L.c_in, L.c_out, L.k, L.stride, L.pad, L.in_from, L.res_from) for L in case[4]][:12])
        return [(c, [(int(a), b, int(g)) for a, b, g in (w.split(":") for w in ln.split()[1:])]) for c, ln in zip(cases, out)]
    return run


JOINED = {"conv_image_pool_kernel", "conv_expand_dw_kernel", "fc_pooled_kernel", "conv_chain_kernel", "conv_block_pool_kernel", "conv_taps16_tall_kernel", "conv_point_kernel", "conv_point_pair_kernel"}


def _resized(name, h, w):
    layers, (c, _, _) = wl.build_net(name)
    out, shapes = [], []
    for L in layers:
        src = (c, h, w) if L.in_from < 0 else shapes[L.in_from]
        if L.op == N.OP_FC:
            L = N.Layer(op=L.op, c_in=src[0] * src[1] * src[2], c_out=L.c_out, act=L.act, in_from=L.in_from)
        out.append(L)
        shapes.append(wl.layer_shapes(out, (c, h, w))[-1])
    return out, (c, h, w)


def test_every_launch_of_the_configured_networks_is_sound(walk):
    rng = np.random.default_rng(23)
    cases = []
    for name in ("tiny", "mobilenet_v2", "resnet18", "resnet50", "vgg16"):
        for i in range(60):
            lo, hi = (32, 97) if name == "tiny" else (160, 257) if name == "vgg16" else (96, 321)
            layers, shp = _resized(name, *((224, 224) if i % 4 == 0 and name != "tiny" else (int(v) for v in rng.integers(lo, hi, 2))))
            cases.append((("fp32", "bf16")[i & 1], shp, int(rng.choice([32, 48, 64, 96, 112, 128, 192, 256])), int(rng.choice([1, 1, 2, 3, 5, 255])), layers))
    ran = {k for _, ls in walk(cases) for _, k, _ in ls}
    assert JOINED <= ran, JOINED - ran


def _random_network(rng, wide):
    """A chain of blocks: what joins, what almost does, residuals over one block, branches that share a launch."""
    layers, c, at = [], int(rng.choice([3, 4, 32, 64])), -1
    shp = (c, int(rng.integers(6, 100)), int(rng.integers(6, 100)))

    def size():
        return shp if at < 0 else wl.layer_shapes(layers, shp)[at]

    def conv(c_out, k=1, s=1, p=0, src=None, res=-1, dw=False):
        nonlocal at
        src = at if src is None else src
        c_in = shp[0] if src < 0 else layers[src].c_out
        layers.append(N.Layer(op=N.OP_CONV, c_in=c_in, c_out=c_in if dw else c_out, k=k, stride=s, pad=p, groups=c_in if dw else 1, act=int(rng.integers(0, 3)), in_from=src, res_from=res))
        at = len(layers) - 1
        return at

    if c < 8:
        conv(int(rng.choice([32, 64, 64])), 7, 2, 3) if rng.random() < .6 else conv(int(rng.choice([16, 64])), 3, 1, 1)
    for _ in range(int(rng.integers(2, 7))):
        c, h, w = size()
        kind = rng.integers(0, 8)
        if kind == 0 and min(h, w) >= 4:                                          # pooling, of either window
            k, s, p = ((3, 2, 1), (2, 2, 0), (3, 1, 1))[rng.integers(0, 3)]
            layers.append(N.Layer(op=N.OP_MAXPOOL, c_in=c, c_out=c, k=k, stride=s, pad=p, in_from=at))
            at = len(layers) - 1
        elif kind == 1:                                                           # an inverted residual block
            conv(c * int(rng.choice([2, 6])) if c <= 160 else c)
            conv(0, 3, int(rng.integers(1, 3)), 1, dw=True)
            conv(int(rng.choice([16, 32, 64, 96])))
        elif kind == 2:                                                           # bottlenecks
            short = conv(256, src=at) if rng.random() < .5 else -1                # (which the first convolution of the block shares a launch with)
            conv(64, src=layers[short].in_from if short >= 0 else None)
            conv(64, 3, 1, 1)
            block = conv(256, res=short)
            conv(int(rng.choice([64, 64, 40, 128])))
            if rng.random() < .7:
                conv(64, 3, 1, 1)
                conv(256, res=block)
        elif kind == 3:                                                           # a basic block, with a shortcut convolution half of the time
            src, s = at, int(rng.integers(1, 3))
            out = int(rng.choice([64, 128, 256])) if wide else 64
            if rng.random() < .5:
                short = conv(out, 1, s, 0, src=src)
                conv(out, 3, s, 1, src=src)
                conv(out, 3, 1, 1, res=short)
            elif c == out:
                conv(out, 3, 1, 1)
                conv(out, 3, 1, 1, res=src)
        elif kind == 4:
            conv(int(rng.choice([16, 24, 64, 128, 256, 512])), 3, 1, 1)
        elif kind == 5:                                                           # a large convolution and 2 x 2 pooling
            conv(int(rng.choice([64, 128, 256])), 3, 1, 1)
            if min(h, w) >= 2:
                layers.append(N.Layer(op=N.OP_MAXPOOL, c_in=layers[at].c_out, c_out=layers[at].c_out, k=2, stride=2, in_from=at))
                at = len(layers) - 1
        else:
            conv(int(rng.choice([16, 40, 64, 256, 512])), 1, int(rng.integers(1, 3)), int(rng.integers(0, 10) == 0))
    if not layers:
        conv(16)
    if rng.random() < .6:
        c = size()[0]
        layers.append(N.Layer(op=N.OP_GAVGPOOL, c_in=c, c_out=c, in_from=at))
        layers.append(N.Layer(op=N.OP_FC, c_in=c, c_out=int(rng.integers(1, 60)), in_from=len(layers) - 1))
    return layers, shp


def test_every_launch_of_random_networks_is_sound(walk):
    rng = np.random.default_rng(29)
    cases = []
    for i in range(3000):
        layers, shp = _random_network(rng, i % 3 > 0)
        cases.append((("fp32", "bf16")[i & 1], shp, int(rng.choice([8, 16, 32, 64, 96, 128, 192, 256])), int(rng.choice([1, 1, 2, 3, 255])), layers))
    ran = {}
    for c, ls in walk(cases):
        for _, k, _ in ls:
            ran[k] = ran.get(k, 0) + 1
    assert JOINED | {"conv_wave_pair_kernel", "splitk_reduce_kernel", "conv_wave_dw_kernel", "gavgpool_kernel", "conv_block_kernel"} <= set(ran), ran
    assert all(ran[k] >= 10 for k in JOINED), ran


def test_two_blocks_of_pixels_for_long_loops_only(walk):
    """16-pixel tiles with three taps per fetch: the short loops of four waves, bf16 with K below 2048, and of fewer than twelve groups of taps keep two blocks of channels."""
    shapes = [("bf16", 128, 15, 16, 256, 128, False), ("bf16", 192, 14, 18, 128, 64, False), ("bf16", 256, 15, 25, 64, 64, True), ("bf16", 256, 14, 14, 256, 128, True),
              ("fp32", 96, 25, 15, 128, 128, False), ("fp32", 128, 16, 24, 128, 96, True), ("fp32", 256, 14, 14, 256, 128, True)]
    cases = [(dtype, (c, h, w), cus, 1, [N.Layer(op=N.OP_CONV, c_in=c, c_out=c_out, k=3, pad=1, in_from=-1)]) for dtype, c, h, w, c_out, cus, _ in shapes]
    for s, (_, ls) in zip(shapes, walk(cases)):
        assert [k for _, k, _ in ls] == ["conv_taps16_tall_kernel" if s[-1] else "conv_taps16_kernel"], (s, ls)


def test_only_convolutions_over_whole_rows_leave_sums_for_the_average(walk):
    """The other kernels store their outputs, which a pooling layer of its own averages."""
    tail = lambda c: [N.Layer(op=N.OP_CONV, c_in=c, c_out=96, k=1, in_from=-1), N.Layer(op=N.OP_GAVGPOOL, c_in=96, c_out=96, in_from=0), N.Layer(op=N.OP_FC, c_in=96, c_out=10, in_from=1)]
    shapes = [("fp32", 32, True), ("fp32", 24, False), ("bf16", 64, True), ("bf16", 48, False)]
    for (dtype, c, sums), (_, ls) in zip(shapes, walk([(dtype, (c, 7, 7), 128, 1, tail(c)) for dtype, c, _ in shapes])):
        assert [k for _, k, _ in ls][1:] == (["fc_pooled_kernel"] if sums else ["gavgpool_kernel", "fc_kernel"]), (dtype, c, ls)


def test_kernels_of_one_by_one_windows(walk):
    """Those of their own wherever rows are fetched whole, but not with padding."""
    conv = lambda c, p=0: [N.Layer(op=N.OP_CONV, c_in=c, c_out=512, k=1, pad=p, in_from=-1)]
    shapes = [("bf16", 64, 0, True), ("bf16", 128, 0, True), ("bf16", 192, 0, True), ("bf16", 256, 0, True), ("fp32", 128, 0, True), ("fp32", 128, 1, False), ("bf16", 256, 1, False)]
    for s, (_, ls) in zip(shapes, walk([(dtype, (c, 28, 28), 128, 1, conv(c, p)) for dtype, c, p, _ in shapes])):
        assert [k for _, k, _ in ls] == ["conv_point_kernel" if s[-1] else "conv_wave_kernel"], (s, ls)
