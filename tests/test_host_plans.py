"""Every launch plan that the planner makes for a dense convolution is one that the encoder accepts: what the planner and the
encoder each assume about a kernel must not differ, or a layer that some kernel could run is refused at registration.  The
planner and the encoders are compiled into a small executable (`tests/host_plans/driver.cpp`), no GPU needed."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_08795_amd", "csrc")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "driver")
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-I/opt/rocm/include", "-o", exe, os.path.join(HERE, "host_plans", "driver.cpp"),
                           os.path.join(CSRC, "net_plan.cpp"), os.path.join(CSRC, "launch.cpp")])

    def run(shapes):
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, s if len(s) == 13 else s + (0, 1, 1, 0))) for s in shapes) + "\n", capture_output=True, text=True, check=True)
        return [ln.split(maxsplit=1) if ln.startswith("-1") else [int(v) for v in ln.split()] for ln in r.stdout.splitlines()]
    return run


# fp32: (c_in, h, w, c_out, k, stride, pad, plan CUs) -- enough tiles for the 64 x 64 kernel, which cannot take them
NOT_FOR_BLOCKS = [
    (64, 112, 112, 64, 7, 1, 3, 128),     # 49 taps
    (512, 28, 28, 512, 7, 1, 3, 128),
    (64, 56, 56, 64, 6, 1, 3, 32),        # 36 taps
    (16, 64, 64, 64, 9, 1, 4, 32),        # 81 taps
    (256, 56, 56, 256, 1, 1, 1, 128),     # padding as wide as the window
    (256, 1500, 1500, 64, 3, 1, 1, 128),  # 2.3 GB of input
]


# (dtype, c_in, h, w, c_out, k, stride, pad, plan CUs), gather: tensors of 2 GiB and more, whose tiles lie within 2 GiB all the same
LARGE_TENSORS = [
    ((0, 256, 1500, 1500, 16, 3, 1, 1, 128), 5),
    ((0, 256, 1500, 1500, 64, 1, 1, 0, 128), 3),
    ((0, 256, 1500, 1500, 64, 3, 2, 1, 128), 3),
    ((0, 32, 1500, 1500, 512, 1, 1, 0, 128), 3),
    ((1, 512, 1500, 1500, 16, 3, 1, 1, 128), 5),
    ((1, 512, 1500, 1500, 64, 1, 1, 0, 128), 3),
    ((1, 32, 1500, 1500, 512, 1, 1, 0, 128), 3),
]


def test_large_tensors_are_fetched_in_whole_rows(plans):
    for (s, gather), p in zip(LARGE_TENSORS, plans([s for s, _ in LARGE_TENSORS])):
        assert p[0] == 1 and p[6] == gather, (s, p)
    both = plans([(0, 256, 1500, 1500, 64, 3, 2, 1, 128, 64, 1, 2, 0)])[0]      # two that could share a launch, which has no kernel for them
    assert both[0] == 1 and not both[5] and both[6] == 3, both


def test_layers_that_the_64_pixel_tiles_cannot_take_keep_a_kernel(plans):
    for s, p in zip(NOT_FOR_BLOCKS, plans([(0,) + s for s in NOT_FOR_BLOCKS])):
        assert p[0] == 1 and p[2] != 64, (s, p)
    for s, p in zip([(64, 112, 112, 64, 5, 1, 2, 128)], plans([(0, 64, 112, 112, 64, 5, 1, 2, 128)])):
        assert p[0] == 1 and p[2] == 64, (s, p)            # 25 taps: one that it takes


def test_every_plan_can_be_encoded(plans):
    rng = np.random.default_rng(17)
    shapes = []
    for i in range(4000):
        k = int(rng.choice([1, 1, 2, 3, 3, 4, 5, 6, 7, 9, 11]))
        big = i % 50 == 0                                   # inputs around 2 GiB
        h, w = (int(v) for v in (rng.integers(900, 1700, 2) if big else 2 ** rng.uniform(0, 8, 2)))
        cin = int(rng.choice([1, 3, 4, 16, 24, 32, 48, 64, 128, 256, 512, 960, 2048])) if not big else 256
        cout = int(rng.choice([4, 8, 24, 64, 128, 192, 256, 512, 1000]))
        p = int(rng.integers(0, k + 2))
        if min(h, w) + 2 * p < k:
            continue
        shapes.append((i & 1, cin, h, w, cout, k, int(rng.integers(1, 4)), p, int(rng.choice([8, 32, 64, 96, 128, 192, 256]))))
    got = plans(shapes)
    assert len(got) == len(shapes) > 3000
    refused = [s for s, p in zip(shapes, got) if p[0] == 0]
    assert not refused, refused[:5]
    for s, p in zip(shapes, got):
        if p[0] == "-1":                                    # refused in words: only where the index arithmetic says so
            assert "index arithmetic" in p[1], (s, p)
    assert {p[2] for p in got if p[0] == 1} == {16, 32, 64} and sum(p[2] == 64 for p in got if p[0] == 1) > 50


def test_a_plan_says_what_is_launched(plans):
    """Kernel, workgroups and threads of a launch are those of the plan, for every gather; what the two special ones assume holds."""
    rng = np.random.default_rng(19)
    shapes = []
    for i in range(40000):
        cin = int(rng.choice([1, 2, 3, 4, 4, 16, 24, 32, 48, 64, 96, 128, 256, 512]))
        k = int(rng.choice([1, 3, 3, 3, 5, 7, 11]))
        h, w = (int(v) for v in 2 ** rng.uniform(0, 8, 2))
        s, p = (1, 1) if k == 3 and rng.random() < 0.7 else (int(rng.integers(1, 5)), int(rng.integers(0, k // 2 + 1)))
        if min(h, w) + 2 * p >= k:
            shapes.append((i & 1, cin, h, w, int(rng.choice([4, 8, 32, 64, 96, 128, 192, 256, 512, 1000])), k, s, p, int(rng.choice([8, 32, 64, 96, 128, 192, 256]))))
    kernels = {g: set() for g in range(7)}
    for shape, got in zip(shapes, plans(shapes)):
        ok, kernel, rows, threads, splitk, _, gather, S, sz, sw, groups = got[:11]
        assert ok == 1 and got[11:] == [kernel, groups, threads], (shape, got)
        dtype, cin, h, w, cout, k, s, p, _ = shape
        kernels[gather].add(kernel)
        if gather == 5:                                     # three taps per fetch: every K slice a whole number of groups of three chunks
            assert (k, s, p) == (3, 1, 1) and S % 6 == 0 and sz % 6 == 0 and sw % 6 == 0, (shape, got)
        if gather in (2, 6):
            assert cin <= 4, (shape, got)
        if gather == 6:                                     # patches of the input: K is not split, the pixels of a tile fit
            nb = (cout + 31) // 32
            wn = 1 if nb % 2 else 2
            high, wide = (8 // wn - 1) * s + k, 15 * s + k
            ho, wo = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
            assert splitk == 1 and sz == sw == S and threads == 256 and high * wide <= 864 and 2 * S + 16 <= 512, (shape, got)
            assert groups == (ho + 8 // wn - 1) // (8 // wn) * ((wo + 15) // 16) * nb // wn, (shape, got)
    assert all(kernels[g] for g in (0, 1, 2, 3, 5, 6))
    assert not any(kernels[g] & kernels[q] for g, q in ((5, 3), (5, 0), (5, 1), (6, 1), (6, 2), (6, 0)))      # kernels of their own, with names of their own
    assert len(kernels[5]) == 18 and len(kernels[6]) == 4                                                     # ... and every one of them is planned for


# (c_in, h, w, c_out, k, stride, pad, plan CUs), and whether the input is fetched in patches in (fp32, bf16)
FIRST_LAYERS = [
    ((3, 224, 224, 64, 7, 2, 3, 128), (True, True)),       # 392 tiles of two channel blocks
    ((3, 63, 64, 64, 7, 2, 3, 64), (False, False)),        # 32 * 32 pixels = 32 tiles of two channel blocks: as many blocks as CUs
    ((3, 65, 64, 64, 7, 2, 3, 64), (True, True)),          # 33 tiles
    ((3, 64, 64, 32, 3, 2, 1, 32), (False, False)),
    ((3, 32, 32, 16, 3, 1, 1, 128), (True, False)),        # few tiles, but small patches
    ((3, 32, 32, 16, 5, 1, 2, 128), (True, False)),
    ((3, 32, 32, 16, 7, 1, 3, 128), (False, False)),
    ((3, 64, 64, 16, 1, 1, 0, 32), (False, True)),         # four times as many tiles as CUs
    ((3, 64, 65, 16, 1, 1, 0, 32), (True, True)),
    ((3, 300, 300, 64, 11, 4, 2, 32), (False, False)),     # more places than the patch has
]


def test_first_layers_in_patches_or_gathered(plans):
    for dtype in (0, 1):
        for (s, want), p in zip(FIRST_LAYERS, plans([(dtype,) + s for s, _ in FIRST_LAYERS])):
            assert p[0] == 1 and p[6] == (6 if want[dtype] else 2), (s, dtype, p)


# (dtype, c_in, h, w, c_out, k, stride, pad, plan CUs), pixels per wave tile: 1x1 convolutions with a short K and a single channel tile
SINGLE_CHANNEL_TILE = [
    ((0, 64, 14, 14, 32, 1, 1, 0, 128), 16),
    ((0, 128, 28, 28, 32, 1, 1, 0, 128), 16),
    ((0, 96, 32, 64, 24, 1, 1, 0, 128), 16),    # 64 tiles on 128 CUs
    ((0, 96, 32, 65, 24, 1, 1, 0, 128), 32),    # 65
    ((0, 64, 56, 56, 64, 1, 1, 0, 128), 32),    # 98 of 64 channels
    ((0, 64, 5, 6, 32, 1, 1, 0, 128), 32),      # one
    ((1, 128, 14, 14, 32, 1, 1, 0, 128), 16),
    ((1, 128, 56, 56, 32, 1, 1, 0, 128), 32),
    ((1, 128, 3, 3, 20, 1, 1, 0, 128), 32),
]


def test_single_channel_tiles_on_16_or_32_pixels(plans):
    for (s, rows), p in zip(SINGLE_CHANNEL_TILE, plans([s for s, _ in SINGLE_CHANNEL_TILE])):
        assert p[0] == 1 and p[2] == rows, (s, p)


# (dtype, c_in, h, w, c_out, k, stride, pad, plan CUs[, c_out, k, stride, pad of one that shares the launch]), waves of a workgroup: fewer where a CU has several tiles,
# but in fp32 not where K is long, nor beside a lighter one that is then soon done
FEWER_WAVES = [
    ((0, 512, 28, 28, 256, 1, 1, 0, 128, 1024, 1, 2, 0), 4),
    ((0, 256, 57, 16, 512, 3, 2, 1, 128, 512, 1, 2, 0), 8),       # 128 tiles, and 128 of a ninth of K
    ((0, 512, 16, 6, 1024, 3, 2, 1, 32, 1024, 1, 2, 0), 8),
    ((0, 256, 64, 20, 512, 3, 2, 1, 128, 512, 1, 2, 0), 4),       # 160
    ((0, 512, 32, 32, 1024, 3, 2, 1, 96, 1024, 1, 2, 0), 8),      # 256 of a long K
    ((0, 64, 44, 44, 64, 3, 1, 1, 48, 0, 1, 1, 0), 4),
    ((1, 128, 28, 35, 256, 3, 1, 1, 48, 0, 1, 1, 0), 2),
    ((0, 128, 12, 34, 256, 3, 2, 1, 32, 256, 1, 2, 0), 4),        # 32, and 32 of a ninth, beside a shorter K
    ((1, 256, 29, 47, 512, 3, 1, 1, 128, 0, 1, 1, 0), 2),
    ((1, 512, 21, 40, 512, 3, 1, 1, 40, 0, 1, 1, 0), 2),
]


def test_waves_of_a_workgroup(plans):
    for (s, waves), p in zip(FEWER_WAVES, plans([s for s, _ in FEWER_WAVES])):
        assert p[0] == 1 and p[5] == (s[9] > 0) and p[3] == 64 * waves, (s, waves, p)


def test_every_joint_launch_can_be_encoded(plans):
    """Two convolutions that read the same tensor: whatever the planner joins, the encoder takes."""
    rng = np.random.default_rng(18)
    shapes = []
    for _ in range(3000):
        h, w = (int(v) for v in 2 ** rng.uniform(2, 7.5, 2))
        ks = [int(rng.choice([1, 1, 3, 5, 7])) for _ in range(2)]
        cin = int(rng.choice([4, 8, 20, 24, 32, 64, 128, 256, 512, 1024]))
        one = [(int(rng.choice([8, 24, 64, 96, 128, 256, 512, 2048])), k, int(rng.integers(1, 3)), int(rng.integers(0, k + 1))) for k in ks]
        if min(h, w) < max(ks):
            continue
        shapes.append((int(rng.integers(0, 2)), cin, h, w) + one[0] + (int(rng.choice([8, 32, 64, 96, 128, 192, 256])),) + one[1])
    got = plans(shapes)
    refused = [s for s, p in zip(shapes, got) if p[0] == 0]
    assert len(got) == len(shapes) > 2000 and not refused, refused[:5]
    assert sum(p[0] == 1 and p[5] for p in got) > 500
