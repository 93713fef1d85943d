"""CPU-only tests of the library's host logic through the C ABI (DARIS_NO_DEVICE | DARIS_VIRTUAL_TIME):
exports, error behaviour, stage split and the scheduler trace against the oracle."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2504_08795_amd as D
import workloads as wl
from lib_helpers import Session, load_et, register_plain_tasks, run_commands
from oracle import des, staging
from sched_helpers import check_trace_invariants, load_golden, model_from_golden

HOST = D.VIRTUAL_TIME | D.NO_DEVICE


def test_library_exports_every_declared_symbol(repo_root):
    hdr = "".join(open(os.path.join(repo_root, "include", f)).read() for f in sorted(os.listdir(os.path.join(repo_root, "include"))) if f.endswith(".h"))
    declared = set(re.findall(r"\b(daris_[a-z_0-9]+)\s*\(", hdr))
    assert declared, "no declarations found"
    lib = ctypes.CDLL(D.binding.LIB_PATH)
    for name in sorted(declared):
        assert hasattr(lib, name), f"{name} declared in daris.h but not exported"
    assert declared == set(D.binding.EXPORTS), declared ^ set(D.binding.EXPORTS)


def test_trace_record_is_32_bytes():
    assert D.binding.TRACE_DTYPE.itemsize == 32


def test_cu_per_partition_formula():
    assert D.daris_cu_per_partition(3, 2, 256, 3) == 128 and D.daris_cu_per_partition(2, 1, 256, 4) == 128
    assert [D.daris_cu_per_partition(n, 2, 256, 4) for n in (2, 3, 4, 5)] == [64, 96, 128, 160]
    for num, den, nmax, nc in [(1, 1, 68, 3), (3, 2, 68, 4), (7, 3, 255, 5), (6, 1, 68, 6), (1, 1, 1, 1)]:
        assert D.daris_cu_per_partition(num, den, nmax, nc) == des.partition_cus(num, den, nmax, nc)
    with pytest.raises(D.DarisError):
        D.daris_cu_per_partition(0, 1, 256, 4)


def test_error_paths():
    with pytest.raises(D.DarisError) as e:
        D.daris_create_partition(8)                      # not initialised
    assert e.value.code == D.ESTATE
    with pytest.raises(D.DarisError):
        D.daris_init(0, 0, D.NO_DEVICE)                  # NO_DEVICE needs VIRTUAL_TIME
    with Session(HOST):
        with pytest.raises(D.DarisError) as e:
            D.daris_init(0, 0, HOST)
        assert e.value.code == D.ESTATE
        for bad in (0, 257, -3):
            with pytest.raises(D.DarisError) as e:
                D.daris_create_partition(bad)
            assert e.value.code == D.EINVAL
        p = D.daris_create_partition(256)
        with pytest.raises(D.DarisError):
            D.daris_partition_set_streams(p, 0)
        with pytest.raises(D.DarisError) as e:
            D.daris_partition_set_streams(p + 1, 1)
        assert e.value.code == D.ERANGE
        layers, shp = wl.build_net("tiny")
        dnn, keep = D.make_dnn(layers, None, shp, "fp32")
        with pytest.raises(D.DarisError):
            D.daris_register_task(dnn, 0, 10, D.HP)      # period must be positive
        with pytest.raises(D.DarisError):
            D.daris_register_task(dnn, 10, 10, 7)        # priority
        t = D.daris_register_task(dnn, 10_000_000, 10_000_000, D.HP)
        with pytest.raises(D.DarisError) as e:
            D.daris_split_stages(t, 99)
        assert e.value.code == D.ERANGE
        with pytest.raises(D.DarisError) as e:
            D.daris_split_stages(t + 5, 2)
        assert e.value.code == D.ERANGE
        with pytest.raises(D.DarisError):
            D.daris_set_afet(t, 3, 100)
        with pytest.raises(D.DarisError):
            D.daris_set_afet(t, 0, 0)
        # malformed networks
        N = wl.nets
        bad = [N.Layer(op=N.OP_CONV, c_in=5, c_out=8, k=3, pad=1, in_from=-1)]
        dnn2, keep2 = D.make_dnn(bad, None, (3, 8, 8), "fp32")
        with pytest.raises(D.DarisError) as e:
            D.daris_register_task(dnn2, 10, 10, D.LP)    # c_in mismatch
        assert e.value.code == D.EINVAL
        bad = [N.Layer(op=N.OP_CONV, c_in=3, c_out=8, k=3, pad=1, in_from=0)]
        dnn3, keep3 = D.make_dnn(bad, None, (3, 8, 8), "fp32")
        with pytest.raises(D.DarisError):
            D.daris_register_task(dnn3, 10, 10, D.LP)    # reads itself
        # virtual time: a release without a table is an error, and time cannot go back
        D.daris_split_stages(t, 2)
        D.daris_release_job(t, None, None, 100)
        with pytest.raises(D.DarisError):
            D.daris_release_job(t, None, None, 50)
        with pytest.raises(D.DarisError):
            D.daris_run_until_idle()                     # no execution-time table
    with pytest.raises(D.DarisError):
        D.daris_shutdown()


def test_partition_masks_follow_cyclic_rule():
    with Session(HOST):
        ps = [D.daris_create_partition(n) for n in (96, 96, 128, 192)]
        masks = [D.daris_partition_get_mask(p) for p in ps]
        cover = np.zeros(256, int)
        start = 0
        for n, m in zip((96, 96, 128, 192), masks):
            bits = np.array([(m[i // 32] >> (i % 32)) & 1 for i in range(256)])
            assert bits.sum() == n
            want = np.zeros(256, int)
            want[[(start + i) % 256 for i in range(n)]] = 1
            assert (bits == want).all()
            cover += bits
            start = (start + n) % 256
        assert (cover == 2).all()        # 512 CUs over 256: every CU shared by exactly two partitions
    with Session(HOST):
        masks = [D.daris_partition_get_mask(D.daris_create_partition(128)) for _ in range(3)]
        cover = sum(np.array([(m[i // 32] >> (i % 32)) & 1 for i in range(256)]) for m in masks)
        assert sorted(set(cover)) == [1, 2]


@pytest.mark.parametrize("net,ks", [("tiny", (1, 2, 3, 4)), ("resnet18", (1, 2, 3, 4, 6)), ("resnet50", (1, 4, 5)),
                                    ("vgg16", (1, 3, 4)), ("mobilenet_v2", (1, 3, 4))])
def test_stage_split_matches_oracle(net, ks):
    layers, shp = wl.build_net(net)
    macs = wl.net_macs(layers, shp)
    legal = staging.legal_cuts(layers)
    with Session(HOST):
        D.daris_create_partition(64)
        dnn, keep = D.make_dnn(layers, None, shp, "fp32")
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        assert D.daris_get_stage_cuts(t) == [0]
        for k in ks:
            D.daris_split_stages(t, k)
            assert D.daris_get_stage_cuts(t) == staging.split(macs, legal, k), (net, k)
        with pytest.raises(D.DarisError):
            D.daris_split_stages(t, len(legal) + 2)


def _check_plan(pl, name):
    """What the kernels and their grids assume about a dense convolution's launch plan."""
    M, N, S = pl["M"], pl["N"], pl["S"]
    z = pl["splitk"]
    rows = pl["rows"]                                                       # pixels per wave tile
    block = 16 if rows == 16 else 32                                        # width of a channel block
    assert rows in (16, 32, 64) and pl["grid_y"] == 1 and pl["grid_z"] == 1 and pl["grid_x"] >= 1, name
    if z > 1:
        assert pl["ws_bytes"] >= z * M * N * 4, name                       # one fp32 partial tile set per K slice
    tn, nw = pl["tn"], pl["nw"]
    assert tn in (1, 2) and nw in (2, 4, 8) and pl["threads"] == 64 * nw, name
    kname = D.daris_kernel_name(pl["kernel_id"])
    gather = pl["gather"]
    special = {D.GATHER_TAPS: "taps_", D.GATHER_IMAGE: "image_"}.get(gather, "")
    family = {16: "conv_wave16_", 32: "conv_wave_", 64: "conv_wave64_"}[rows]
    assert kname.endswith(f"t{tn}w{nw}") and kname.startswith((family + special + "f32_", family + special + "bf16_")), (name, kname, gather)
    if rows != 32:
        assert gather in (D.GATHER_ROWS, D.GATHER_TAPS), name
    if rows == 64:
        assert tn == 2 and "f32" in kname, name
    nb = (N + block - 1) // block
    if gather == D.GATHER_IMAGE:                                             # a wave owns two rows of 16 pixels and a channel block over all of K
        wn = 1 if nb % 2 else 2
        assert rows == 32 and tn == 1 and nw == 4 and z == 1 and pl["ws_bytes"] == 0 and pl["sz"] == pl["sw"] == S, name
        assert S * (8 if "f32" in kname else 16) == pl["Kpad"] and pl["NTn"] == nb and pl["G"] == nb // wn and pl["xmode"] == 0, name
        assert pl["grid_x"] == pl["G"] * pl["MT"] and pl["MT"] * (128 // wn) >= M and f"_n{wn}_" in kname, name
        return
    assert (nb + tn - 1) // tn == pl["NTn"] and pl["MT"] == (M + rows - 1) // rows, name
    if rows >= 32:
        assert nb % tn == 0, name
    assert S * (8 if "f32" in kname else 16) * (32 // block) == pl["Kpad"], name
    if rows == 16:
        assert z == 1, name                                                  # the reason these tiles exist
    # the z slices cover all K steps and none is empty; the nw waves cover their slice
    assert z >= 1 and pl["sz"] * z >= S and pl["sz"] * (z - 1) < S, name
    assert pl["sw"] * nw >= pl["sz"] and pl["sw"] >= 1, name
    assert pl["G"] == pl["NTn"] * z, name
    # workgroup order: every (pixel tile, weight group) is reached, groups with equal id mod 8 stay together
    if pl["xmode"] == 1:
        assert pl["G"] % 8 == 0 and pl["grid_x"] == pl["G"] * pl["MT"], name
    elif pl["xmode"] == 2:
        r = 8 // pl["G"]
        assert 8 % pl["G"] == 0 and pl["grid_x"] == 8 * ((pl["MT"] + r - 1) // r), name
    else:
        assert pl["xmode"] == 0 and pl["grid_x"] == pl["G"] * pl["MT"], name


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("net", ["tiny", "resnet18", "resnet50", "vgg16", "mobilenet_v2"])
def test_launch_plans_satisfy_kernel_assumptions(net, dtype):
    layers, shp = wl.build_net(net)
    with Session(HOST):
        D.daris_create_partition(64)
        dnn, keep = D.make_dnn(layers, None, shp, dtype)
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        plans = [D.daris_get_launch_plan(t, l) for l in range(len(layers))]
    n_pairs = n_fused = 0
    es = 4 if dtype == "fp32" else 2
    for l, (L, pl) in enumerate(zip(layers, plans)):
        if not pl["dense_conv"]:
            if pl["pair_with"] >= 0:
                # a depthwise 3x3 convolution computed inside the launch of the 1x1 convolution that follows it: what that
                # kernel's producer assumes about the two layers and about the plan
                o, Lo = plans[l + 1], layers[l + 1]
                assert pl["pair_with"] == l + 1 and not pl["pair_lead"] and o["pair_with"] == l and o["pair_lead"]
                assert L.op == wl.nets.OP_CONV and L.groups == L.c_in == L.c_out and L.k == 3 and L.pad == 1 and L.stride in (1, 2)
                assert Lo.op == wl.nets.OP_CONV and Lo.groups == 1 and Lo.k == 1 and Lo.stride == 1 and Lo.pad == 0 and Lo.in_from == l
                assert all(q.in_from != l and q.res_from != l for q in layers[l + 2:])      # nobody else needs the tensor
                assert (L.c_out * es) % 64 == 0 and o["rows"] == 32 and o["Kpad"] == L.c_out
                assert o["S"] % 2 == 0 and o["sz"] % 2 == 0 and o["sw"] % 2 == 0             # K in whole chunks of two steps
                assert dtype == "bf16" or o["tn"] == 1
                assert not (dtype == "bf16" and o["nw"] == 8)                                 # no such kernel variant
                assert o["MT"] >= 96 and o["NTn"] == 1                                         # the shapes for which it is faster
                n_fused += 1
            continue
        _check_plan(pl, f"{net} {dtype} layer {l} {L.name}")
        if pl["pair_with"] >= 0 and not plans[pl["pair_with"]]["dense_conv"]:
            continue                                                           # leads a fused depthwise layer (checked above)
        if pl["pair_with"] >= 0:
            o = plans[pl["pair_with"]]
            assert abs(pl["pair_with"] - l) == 1 and o["pair_with"] == l and pl["pair_lead"] != o["pair_lead"]
            assert pl["pair_lead"] == (pl["pair_with"] < l)                    # issued at the later layer
            assert layers[l].in_from == layers[pl["pair_with"]].in_from       # both read the same tensor
            assert o["kernel_id"] == pl["kernel_id"]
            light = pl if wl.net_macs(layers, shp)[l] < wl.net_macs(layers, shp)[pl["pair_with"]] else o
            assert light["splitk"] == 1                                        # the second problem never splits K across workgroups
            n_pairs += 1
    assert n_pairs // 2 == {"tiny": 0, "resnet18": 3, "resnet50": 4, "vgg16": 0, "mobilenet_v2": 0}[net]
    # MobileNetV2: the blocks on the 112 x 112 and 56 x 56 maps (enough pixel tiles, one channel block); in bf16 the 144-channel
    # hidden layer is not a whole number of 64-byte rows
    assert n_fused == ({"fp32": 3, "bf16": 2}[dtype] if net == "mobilenet_v2" else 0)


@pytest.mark.parametrize("plan_cus", [32, 64, 96, 160, 256])
def test_launch_plans_for_other_partition_sizes(plan_cus):
    """daris_set_plan_cus: the plans still satisfy what the kernels assume, and they do change with the size."""
    with pytest.raises(D.DarisError):
        D.daris_set_plan_cus(96)                      # needs an initialised library
    changed = 0
    for net in ("resnet18", "resnet50", "vgg16", "mobilenet_v2"):
        layers, shp = wl.build_net(net)
        for dtype in ("fp32", "bf16"):
            got = []
            for cus in (plan_cus, 128):
                with Session(HOST):
                    for bad in (0, 7, 257):
                        with pytest.raises(D.DarisError):
                            D.daris_set_plan_cus(bad)
                    D.daris_set_plan_cus(cus)
                    D.daris_create_partition(64)
                    dnn, keep = D.make_dnn(layers, None, shp, dtype)
                    t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
                    got.append([D.daris_get_launch_plan(t, l) for l in range(len(layers))])
            for l, pl in enumerate(got[0]):
                if pl["dense_conv"]:
                    _check_plan(pl, f"{net} {dtype} plan_cus {plan_cus} layer {l}")
            changed += got[0] != got[1]
    assert changed >= 4
    if plan_cus == 96:      # 98 tiles of 64 channels would take two rounds on 96 CUs: ResNet-18's first block uses 196 tiles of 32
        layers, shp = wl.build_net("resnet18")
        with Session(HOST):
            D.daris_set_plan_cus(96)
            D.daris_create_partition(96)
            dnn, keep = D.make_dnn(layers, None, shp, "fp32")
            t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
            pl = D.daris_get_launch_plan(t, 2)
        assert layers[2].name == "l1b0.c1" and pl["tn"] == 1 and pl["MT"] * pl["NTn"] == 196 and pl["splitk"] == 1


def test_fused_depthwise_follows_the_stage_split():
    """A depthwise layer computed inside the next layer's launch is taken out of it while a stage cut separates the two (else
    a stage could consist of that layer alone and launch nothing), and put back when the cut goes away."""
    layers, shp = wl.build_net("mobilenet_v2")
    legal = staging.legal_cuts(layers)
    with Session(HOST):
        D.daris_create_partition(128)
        dnn, keep = D.make_dnn(layers, None, shp, "fp32")
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        fused = lambda: [l for l in range(len(layers)) if D.daris_get_launch_plan(t, l)["pair_with"] == l + 1]      # noqa: E731
        at_first = fused()
        assert len(at_first) == 3 and all(layers[l].groups > 1 for l in at_first)
        cuttable = [l for l in at_first if l in legal]                # (inside a block with a shortcut no cut is legal)
        assert len(cuttable) == 2
        D.daris_split_stages(t, len(legal) + 1)                        # with every legal cut in use, only the uncuttable one stays fused
        assert D.daris_get_stage_cuts(t) == [0] + [c + 1 for c in legal]
        assert fused() == [l for l in at_first if l not in legal]
        for l in cuttable:
            assert D.daris_get_launch_plan(t, l + 1)["pair_with"] == -1
        D.daris_split_stages(t, 3)
        assert fused() == at_first
        D.daris_split_stages(t, 1)
        assert fused() == at_first


def test_launch_plans_of_odd_shapes():
    rng = np.random.default_rng(5)
    N = wl.nets
    with Session(HOST):
        D.daris_create_partition(64)
        for i in range(150):
            cin, cout = int(rng.integers(1, 700)), int(rng.integers(1, 700))
            k = int(rng.choice([1, 3, 5, 7]))
            h, w = int(rng.integers(k, 70)), int(rng.integers(k, 70))
            s = int(rng.choice([1, 2]))
            layers = [N.Layer(op=N.OP_CONV, c_in=cin, c_out=cout, k=k, stride=s, pad=k // 2, act=1, in_from=-1)]
            for dtype in ("fp32", "bf16"):
                dnn, keep = D.make_dnn(layers, None, (cin, h, w), dtype)
                t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
                _check_plan(D.daris_get_launch_plan(t, 0), f"{cin}x{h}x{w}->{cout} k{k} s{s} {dtype}")


def test_stage_split_known_results():
    """Per-stage MAC totals at the benchmark configurations (integers from the layer tables)."""
    def stage_macs(net, k):
        layers, shp = wl.build_net(net)
        macs = wl.net_macs(layers, shp)
        first = staging.split(macs, staging.legal_cuts(layers), k) + [len(layers)]
        return [sum(macs[a:b]) for a, b in zip(first, first[1:])], first
    m, first = stage_macs("tiny", 2)
    assert m == [5_160_960, 7_118_848]
    m, first = stage_macs("resnet18", 3)
    assert sum(m) == 1_814_073_344 and max(m) < 650_000_000
    # a residual block is never cut in the middle: every stage starts at a block boundary (or the stem pool)
    layers, _ = wl.build_net("resnet18")
    for f in first[1:-1]:
        assert layers[f].name.endswith((".ds", ".c1")) or layers[f].name in ("stem.pool", "gap", "fc")


@pytest.mark.parametrize("name", ["sched_single_task.json", "sched_hp_preempts_lp.json", "sched_admission_migration.json",
                                  "sched_migration_target_choice.json", "sched_forced_migration_at_boundary.json",
                                  "sched_hp_admission.json"])
def test_library_reproduces_golden_traces(name):
    g, cmds, et, want = load_golden(name)
    lib_flags = {"no_last": D.NO_LAST, "no_prior": D.NO_PRIOR, "no_fixed": D.NO_FIXED, "hp_admission": D.HP_ADMISSION}
    with Session(HOST | sum(lib_flags[f] for f in g.get("flags", []))):
        register_plain_tasks(g["partitions"], g["tasks"])
        load_et(et, len(g["partitions"]))
        run_commands(cmds)
        got = D.trace_read_all()
    for a, b in zip(got, want):
        assert a == b, f"first difference at seq {a[0]}: got {a}, want {b}"
    assert len(got) == len(want)


def _oracle_and_library(ts, et, afet, flags=0, n_streams=None, migrations=()):
    n_streams = n_streams or [1] * len(ts.partitions)
    tasks = [des.TaskParam(t.period_ns, t.deadline_ns, t.priority, list(afet[i])) for i, t in enumerate(ts.tasks)]
    cmds = [("release", t, i) for t, i, _ in ts.releases()] + list(migrations)
    cmds.sort(key=lambda c: c[1])
    oflags = 0
    for lf, of in ((D.NO_LAST, des.F_NO_LAST), (D.NO_PRIOR, des.F_NO_PRIOR), (D.NO_FIXED, des.F_NO_FIXED), (D.HP_ADMISSION, des.F_HP_ADMISSION)):
        if flags & lf:
            oflags |= of
    m = des.SchedulerModel(n_streams, tasks, flags=oflags)
    want = des.run_virtual(m, cmds, et)
    with Session(HOST | flags):
        register_plain_tasks(n_streams, [dict(period=t.period, deadline=t.deadline, prio=t.prio, afet=t.afet) for t in tasks])
        load_et(et, len(n_streams))
        dec = run_commands(cmds)
        got = D.trace_read_all()
        stats = [D.daris_get_stats(i) for i in range(len(tasks))]
    return m, want, got, stats, dec


def test_response_percentiles_agree_with_the_library_statistics():
    """The harness derives per-job response times from the trace; their extremes and mean must be the library's."""
    from paper_2504_08795_amd import harness
    ts = wl.make_taskset(2, n_jobs=25)
    et = wl.virtual_et_table(ts, load_scale=25.0)
    afet = [[int(np.mean(et[i][j][0][:8])) for j in range(t.n_stages)] for i, t in enumerate(ts.tasks)]
    m, want, got, stats, dec = _oracle_and_library(ts, et, afet)
    prios = [t.priority for t in ts.tasks]
    pct = harness.response_percentiles(got, prios)
    for name, prio in (("hp", wl.HP), ("lp", wl.LP)):
        sel = [s for s, p in zip(stats, prios) if p == prio and s["completed"] > 0]
        assert pct[name]["jobs"] == sum(s["completed"] for s in sel)
        assert pct[name]["min_ms"] == round(min(s["resp_min_ns"] for s in sel) / 1e6, 4)
        assert pct[name]["max_ms"] == round(max(s["resp_max_ns"] for s in sel) / 1e6, 4)
        assert pct[name]["min_ms"] <= pct[name]["p50_ms"] <= pct[name]["p99_ms"] <= pct[name]["max_ms"]


@pytest.mark.parametrize("config,load,flags,ns", [
    (1, 300.0, 0, 1), (2, 25.0, 0, 1), (3, 18.0, 0, 1), (4, 22.0, 0, 1), (2, 30.0, 0, 2), (3, 14.0, D.NO_LAST, 1), (2, 25.0, D.NO_PRIOR, 1),
    (4, 22.0, D.NO_FIXED, 1), (2, 45.0, D.HP_ADMISSION, 1), (5, 12.0, 0, 1)])
def test_trace_bit_exact_against_oracle(config, load, flags, ns):
    ts = wl.make_taskset(config, n_jobs=80 if config != 5 else 40)
    et = wl.virtual_et_table(ts, load_scale=load)
    afet = [[int(np.mean(et[i][j][0][:8])) for j in range(t.n_stages)] for i, t in enumerate(ts.tasks)]
    rel = ts.releases()
    mig = [("migrate", rel[n][0], (n // 7) % len(ts.tasks), (n // 3) % len(ts.partitions)) for n in range(25, len(rel), 61)]
    m, want, got, stats, dec = _oracle_and_library(ts, et, afet, flags, [ns] * len(ts.partitions), mig)
    for a, b in zip(got, want):
        assert a == b, f"first difference at seq {a[0]}: library {a}, oracle {b}"
    assert len(got) == len(want) and len(got) > 100
    check_trace_invariants(got, m.n_streams, [t.p.prio for t in m.tasks], [len(t.p.afet) for t in m.tasks],
                           flags=m.flags)
    for s, o in zip(stats, m.stats()):
        assert (s["released"], s["accepted"], s["completed"], s["missed"], s["rejected_admission"], s["rejected_overrun"]) == \
               (o["released"], o["accepted"], o["completed"], o["missed"], o["rejected_admission"], o["rejected_overrun"])
        if o["responses"]:
            assert (s["resp_min_ns"], s["resp_max_ns"], s["resp_sum_ns"]) == (min(o["responses"]), max(o["responses"]), sum(o["responses"]))
        assert s["partition"] == o["ctx"]


def test_run_periodic_equals_explicit_releases():
    ts = wl.make_taskset(2, n_jobs=30)
    et = wl.virtual_et_table(ts, load_scale=25.0)
    afet = [[int(np.mean(et[i][j][0][:8])) for j in range(t.n_stages)] for i, t in enumerate(ts.tasks)]
    m, want, got, stats, dec = _oracle_and_library(ts, et, afet)
    with Session(HOST):
        register_plain_tasks([1] * 3, [dict(period=t.period_ns, deadline=t.deadline_ns, prio=t.priority, afet=afet[i]) for i, t in enumerate(ts.tasks)])
        load_et(et, 3)
        for i in range(len(ts.tasks)):
            D.daris_task_set_io(i, None, 4, None, 4)
        D.daris_run_periodic(None, [30] * len(ts.tasks))
        got2 = D.trace_read_all()
    assert got2 == got == want


def test_mret_accessor_and_window():
    with Session(HOST):
        register_plain_tasks([1], [dict(period=1000, deadline=1000, prio=D.LP, afet=[50])])
        D.daris_set_window(3)
        vals = [10, 90, 20, 20, 20, 20]
        D.daris_set_virtual_time(0, 0, 0, 0, len(vals), np.array(vals))
        assert D.daris_get_mret(0, 0) == 50          # AFET until the stage has run
        seen = []
        for m in range(len(vals)):
            D.daris_release_job(0, None, None, m * 1000)
            D.daris_run_until_idle()
            seen.append(D.daris_get_mret(0, 0))
        assert seen == [10, 90, 90, 90, 20, 20]      # window of 3 executions


def test_limits_and_degenerate_schedules():
    """Maximum stream count, one-job and zero-job runs, a window of one, the deepest legal split of a network."""
    with Session(HOST):
        p = D.daris_create_partition(1)                   # smallest partition
        D.daris_partition_set_streams(p, 8)               # largest stream count
        with pytest.raises(D.DarisError):
            D.daris_partition_set_streams(p, 9)
        layers, shp = wl.build_net("resnet18")
        legal = staging.legal_cuts(layers)
        dnn, keep = D.make_dnn(layers, None, shp, "fp32")
        t = D.daris_register_task(dnn, 1000, 1000, D.LP)
        kmax = len(legal) + 1
        D.daris_split_stages(t, kmax)                     # every legal cut taken
        assert D.daris_get_stage_cuts(t) == [0] + [c + 1 for c in legal]
        D.daris_set_window(1)
        for j in range(kmax):
            D.daris_set_afet(t, j, 1)
            D.daris_set_virtual_time(t, j, p, 0, 3, np.array([1, 1, 1]))
        D.daris_task_set_io(t, None, 1, None, 1)
        D.daris_run_periodic(None, [0])                   # nothing to release: returns at once
        assert D.trace_read_all() == []
        D.daris_run_periodic(None, [3])
        st = D.daris_get_stats(t)
        assert (st["released"], st["completed"], st["missed"]) == (3, 3, 0) and st["resp_max_ns"] == kmax
        tr = D.trace_read_all()
        assert sum(1 for r in tr if r[2] == D.T_DISPATCH) == 3 * kmax
    with Session(HOST):
        for _ in range(255):
            D.daris_create_partition(256)                 # as many fully overlapping partitions as the handle type allows
        with pytest.raises(D.DarisError):
            D.daris_create_partition(256)


def test_overrun_and_hp_queue_order():
    """A period far shorter than the execution time: LP releases are rejected as overruns, HP releases queue up FIFO and
    every one of them is eventually served in release order."""
    # the LP task's AFET (5) under-estimates its real time (25): job 0 is admitted (u = 0.5), the releases at 10 and 20
    # find it still active (overrun), and from then on MRET = 25 makes u = 2.5, which eq. 12 rejects
    tasks = [dict(period=10, deadline=10, prio=D.HP, afet=[25]), dict(period=10, deadline=10, prio=D.LP, afet=[5])]
    with Session(HOST):
        register_plain_tasks([1, 1], tasks)
        for i in range(2):
            for k in range(2):
                D.daris_set_virtual_time(i, 0, k, 0, 6, np.full(6, 25))
        dec = []
        for m in range(6):
            for i in range(2):
                dec.append((i, D.daris_release_job(i, None, None, m * 10)))
        D.daris_run_until_idle()
        hp, lp = D.daris_get_stats(0), D.daris_get_stats(1)
        assert hp["completed"] == 6 and hp["rejected_overrun"] == 0 and hp["missed"] >= 4
        assert (lp["completed"], lp["rejected_overrun"], lp["rejected_admission"]) == (1, 2, 3)
        assert [d for i, d in dec if i == 0][:3] == [D.ACCEPTED, D.QUEUED, D.QUEUED]
        tr = D.trace_read_all()
        started = [r[8] for r in tr if r[2] == D.T_ACCEPT and r[6] == 0]
        assert started == sorted(started) == list(range(6))


def _code_object_kernels(name):
    """[(mangled name, {what: number})] of a device code object, as its metadata has them."""
    import shutil
    import subprocess
    co = os.path.join(os.path.dirname(D.LIB_PATH), "csrc", name + ".co")
    tool = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
    if not (os.path.exists(co) and os.path.exists(tool)):
        pytest.skip("code object or llvm-readelf not available")
    notes = subprocess.run([tool, "--notes", co], check=True, capture_output=True, text=True).stdout
    assert "hidden_" not in notes
    what = ("kernarg_segment_size", "private_segment_fixed_size", "group_segment_fixed_size", "vgpr_count", "max_flat_workgroup_size")
    return [(re.search(r"\.name:\s+(\S+)", block).group(1), {w: int(re.search(r"\." + w + r":\s+(\d+)", block).group(1)) for w in what}) for block in notes.split(".agpr_count:")[1:]]


# code object: {kernel: (bytes of its argument block, how many instances)}
DEVICE_KERNELS = {
    "daris_kernels": {"conv_wave_kernel": (160, 42), "conv_wave_pair_kernel": (324, 30), "conv_wave16_kernel": (160, 12), "conv_wave16_pair_kernel": (324, 12), "conv_wave_dw_kernel": (192, 7), "conv_large_kernel": (160, 4),
                      "splitk_reduce_kernel": (48, 2), "dwconv_kernel": (72, 2), "maxpool_kernel": (48, 2), "gavgpool_kernel": (48, 2), "fc_kernel": (56, 2), "ingest_kernel": (28, 2),
                      "egress_kernel": (28, 2), "cu_probe_kernel": (12, 1)},
    "daris_taps_kernels": {"conv_taps_kernel": (160, 9), "conv_taps16_kernel": (160, 6), "conv_taps_large_kernel": (160, 4)},
    "daris_image_kernels": {"conv_image_kernel": (160, 4)},
    "daris_block_kernels": {"conv_block_kernel": (160, 6)},
    "daris_point_kernels": {"dwconv_window_kernel": (88, 2), "maxpool_window_kernel": (64, 4)},
}


@pytest.mark.parametrize("co", sorted(DEVICE_KERNELS))
def test_code_object_kernels_match_the_argument_structures(co):
    """Every kernel of every device code object takes exactly the argument block the host encoders write (sizes of the
    structures in csrc/kernels.h), needs no hidden arguments and no scratch: what a bare AQL packet can provide."""
    want, seen = DEVICE_KERNELS[co], {}
    for name, has in _code_object_kernels(co):
        size, scratch, lds = has["kernarg_segment_size"], has["private_segment_fixed_size"], has["group_segment_fixed_size"]
        base = [k for k in want if re.search(r"\d+" + k + r"(I|E)", name)]
        assert len(base) == 1, name
        assert size == want[base[0]][0], (name, size)
        assert scratch == 0 and lds <= 65536, (name, scratch, lds)
        seen[base[0]] = seen.get(base[0], 0) + 1
    assert seen == {k: n for k, (_, n) in want.items()}


def test_every_code_object_is_checked():
    from paper_2504_08795_amd import build
    assert set(build.DEVICE_SOURCES.values()) == set(DEVICE_KERNELS)


def test_a_simd_has_room_for_three_wide_bf16_row_tiles():
    """Tiles of 32 x 64 in bf16 over whole rows, in workgroups of two and four waves: grids of up to three such workgroups a CU run in one round
    if a SIMD, whose lanes have 512 registers handed out in eights, has room for three of the waves."""
    found = {name: has["vgpr_count"] for name, has in _code_object_kernels("daris_kernels") if re.search(r"conv_wave_(pair_)?kernelILb1ELi2ELi[24]ELi3E", name)}
    assert len(found) == 4 and all(512 // (-(-v // 8) * 8) >= 3 for v in found.values()), found


def test_layer_rooflines_follow_the_layer_tables():
    """The harness's roofline helper is host arithmetic on the layer tables: FLOPs are twice the pinned MAC counts, bytes
    count every weight once, and the per-network sums are the figures the profiles quote."""
    from paper_2504_08795_amd import harness
    want_macs = {"resnet18": 1814073344, "resnet50": 4089184256, "vgg16": 15470264320, "mobilenet_v2": 300774272, "tiny": 12279808}
    want_us = {("resnet18", "fp32"): 12.06, ("resnet50", "bf16"): 13.51, ("vgg16", "fp32"): 140.59, ("mobilenet_v2", "fp32"): 8.61}
    for net, macs in want_macs.items():
        layers, shp = wl.build_net(net)
        r = harness.layer_rooflines(layers, shp, "fp32")
        assert sum(x[0] for x in r) == 2.0 * macs
        es = 4
        weights = sum(L.c_out * (L.c_in // L.groups) * L.k * L.k for L in layers if L.op == wl.nets.OP_CONV) + \
            sum(L.c_out * L.c_in for L in layers if L.op == wl.nets.OP_FC)
        assert sum(x[1] for x in r) > weights * es                       # plus activations and biases
        for x in r:
            assert x[2] == max(x[0] / 416.7e12, x[1] / 8e12) * 1e6
    for (net, dtype), us in want_us.items():
        layers, shp = wl.build_net(net)
        assert round(sum(x[2] for x in harness.layer_rooflines(layers, shp, dtype)), 2) == us
    # a launch of several layers: the tensors between them are neither read nor written
    assert harness.launches_of([0, 0, 3, 1, 0, 2]) == [[0, 1, 2], [3], [4, 5]]
    layers, shp = wl.build_net("resnet18")
    (f0, b0, _), (f1, b1, _) = harness.layer_rooflines(layers, shp, "fp32")[:2]
    assert harness.launch_roofline(layers, shp, "fp32", [0, 1])[:2] == (f0 + f1, b0 + b1 - 2 * 4 * 64 * 112 * 112)
    ds = next(l for l, L in enumerate(layers) if layers[l + 1].in_from == L.in_from)                        # a shortcut and its block's first convolution read one tensor
    (f0, b0, _), (f1, b1, _) = harness.layer_rooflines(layers, shp, "fp32")[ds:ds + 2]
    assert harness.launch_roofline(layers, shp, "fp32", [ds, ds + 1])[:2] == (f0 + f1, b0 + b1 - 4 * 64 * 56 * 56)
    ts = wl.make_taskset(2)
    assert [round(v, 2) for v in harness.taskset_roofline_us(ts)] == [12.06] * 4


def _check_slot_lifetimes(layers, plans, name):
    """Replay the launches in issue order: a launch group (a layer, or the two layers of a joint launch, issued at the later
    one) must not write a slot that holds a tensor some launch at or after this group still reads, and must not write a
    slot it reads itself."""
    n = len(layers)
    issue = [max(l, plans[l]["pair_with"]) for l in range(n)]                     # when layer l's launch is issued
    # a depthwise layer computed inside the next layer's launch: its output is neither written nor read, and its input is
    # read by that launch
    fused_dw = [not plans[l]["dense_conv"] and plans[l]["pair_with"] >= 0 for l in range(n)]
    readers = {}                                                                  # tensor (layer index, -1 = input) -> issue times of its readers
    for l, L in enumerate(layers):
        if L.in_from >= 0 and fused_dw[L.in_from]:
            continue
        readers.setdefault(L.in_from, []).append(issue[l])
        if L.res_from >= 0:
            readers.setdefault(L.res_from, []).append(issue[l])
    holds = {}                                                                    # slot -> tensor it holds
    if plans[0]["in_slot"] >= 0 and layers[0].in_from == -1:
        holds[plans[0]["in_slot"]] = -1
    for l in range(n):
        group = [q for q in range(n) if issue[q] == issue[l]]
        s = plans[l]["out_slot"]
        if s < 0 or fused_dw[l]:
            continue
        for q in group:                                                           # nothing the group reads may be overwritten by it
            reads_input = not (layers[q].in_from >= 0 and fused_dw[layers[q].in_from])
            assert (s != plans[q]["in_slot"] or not reads_input) and s != plans[q]["res_slot"], (name, l, q, s)
        if s in holds:
            old = holds[s]
            assert all(t < issue[l] for t in readers.get(old, [])), (name, "layer", l, "overwrites tensor", old, "still read at", readers.get(old))
        holds[s] = l
    for l, L in enumerate(layers):                                                # and every read finds its tensor where the plan says
        assert plans[l]["in_slot"] == (plans[L.in_from]["out_slot"] if L.in_from >= 0 else plans[l]["in_slot"])
        if L.res_from >= 0:
            assert plans[l]["res_slot"] == plans[L.res_from]["out_slot"]


def paired_residual_net():
    """A graph none of the configured networks has: the EARLIER member of a joint launch (L2) carries a residual operand
    (L0's output) whose last reader it is, so that operand's buffer falls free exactly when the later member's output is
    placed."""
    c = lambda i, r=-1, co=32, k=3: N_.Layer(op=N_.OP_CONV, c_in=32 if i >= 0 else 3, c_out=co, k=k, stride=1, pad=k // 2, act=1, in_from=i, res_from=r)  # noqa: E731
    layers = [c(-1), c(0), c(1, 0), c(1, -1, 32, 1), c(3, 2), N_.Layer(op=N_.OP_GAVGPOOL, c_in=32, c_out=32, in_from=4),
              N_.Layer(op=N_.OP_FC, c_in=32, c_out=10, in_from=5)]
    return layers, (3, 12, 12)


N_ = wl.nets


@pytest.mark.parametrize("net", ["resnet18", "resnet50", "mobilenet_v2", "vgg16", "paired_residual"])
def test_activation_slots_outlive_their_readers(net):
    layers, shp = paired_residual_net() if net == "paired_residual" else wl.build_net(net)
    with Session(HOST):
        D.daris_create_partition(64)
        dnn, keep = D.make_dnn(layers, None, shp, "fp32")
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        plans = [D.daris_get_launch_plan(t, l) for l in range(len(layers))]
    if net == "paired_residual":
        assert plans[2]["pair_with"] == 3 and plans[3]["pair_lead"] == 1          # the case is what it claims to be
        assert plans[3]["out_slot"] != plans[2]["res_slot"]
    _check_slot_lifetimes(layers, plans, net)
    assert len({p["out_slot"] for p in plans if p["out_slot"] >= 0}) <= 6         # and buffers are still shared


@pytest.mark.parametrize("read", [0, 1])
def test_members_of_a_joint_launch_write_to_places_of_their_own(read):
    """... also where nothing reads one of them."""
    layers = [N_.Layer(op=N_.OP_CONV, c_in=64, c_out=64, k=3, stride=2, pad=1, in_from=-1), N_.Layer(op=N_.OP_CONV, c_in=64, c_out=64, k=1, stride=2, in_from=-1),
              N_.Layer(op=N_.OP_CONV, c_in=64, c_out=64, k=1, in_from=read)]
    with Session(HOST):
        D.daris_create_partition(64)
        dnn, keep = D.make_dnn(layers, None, (64, 28, 28), "fp32")
        t = D.daris_register_task(dnn, 10**7, 10**7, D.LP)
        plans = [D.daris_get_launch_plan(t, l) for l in range(3)]
    assert plans[0]["pair_with"] == 1
    assert len({plans[0]["in_slot"], plans[0]["out_slot"], plans[1]["out_slot"]}) == 3, plans
    _check_slot_lifetimes(layers, plans, "one member unread")


def test_timeout_setter_validates():
    with pytest.raises(D.DarisError) as e:
        D.daris_set_timeout(0)
    assert e.value.code == D.EINVAL
    D.daris_set_timeout(20_000_000_000)


def test_bench_roofline_helpers():
    """`bench.py`'s pure helpers: every convolution kernel family is priced against the MFMA peak of its arithmetic type, the
    memory-bound kernels against HBM, and the committed traffic summaries carry a figure for every dominant-kernel candidate."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    for i in range(1, 64):
        name = D.daris_kernel_name(i)
        if name == "?":
            break
        r = bench.kernel_roofline(name, 10, 0.1, 2.0e9)               # 10 launches, 0.1 ms, 2 GFLOP
        if name.startswith("conv_wave"):
            peak = 2500.0 if "_bf16_" in name else 416.7
            assert r["bound"] == "mfma" and r["peak"] == peak and r["unit"] == "TFLOP/s", name
            assert r["achieved"] == 20.0 and r["frac"] == round(20.0 / peak, 5) and r["avg_launch_us"] == 10.0, (name, r)
        else:
            assert r["bound"] == "hbm" and r["peak"] == 8000.0 and r["achieved"] is None, name
    assert i > 30
    for config, kernels in ((4, ("conv_wave_f32_t2w8", "conv_wave_f32_t1w8", "conv_wave_taps_f32_t1w8", "conv_wave_taps_f32_t2w8", "conv_wave16_taps_f32_t1w8", "conv_wave16_taps_f32_t2w8",
                                 "conv_wave64_taps_f32_t2w2", "conv_wave64_taps_f32_t2w4", "conv_wave64_taps_f32_t2w8", "fc")),
                            (3, ("conv_wave_bf16_t2w4", "conv_wave_bf16_t1w4", "conv_wave16_bf16_t2w4", "conv_wave16_taps_bf16_t1w8", "conv_wave16_taps_bf16_t2w8")),
                            (2, ("conv_wave16_f32_t1w8", "conv_wave16_taps_f32_t1w8", "conv_wave16_taps_f32_t2w8", "conv_wave_taps_f32_t2w8"))):
        for k in kernels:
            t = bench.read_traffic(config, k)
            assert isinstance(t, int) and t > 10_000, (config, k, t)
    assert bench.read_traffic(4, "no_such_kernel") is None
    assert set(bench.WORKLOADS) == {2, 3, 4} and bench.JOBS_PER_TASK_PER_STEP == 32
