"""The work whose speed counts: batch-1 inference of the configured networks through the public calls of the library.

Three ways in which a program uses it, and every listed case is one of them:

* ``forward`` / ``static``  one frame, now: ``daris_forward`` (or its no-allocation twin ``daris_forward_static``) on one
  partition, the call returns with the logits;
* ``jobs``   a synchronous release: every task of a set gets one frame through ``daris_release_job``, and the program
  waits until all jobs have passed the scheduler stage by stage;
* ``loop``   a saturated server: buffers full of frames are given to every task (``daris_task_set_io``), and each task's
  next job is released the instant its previous one ends (``daris_run_closed_loop``).

A case is text and numbers: ``tasks`` = "n*net/dtype/priority/stages+..." in registration order, ``parts`` = CUs of each
partition, ``h`` x ``w`` = frame size, ``jobs`` = jobs of a task that costs as much as one ResNet-18 (heavier networks get
fewer, so that the partitions stay busy to the end).

The networks' weights belong to the program and stay as they are; the frames (and nothing else) come from the seed.  The
library is one per process: preparing a case of another set of tasks shuts it down and sets it up again.
"""
import dataclasses
import functools

import torch

import paper_2504_08795_amd as D
import workloads as wl
from workloads.nets import OP_CONV, OP_FC

WEIGHT_SEED = 20250408
PERIOD_NS = {"hp": 100_000_000, "lp": 200_000_000}  # far above what a job takes: every release is admitted
JOB_WEIGHT = {"tiny": 2.0, "mobilenet_v2": 1.0, "resnet18": 1.0, "resnet50": 0.7, "vgg16": 0.25}


def listed():
    return [
        # the oracle-sized network: launches and host work are all there is
        dict(name="forward tiny fp32", how="forward", tasks="1*tiny/fp32/hp/1", parts="128", h=32, w=32, jobs=1),
        # one camera frame on one partition, each configured network in its configured type
        dict(name="forward mobilenet_v2 fp32", how="forward", tasks="1*mobilenet_v2/fp32/hp/1", parts="128", h=224, w=224, jobs=1),
        dict(name="forward resnet18 fp32", how="forward", tasks="1*resnet18/fp32/hp/1", parts="128", h=224, w=224, jobs=1),
        dict(name="forward resnet50 bf16", how="forward", tasks="1*resnet50/bf16/hp/1", parts="128", h=224, w=224, jobs=1),
        dict(name="forward vgg16 fp32", how="forward", tasks="1*vgg16/fp32/hp/1", parts="128", h=224, w=224, jobs=1),
        # a frame size that fits no tile, on a quarter of the chip
        dict(name="forward resnet50 fp32 odd", how="forward", tasks="1*resnet50/fp32/hp/1", parts="64", h=189, w=253, jobs=1),
        # callers that may not allocate
        dict(name="static resnet18 bf16", how="static", tasks="1*resnet18/bf16/hp/1", parts="192", h=224, w=224, jobs=1),
        # one job of a staged task through admission, dispatch and the stage boundaries
        dict(name="job resnet18 fp32 k=3", how="jobs", tasks="1*resnet18/fp32/hp/3", parts="96", h=224, w=224, jobs=1),
        # the configurations' task sets: all tasks released at one instant, and saturated
        dict(name="jobs mixed 8 tasks", how="jobs", h=224, w=224, jobs=1, parts="96,96,128,192",
             tasks="2*resnet18/fp32/hp/3+2*resnet50/fp32/lp/3+2*vgg16/fp32/lp/3+2*mobilenet_v2/fp32/lp/3"),
        dict(name="loop resnet18 fp32 x4", how="loop", h=224, w=224, jobs=16, parts="128,128,128",
             tasks="2*resnet18/fp32/hp/3+2*resnet18/fp32/lp/3"),
        dict(name="loop resnet50 bf16 x6", how="loop", h=224, w=224, jobs=20, parts="128,128,128,128",
             tasks="2*resnet50/bf16/hp/4+4*resnet50/bf16/lp/4"),
        dict(name="loop mixed 8 tasks", how="loop", h=224, w=224, jobs=16, parts="96,96,128,192",
             tasks="2*resnet18/fp32/hp/3+2*resnet50/fp32/lp/3+2*vgg16/fp32/lp/3+2*mobilenet_v2/fp32/lp/3"),
    ]


# ---- what a case says -----------------------------------------------------------------------------------------------------


def _tasks(case):
    """[(net, dtype, priority, stages)] in registration order."""
    out = []
    for part in case["tasks"].split("+"):
        n, spec = part.split("*")
        net, dtype, prio, k = spec.split("/")
        out += [(net, dtype, prio, int(k))] * int(n)
    return out


def _parts(case):
    return [int(v) for v in case["parts"].split(",")]


@functools.lru_cache(maxsize=None)
def _net(name, h, w):
    """(layers, input shape) of a network for h x w frames: the first fully connected layer takes what the pools leave."""
    layers, (c, _, _) = wl.build_net(name)
    layers = list(layers)
    shape, shapes = (c, h, w), []
    for i, L in enumerate(layers):
        c, y, x = shape if L.in_from < 0 else shapes[L.in_from]
        if L.op == OP_FC and L.c_in != c * y * x:
            layers[i] = dataclasses.replace(L, c_in=c * y * x)
        shapes.append(wl.nets.layer_shapes(layers[: i + 1], shape)[-1])
    return layers, shape


def _jobs(case, net):
    return max(1, round(case["jobs"] * JOB_WEIGHT[net])) if case["how"] == "loop" else 1


def _estimate_us(case):
    """A rough service time of one pass, for the AFETs and to keep drawn cases below the largest listed one."""
    total = 0.0
    for net, dtype, _, _ in _tasks(case):
        total += _jobs(case, net) * _job_us(net, dtype, case["h"], case["w"])
    return total


def _job_us(net, dtype, h, w):
    layers, shape = _net(net, h, w)
    return 5.0 * len(layers) + sum(wl.nets.net_macs(layers, shape)) / (25e6 if dtype == "fp32" else 200e6)


def draw(rng):
    """Any network in either type (the depthwise one in fp32, as configured), frames of 96 to 320 pixels a side (32 to 96 for
    the small one), partitions of 32 to 256 CUs, one task alone or a set of up to ten on two to four partitions."""
    most = max(_estimate_us(c) for c in listed())

    def side(net):
        lo, hi = (32, 96) if net == "tiny" else (160, 256) if net == "vgg16" else (96, 320)
        return rng.randint(lo, hi)

    def stages(net):
        return rng.randint(1, 3 if net == "tiny" else 5)

    while True:
        how = rng.choice(["forward", "forward", "static", "jobs", "loop", "loop"])
        if how in ("forward", "static"):
            net = rng.choice(["tiny", "mobilenet_v2", "resnet18", "resnet50", "vgg16"] if how == "forward" else ["tiny", "mobilenet_v2", "resnet18", "resnet50"])
            dtype = rng.choice(["fp32", "bf16"]) if net != "mobilenet_v2" else "fp32"
            h, w = (side(net), side(net)) if how == "forward" else (min(side(net), 224), min(side(net), 224))  # 16 MiB of tensors
            case = dict(how=how, tasks="1*%s/%s/hp/1" % (net, dtype), parts=str(8 * rng.randint(4, 32)), h=h, w=w, jobs=1)
        else:
            pool = rng.sample(["mobilenet_v2", "resnet18", "resnet50", "vgg16"], rng.randint(1, 3))
            dtype = rng.choice(["fp32", "bf16", "mixed"])
            tasks = []
            for i, net in enumerate(pool):
                for prio in ("hp", "lp"):
                    n = rng.randint(0 if tasks else 1, 2)
                    t = "fp32" if net == "mobilenet_v2" else dtype if dtype != "mixed" else rng.choice(["fp32", "bf16"])
                    if n:
                        tasks.append("%d*%s/%s/%s/%d" % (n, net, t, prio, stages(net)))
            net = "vgg16" if "vgg16" in pool else pool[0]
            parts = [8 * rng.randint(6, 24) for _ in range(rng.randint(2, 4))]
            if rng.random() < 0.5:
                parts = [parts[0]] * len(parts)
            jobs = 1 if how == "jobs" else max(2, round(2 * 12 ** rng.random()))
            case = dict(how=how, tasks="+".join(tasks), parts=",".join(map(str, parts)), h=side(net), w=side(net), jobs=jobs)
        if _estimate_us(case) <= most:
            return case


# ---- the program's library session ------------------------------------------------------------------------------------------

_open = {"key": None}


def _weights(net, h, w, seed):
    """He-normal weights with a folded batch normalisation where the architecture has one, drawn on the GPU."""
    layers, _ = _net(net, h, w)
    g = torch.Generator(device="cuda").manual_seed(WEIGHT_SEED + seed)
    out = []
    for L in layers:
        if L.op not in (OP_CONV, OP_FC):
            out.append((None, None))
            continue
        cg, kk = (L.c_in // L.groups, L.k) if L.op == OP_CONV else (L.c_in, 1)
        x = torch.randn((L.c_out, cg, kk, kk), generator=g, device="cuda") * (2.0 / (cg * kk * kk)) ** 0.5
        b = torch.randn(L.c_out, generator=g, device="cuda") * (0.1 if L.has_bn else 0.05)
        if L.has_bn:
            u = torch.rand((2, L.c_out), generator=g, device="cuda") + 0.5
            x = x * (u[0] * torch.rsqrt(u[1] + 1e-5)).view(-1, 1, 1, 1)
        out.append((x.cpu().numpy(), b.cpu().numpy()))
    return out


def _session(case):
    """The library set up for the case's tasks and partitions."""
    key = tuple(case[k] for k in ("tasks", "parts", "h", "w"))
    if _open["key"] == key:
        return
    if _open["key"] is not None:
        _open["key"] = None
        D.daris_shutdown()
    D.daris_init(0, WEIGHT_SEED, 0)
    parts = _parts(case)
    D.daris_set_plan_cus(parts[0] if len(set(parts)) == 1 else 128)
    for n in parts:
        D.daris_create_partition(n)
    made = {}
    for net, dtype, prio, k in _tasks(case):
        layers, shape = _net(net, case["h"], case["w"])
        if net not in made:
            made[net] = _weights(net, case["h"], case["w"], len(made))
        dnn, keep = D.make_dnn(layers, made[net], shape, dtype)
        t = D.daris_register_task(dnn, PERIOD_NS[prio], PERIOD_NS[prio], D.HP if prio == "hp" else D.LP)
        del keep
        D.daris_split_stages(t, k)
        for j in range(k):
            D.daris_set_afet(t, j, int(1e3 * _job_us(net, dtype, case["h"], case["w"]) / k) + 1)
    D.daris_commit()
    _open["key"] = key


def prepare(case, seed):
    """The library set up for the tasks, and frames (N(0,1); U(0,1) for the small network) with room for their logits."""
    _session(case)
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    frames, logits = [], []
    for net, _, _, _ in _tasks(case):
        layers, shape = _net(net, case["h"], case["w"])
        n = _jobs(case, net)
        make = torch.rand if net == "tiny" else torch.randn
        frames.append(make((n,) + shape, generator=g, device="cuda"))
        logits.append(torch.zeros((n, layers[-1].c_out), device="cuda"))
    return dict(case=case, frames=frames, logits=logits, n_jobs=[len(f) for f in frames])


def run(state):
    case, frames, logits = state["case"], state["frames"], state["logits"]
    _session(case)
    if case["how"] == "forward":
        D.daris_forward(0, frames[0], logits[0], 0)
    elif case["how"] == "static":
        D.daris_forward_static(0, frames[0], logits[0], 0)
    elif case["how"] == "jobs":
        for t in range(len(frames)):
            D.daris_release_job(t, frames[t], logits[t])
        D.daris_run_until_idle()
    else:
        for t in range(len(frames)):
            D.daris_task_set_io(t, frames[t], len(frames[t]), logits[t], len(logits[t]))
        D.daris_run_closed_loop(state["n_jobs"])
    return logits


def work(case):
    """Weights of every task once, every frame and every row of logits once; two operations per multiply-accumulate."""
    bytes_, flops = 0, 0
    for net, dtype, _, _ in _tasks(case):
        layers, shape = _net(net, case["h"], case["w"])
        n = _jobs(case, net)
        bytes_ += wl.nets.net_params(layers) * (2 if dtype == "bf16" else 4)
        bytes_ += 4 * n * (shape[0] * shape[1] * shape[2] + layers[-1].c_out)
        flops += 2 * n * sum(wl.nets.net_macs(layers, shape))
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """fp32: sums of up to 25088 terms through up to 53 layers in another order; bf16: roundings that tip, as deep."""
    if "/bf16/" in case["tasks"]:
        return {"rel": 2e-2, "max": 0.2}
    return {"rel": 2e-5, "max": 2e-4}
