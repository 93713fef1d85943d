"""Whatever wrote the caller's input last -- a copy from the host, a copy on the device, a kernel -- the next job sees it, in
the same buffer again and again and through buffers that change from call to call; and every job's logits reach its own."""
import numpy as np
import pytest
import torch

import paper_2504_08795_amd as D
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("net,dtype,hw", [("tiny", "fp32", None), ("mobilenet_v2", "fp32", 64), ("resnet18", "bf16", 64)])
def test_rewritten_inputs_and_changing_buffers(net, dtype, hw):
    layers, shp = wl.build_net(net)
    shp = shp if hw is None else (shp[0], hw, hw)
    weights = wl.make_weights(layers, 3)
    n_out, rounds, kinds = layers[-1].c_out, 120, 6
    frames = np.random.default_rng(8).normal(0, 1, (kinds,) + shp).astype(np.float32)
    on_device = torch.from_numpy(frames).cuda()
    D.daris_init(0, 0, 0)
    try:
        parts = [D.daris_create_partition(128), D.daris_create_partition(64)]
        dnn, keep = D.make_dnn(layers, weights, shp, dtype)
        t = D.daris_register_task(dnn, 10**8, 10**8, D.HP)
        D.daris_split_stages(t, 2)
        D.daris_commit()
        want = torch.empty((kinds, n_out), device="cuda")
        for i in range(kinds):
            D.daris_forward(t, on_device[i], want[i], parts[0])
        assert len({tuple(r) for r in want.cpu().numpy().round(6).tolist()}) == kinds      # the frames can be told apart
        x = torch.zeros(shp, device="cuda")
        outs = torch.zeros((7, n_out), device="cuda")
        run = [lambda a, y, r: D.daris_forward(t, a, y, parts[r % 2]), lambda a, y, r: D.daris_forward_static(t, a, y, parts[r % 2]),
               lambda a, y, r: (D.daris_release_job(t, a, y), D.daris_run_until_idle())]
        for r in range(rounds):
            k = (r * 5 + r // 7) % kinds
            how = r % 4
            if how == 0:
                x.copy_(torch.from_numpy(frames[k]))          # from the host
            elif how == 1:
                x.copy_(on_device[k])                          # on the device
            elif how == 2:
                torch.mul(on_device[k], 1.0, out=x)            # by a kernel
            src = on_device[k] if how == 3 else x              # another buffer
            torch.cuda.synchronize()
            y = outs[r % 7]
            run[r % 3](src, y, r)
            assert torch.equal(y, want[k]), (r, k, how)
    finally:
        D.daris_shutdown()


def test_inputs_in_host_memory():
    """An input that does not lie in the GPU's own memory (pinned host memory here; a peer's is alike) is acquired at system
    scope: what the host wrote last is what the next job reads, through every entry point, in one buffer again and again."""
    layers, shp = wl.build_net("tiny")
    weights = wl.make_weights(layers, 3)
    n_out, kinds = layers[-1].c_out, 5
    frames = np.random.default_rng(9).normal(0, 1, (kinds,) + shp).astype(np.float32)
    on_device = torch.from_numpy(frames).cuda()
    D.daris_init(0, 0, 0)
    try:
        part = D.daris_create_partition(128)
        dnn, keep = D.make_dnn(layers, weights, shp, "fp32")
        t = D.daris_register_task(dnn, 10**8, 10**8, D.HP)
        D.daris_commit()
        want = torch.empty((kinds, n_out), device="cuda")
        for i in range(kinds):
            D.daris_forward(t, on_device[i], want[i], part)
        x = torch.zeros((2,) + shp, pin_memory=True)
        y = torch.zeros((2, n_out), device="cuda")
        for r in range(60):
            a, b = r % kinds, (3 * r + 1) % kinds
            x[0], x[1] = torch.from_numpy(frames[a]), torch.from_numpy(frames[b])
            y.zero_()
            torch.cuda.synchronize()
            if r % 4 == 3:
                D.daris_task_set_io(t, x, 2, y, 2)
                first = D.daris_get_stats(t)["released"] % 2
                D.daris_run_closed_loop([2])
                assert torch.equal(y[first], want[(a, b)[first]])
            else:
                for i in range(2):
                    if r % 4 == 2:
                        D.daris_release_job(t, x[i], y[i])
                        D.daris_run_until_idle()
                    else:
                        (D.daris_forward, D.daris_forward_static)[r % 4](t, x[i], y[i], part)
            assert torch.equal(y[0], want[a]) and torch.equal(y[1], want[b]), r
    finally:
        D.daris_shutdown()
