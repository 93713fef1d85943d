"""Layers that are computed in the launch of another one, against the oracle and, bit for bit, against launches of their own (a stage cut between the
two layers parts them)."""
import numpy as np
import pytest

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


# c_in, h, w, c_out, k, stride, pad: the edges of a workgroup's 3 x 7 pooled pixels, outputs of odd and even sizes, and frames larger than one round
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
    # Which tiles the NaN and the infinity have walked again in plain fp32 depends on the tiles (both roundings within 147 * 2^-24 of the sum's terms)
    np.testing.assert_allclose(*outs[1], rtol=1e-5, atol=1e-4 if dtype == "fp32" else 0)
    e_max, e_l2 = rel_err(outs[0][0], oracle_logits(layers, weights, x, dtype))
    assert e_max <= TOL[dtype] and e_l2 <= TOL[dtype], (e_max, e_l2)
