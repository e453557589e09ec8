"""dlf_plan_refine times every kernel form that a plan may hold: groups planned on a slower kernel (the others switched off
by the testing hooks) come out on the split-K and register-weight kernels, with the same results."""
import pytest
import torch

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


def _refined(layers, h, w, c, batch, last, off):
    """The layers as one group planned with `off` (a pair of binding calls: switch off, switch back), refined.
    -> (configuration before, after)."""
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    net = dict(name="refine", layers=layers, in_h=h, in_w=w, in_c=c, input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 37)
    off[0](B)
    try:
        s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[last], group_budget=[256])
    finally:
        off[1](B)
    before = B.dlf_plan_group_config(s.plan, 0)
    xt = torch.from_numpy(x).cuda()
    changed = s.refine(xt, top_k=4, reps=3)
    after = B.dlf_plan_group_config(s.plan, 0)
    y = s.run(xt)
    torch.cuda.synchronize()
    compare(y[:1].cpu().numpy(), o.run_net(net, x[:1], ws, bs), "after refinement")
    s.close()
    assert changed == 1
    return before, after


SMALL = (lambda B: B.dlf_debug_small_mode(2), lambda B: B.dlf_debug_small_mode(0))
PAIR = (lambda B: B.dlf_debug_small_pair_mode(2), lambda B: B.dlf_debug_small_pair_mode(0))
BLOCK = (lambda B: B.dlf_debug_block3x3_mode(1, 0, 8, 32), lambda B: B.dlf_debug_block3x3_mode(0))
GROUP = (lambda B: B.dlf_debug_block3x3_mode(2), lambda B: B.dlf_debug_block3x3_mode(0))


def test_split_k_forms():
    announce("refine split-K")
    # 11 us without the kernel, 7 with it
    before, after = _refined([nets.conv(512, 512, 3, 1, 1, "relu")], 7, 7, 512, 1, 0, SMALL)
    assert before["variant"] < 16 and after["kind"] == 10 and after["variant"] >= 16, (before, after)
    # 13.5 us without, 7.4 with
    before, after = _refined([nets.dwconv(512, 3, 2, "relu"), nets.conv(512, 1024, 1, 1, 0, "relu")], 14, 14, 512, 1, 1, PAIR)
    assert before["variant"] < 16 and after["kind"] == 6 and after["variant"] >= 16, (before, after)


def test_register_weight_forms():
    announce("refine register weights")
    # 97 us on the first block shape, 70 with the weights in registers
    before, after = _refined([nets.conv(64, 64, 3, 1, 1, "relu")], 224, 224, 64, 8, 0, BLOCK)
    assert (before["kind"], before["variant"]) == (4, 0) and after["kind"] == 4 and after["variant"] in range(16, 22), (before, after)
    # a first layer in front: 35 us on the fused-group kernel, 23 with it
    before, after = _refined([nets.conv(3, 64, 3, 1, 1, "relu"), nets.conv(64, 64, 3, 1, 1, "relu")], 160, 160, 3, 8, 1, GROUP)
    assert before["kind"] == 0 and (after["kind"], after["variant"]) == (4, 22), (before, after)
