"""GPU parity of the kernel for a first 3x3 layer of stride 2 with the depthwise layer and the 1x1 layer behind it, against the CPU
oracle: maps smaller than a tile, of whole tiles and ragged in both directions, odd images, ragged channel blocks, every activation."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cout,h,w,batch,acts", [
    (64, 1, 1, 1, ("relu6", "relu6", "relu6")), (8, 2, 5, 3, ("none", "relu", "none")), (32, 16, 32, 2, ("relu", "none", "relu6")),
    (40, 17, 33, 1, ("relu6", "relu6", "none")), (64, 31, 67, 2, ("relu", "relu", "relu")), (96, 45, 30, 1, ("relu6", "relu", "relu")),
    (128, 15, 34, 5, ("none", "none", "none")), (64, 112, 112, 40, ("relu6", "relu6", "relu6"))])
def test_first_pair(cout, h, w, batch, acts):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("first pair", cout, h, w, batch, acts)
    net = dict(name="t", layers=[nets.conv(3, 32, 3, 2, 1, acts[0]), nets.dwconv(32, 3, 1, acts[1]), nets.conv(32, cout, 1, 1, 0, acts[2])],
               in_h=h, in_w=w, in_c=3, input_dist="uniform")
    x, ws, bs = gen.make_params(net, batch, 29)
    B.dlf_debug_depthwise_mode(5)
    try:
        s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[2], group_budget=[256])
    finally:
        B.dlf_debug_depthwise_mode(0)
    try:
        cfg = B.dlf_plan_group_config(s.plan, 0)
        assert (cfg["kind"], cfg["variant"]) == (7, 16 + (4 if cout > 64 else (cout + 31) // 32)), cfg
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "first pair")
