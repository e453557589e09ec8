"""GPU parity of the split-K kernel for a depthwise 3x3 layer with the 1x1 layer behind it, forced through its
testing hook, against the CPU oracle: every item shape and number of waves, both strides, maps of one pixel and
odd maps, ragged pixel and channel groups, one K step, steps that do not divide among the waves, and more than 64 KiB of LDS."""
import pytest
import torch

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [0, 1])
@pytest.mark.parametrize("c,cout,stride,h,w,batch", [
    (32, 8, 1, 1, 1, 1), (32, 64, 2, 15, 8, 3), (96, 40, 1, 9, 13, 2), (160, 136, 2, 6, 7, 2), (512, 512, 1, 14, 14, 1),
    (512, 72, 2, 5, 5, 3), (1024, 200, 1, 7, 7, 1), (64, 128, 2, 33, 21, 2),
    # 33, 36 and 43 steps: eight waves with shares of 5 (the last idle), 5 and 6
    (1056, 72, 1, 5, 4, 2), (1152, 320, 1, 7, 7, 1), (1376, 40, 2, 9, 6, 2)])
def test_pair(shape, c, cout, stride, h, w, batch):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("small pair", shape, c, cout, stride, h, w, batch)
    acts = ("relu6", "none") if cout == 40 else ("relu", "relu6")
    net = dict(name="t", layers=[nets.dwconv(c, 3, stride, acts[0]), nets.conv(c, cout, 1, 1, 0, acts[1])], in_h=h, in_w=w, in_c=c,
               input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 23)
    ref = o.run_net(net, x, ws, bs)
    for waves in (0, 1, 2, 4, 8):
        B.dlf_debug_small_pair_mode(1, shape, waves)
        try:
            s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[1], group_budget=[256])
        finally:
            B.dlf_debug_small_pair_mode(0)
        try:
            cfg = B.dlf_plan_group_config(s.plan, 0)
            assert (cfg["kind"], cfg["variant"]) == (6, 16 + shape), cfg
            got = s.run_numpy(x)
        finally:
            s.close()
        compare(got, ref, "pair shape %d waves %d" % (shape, waves))


@pytest.mark.parametrize("c,cout", [(1056, 1056), (1152, 320), (1280, 1280), (1376, 320)])
def test_pairs_above_1024_channels_as_planned(c, cout):
    """The library's own plan of such a pair runs, and so do all the forms that dlf_plan_refine times."""
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("planned pair", c, cout)
    net = dict(name="t", layers=[nets.dwconv(c, 3, 1, "relu6"), nets.conv(c, cout, 1, 1, 0, "none")], in_h=7, in_w=7, in_c=c,
               input_dist="normal")
    x, ws, bs = gen.make_params(net, 1, 41)
    ref = o.run_net(net, x, ws, bs)
    for kw in ({}, dict(mode=B.TUNER_MANUAL, group_last=[1], group_budget=[256])):
        s = Session(net, 1, ws, bs, **kw)
        try:
            compare(s.run_numpy(x), ref, "planned")
            s.refine(torch.from_numpy(x).cuda(), top_k=3, reps=2)
            compare(s.run_numpy(x), ref, "refined")
        finally:
            s.close()
