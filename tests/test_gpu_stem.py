"""GPU parity of the kernel for a first 7x7 layer of stride 2 with the 3x3 max pool behind it, against the CPU oracle: maps smaller
than a tile, ragged in both directions, odd images and rows at odd addresses, every activation (a pool over negative values sees its
padding), more tiles than workgroups, an LDS limit."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,batch,act,budget,max_lds", [
    (1, 1, 1, "none", 256, 0), (2, 3, 3, "relu", 256, 0), (7, 9, 2, "none", 256, 0), (16, 33, 2, "relu6", 256, 0), (61, 47, 3, "none", 256, 0),
    (64, 64, 1, "relu", 256, 0), (113, 75, 5, "none", 8, 0), (224, 224, 2, "relu", 16, 0), (99, 101, 2, "none", 256, 12288)])
def test_stem(h, w, batch, act, budget, max_lds):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("stem", h, w, batch, act, budget, max_lds)
    net = dict(name="t", layers=[nets.conv(3, 64, 7, 2, 3, act), nets.maxpool(64, 3, 2, 1)], in_h=h, in_w=w, in_c=3, input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 31)
    s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[1], group_budget=[budget], max_lds_bytes=max_lds)
    try:
        cfg = B.dlf_plan_group_config(s.plan, 0)
        assert (cfg["kind"], cfg["variant"]) == (0, 16) and cfg["lds_bytes"] <= (max_lds or 163840), cfg
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "stem")
