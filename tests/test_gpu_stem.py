"""GPU parity of the kernel for a first 7x7 layer of stride 2 with the 3x3 max pool behind it, against the CPU oracle: one pooled pixel
and more, odd images and rows at odd addresses, every activation (a pool over negative values sees its padding), more tiles than
workgroups; narrow and large tiles, ragged in both directions (no plan has a tile larger than the map), an LDS limit that asks for
a smaller tile."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,batch,act,budget,max_lds", [
    (1, 1, 1, "none", 256, 0), (2, 3, 3, "relu", 256, 0), (7, 9, 2, "none", 256, 0), (16, 33, 2, "relu6", 256, 0), (61, 47, 3, "none", 256, 0),
    (64, 64, 1, "relu", 256, 0), (113, 75, 5, "none", 8, 0), (224, 224, 2, "relu", 16, 0), (99, 101, 2, "none", 256, 12288)])
def test_stem(h, w, batch, act, budget, max_lds):
    _run(h, w, batch, act, budget, max_lds)


@pytest.mark.parametrize("h,w,batch,act,budget,max_lds,tile", [
    (35, 78, 2, "none", 32, 16384, (2, 7)), (52, 88, 1, "none", 8, 0, (3, 8)), (119, 36, 1, "relu", 4, 0, (8, 5)), (74, 149, 1, "none", 1, 0, (7, 8)),
    (146, 49, 2, "relu6", 1, 0, (8, 7)), (113, 75, 5, "none", 8, 12288, (2, 5))])
def test_ragged_tiles(h, w, batch, act, budget, max_lds, tile):
    info, (oh, ow) = _run(h, w, batch, act, budget, max_lds)
    assert (info["tile_h"], info["tile_w"]) == tile and oh % tile[0] and ow % tile[1], (info, oh, ow)


def test_tile_shrinks_under_an_lds_limit():
    free = _run(113, 75, 1, "none", 8, 0)[0]
    held = _run(113, 75, 1, "none", 8, 9600)[0]
    assert held["lds_bytes"] <= 9600 < free["lds_bytes"] and held["tile_h"] * held["tile_w"] < free["tile_h"] * free["tile_w"], (free, held)


def _run(h, w, batch, act, budget, max_lds):
    """-> (the group as planned, the pooled map's size)"""
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
        cfg.update(B.dlf_plan_groups(s.plan)[0])
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "stem")
    return cfg, got.shape[1:3]
