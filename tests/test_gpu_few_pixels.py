"""GPU parity of fused 3x3 layers whose stages hold one channel block and few pixels: one 32-pixel block, exactly and just over one,
two and four of them, tiles at ragged edges, 16 to 40 channels, the 2x2 pool folded in, against the CPU oracle."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels,h,w,batch,th,tw", [
    ((16, 16), 9, 11, 2, 4, 4), ((32, 32), 17, 13, 1, 2, 14), ((32, 16, 24), 20, 23, 2, 4, 8), ((16, 32), 24, 24, 1, 8, 8),
    ((24, 16), 26, 31, 3, 8, 16), ((32, 32), 21, 18, 2, 9, 13), ((40, 32), 15, 15, 2, 6, 6), ((16, 16, 16, 16), 8, 8, 3, 0, 0)])
def test_few_pixels(channels, h, w, batch, th, tw):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("few pixels", channels, h, w, batch, th, tw)
    layers, cin = [], 16
    for c in channels:
        layers.append(nets.conv(cin, c, 3, 1, 1, "relu"))
        cin = c
    for pool in (False, True):
        ls = layers + ([nets.maxpool(cin, 2, 2, 0)] if pool else [])
        if pool and (h % 2 or w % 2 or th % 2 or tw % 2):
            continue
        net = dict(name="t", layers=ls, in_h=h, in_w=w, in_c=16, input_dist="uniform")
        x, ws, bs = gen.make_params(net, batch, 35)
        if th > 0:
            B.dlf_debug_force_config(th, tw, 2, 1, 0, 0)
        try:
            s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[len(ls) - 1], group_budget=[256])
        finally:
            B.dlf_debug_force_config(0)
        try:
            # the kernel and the register tile (32 x 64) that hold the half items, on the tile asked for
            cfg, g = B.dlf_plan_group_config(s.plan, 0), B.dlf_plan_groups(s.plan)[0]
            assert (cfg["kind"], cfg["variant"], cfg["nslices"]) == (0, 2, 1), cfg
            assert (g["tile_h"], g["tile_w"]) == (th, tw) if th > 0 else g["tile_h"] * g["tile_w"] <= 128, g
            got = s.run_numpy(x)
        finally:
            s.close()
        compare(got, o.run_net(net, x, ws, bs), "few pixels %s %dx%d" % (channels, th, tw))
