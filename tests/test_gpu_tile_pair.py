"""The depthwise + 1x1 tile kernel with numbers of tiles that are no multiple of the eight XCDs: parity with the CPU oracle, and every
tile in the launch's one round of workgroups."""
import pytest
import torch

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


def _session(c, cout, hw, batch):
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    net = dict(name="t", layers=[nets.dwconv(c, 3, 1, "relu6"), nets.conv(c, cout, 1, 1, 0, "relu")], in_h=hw, in_w=hw, in_c=c,
               input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 53)
    B.dlf_debug_depthwise_mode(1)
    B.dlf_debug_depthwise_tile(4, 1)                     # rows of 4 * 512 / (2 * c) pixels, one to a wave
    try:
        s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[1], group_budget=[256])
    finally:
        B.dlf_debug_depthwise_tile(0, 0)
        B.dlf_debug_depthwise_mode(0)
    assert B.dlf_plan_group_config(s.plan, 0)["kind"] == 7
    return net, x, ws, bs, s


@pytest.mark.parametrize("batch", [1, 2, 3, 5, 6, 7, 8])
def test_tiles_of_any_number(batch):
    from oracle import oracle as o
    announce("tile pair", batch)
    net, x, ws, bs, s = _session(128, 72, 9, batch)      # nine tiles of 1 x 16 pixels per image
    try:
        assert (s.groups[0]["tile_h"], s.groups[0]["tile_w"]) == (1, 16), s.groups
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "%d tiles" % (9 * batch))


def test_no_workgroup_has_a_second_tile():
    """84 tiles take what 112 do (256 -> 256 channels: 6.8 us, 11.3 while four of 84 workgroups had two)."""
    announce("tile pair, one round")
    us = {}
    for batch in (3, 4):
        _, x, _, _, s = _session(256, 256, 14, batch)    # 28 tiles of 1 x 8 pixels per image
        try:
            assert (s.groups[0]["tile_h"], s.groups[0]["tile_w"]) == (1, 8), s.groups
            xt = torch.from_numpy(x).cuda()
            y = s.run(xt)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            us[batch] = 1e9
            for _ in range(6):
                a.record()
                for _ in range(100):
                    s.run(xt, y)
                b.record()
                torch.cuda.synchronize()
                us[batch] = min(us[batch], a.elapsed_time(b) * 10)
        finally:
            s.close()
    assert us[3] <= 1.25 * us[4], us
