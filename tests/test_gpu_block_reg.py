"""GPU parity of the 3x3 block kernel with its weights in registers, forced through the testing hook,
against the CPU oracles: every shape (fp16 and int8), tiles that fill and that underfill a wave's pixel
blocks, ragged maps and channel groups, one and several blocks of K, residual operand, folded pool,
several items per workgroup."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu

HOOK = 8          # first shape number of the testing hook
# (shape, tile, cin, cout, h, w, batch, budget)
CASES = [(0, 7, 28, 64, 128, 28, 28, 1, 256), (0, 8, 28, 192, 200, 18, 62, 2, 8), (0, 16, 14, 128, 40, 16, 15, 3, 256),
         (0, 7, 32, 64, 136, 9, 70, 2, 16), (0, 2, 4, 256, 64, 3, 5, 2, 8),
         (1, 8, 16, 128, 128, 26, 34, 2, 8), (1, 4, 28, 64, 72, 11, 57, 1, 256), (1, 7, 7, 320, 256, 7, 7, 2, 256),
         (2, 14, 32, 64, 64, 30, 66, 2, 8), (2, 16, 28, 128, 40, 16, 29, 1, 256), (3, 8, 32, 64, 104, 20, 40, 2, 256),
         (3, 16, 16, 192, 32, 16, 16, 3, 8), (4, 8, 28, 32, 128, 14, 30, 2, 256), (4, 7, 32, 96, 168, 20, 33, 1, 8),
         (5, 14, 32, 32, 64, 30, 36, 2, 8), (5, 16, 28, 160, 48, 31, 30, 1, 256), (5, 2, 2, 64, 64, 1, 1, 2, 8)]


def _mk(layers, h, w, c):
    return dict(name="t", layers=layers, in_h=h, in_w=w, in_c=c, input_dist="normal")


def _fp16(layers, lasts, h, w, cin, batch, shape, th, tw, budget):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    net = _mk(layers, h, w, cin)
    x, ws, bs = gen.make_params(net, batch, 31)
    B.dlf_debug_block3x3_mode(1, HOOK + shape, th, tw)
    try:
        s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=list(lasts), group_budget=[budget] * len(lasts))
    finally:
        B.dlf_debug_block3x3_mode(0)
    try:
        cfg = B.dlf_plan_group_config(s.plan, len(lasts) - 1)
        assert cfg["kind"] == 4 and cfg["variant"] == 16 + shape, cfg
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "shape %d tile %dx%d" % (shape, th, tw))


@pytest.mark.parametrize("shape,th,tw,cin,cout,h,w,batch,budget", CASES)
def test_layer_pool_and_residual(shape, th, tw, cin, cout, h, w, batch, budget):
    announce("block reg", shape, th, tw, cin, cout, h, w, batch, budget)
    args = (h, w, cin, batch, shape, th, tw, budget)
    _fp16([nets.conv(cin, cout, 3, 1, 1, "relu")], [0], *args)
    # the residual operand: the layer's own output shape, made by a 1x1 layer in front
    _fp16([nets.conv(cin, cin, 1, 1, 0, "relu"), nets.conv(cin, cout, 1, 1, 0, "none", input_from=0),
           nets.conv(cin, cout, 3, 1, 1, "relu6", input_from=0, residual_from=1)], [0, 1, 2], *args)
    if th % 2 == 0 and tw % 2 == 0 and tw >= 4 and h % 2 == 0 and w % 2 == 0:       # (odd maps keep the pool apart)
        _fp16([nets.conv(cin, cout, 3, 1, 1, "none"), nets.maxpool(cout, 2, 2, 0)], [1], *args)


@pytest.mark.parametrize("cin,cout,h,w,batch,th,tw,budget", [
    (3, 64, 30, 66, 2, 14, 32, 8), (3, 40, 16, 28, 1, 16, 28, 256), (1, 128, 13, 9, 3, 4, 14, 8), (2, 64, 1, 1, 2, 2, 4, 8),
    (3, 96, 31, 45, 1, 8, 16, 16)])
def test_first_layer_in_front(cin, cout, h, w, batch, th, tw, budget):
    announce("block reg stem", cin, cout, h, w, batch, th, tw)
    layers = [nets.conv(cin, 64, 3, 1, 1, "relu6" if cin == 2 else "relu"), nets.conv(64, cout, 3, 1, 1, "relu")]
    _fp16(layers, [1], h, w, cin, batch, 6, th, tw, budget)
    if h % 2 == 0 and w % 2 == 0:
        _fp16(layers + [nets.maxpool(cout, 2, 2, 0)], [2], h, w, cin, batch, 6, th, tw, budget)


@pytest.mark.parametrize("shape,th,tw,cin,cout,h,w,batch,budget", CASES)
def test_int8_layer(shape, th, tw, cin, cout, h, w, batch, budget):
    from paper_2011_05630_amd import binding as B
    from test_gpu_i8 import _check
    cout = (cout + 15) // 16 * 16
    x, wt, sc, b = gen.make_i8_layer(batch, h, w, 2 * cin, cout, 3, seed=90 + shape)
    for pool in (False, True):
        if pool and (th % 2 or tw % 2 or tw < 4 or h < 2 or w < 2):
            continue
        B.dlf_debug_block3x3_mode(0, HOOK + shape, th, tw)
        try:
            info = _check(("reg", shape, th, tw), x, wt, sc, b, not pool, budget=budget, pool=pool)
        finally:
            B.dlf_debug_block3x3_mode(0)
        assert (info["shape"], info["th"], info["tw"]) == (HOOK + shape, th, tw), info
