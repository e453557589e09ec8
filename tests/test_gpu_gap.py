"""GPU parity of global average pooling against the CPU oracle: whole vectors and odd channel counts, the last group of 256 channels
ragged, one pixel, a trip's worth of pixels per thread and one more, an LDS limit that holds no partial sums,
a tensor that is not on a 16-byte line."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_lds", [0, 4096])
@pytest.mark.parametrize("c,h,w,batch", [(8, 1, 1, 1), (264, 7, 7, 3), (2048, 7, 8, 2), (512, 3, 19, 5), (1000, 12, 11, 1), (20, 7, 7, 2), (13, 9, 5, 3)])
def test_global_average_pool(c, h, w, batch, max_lds):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("gap", c, h, w, batch, max_lds)
    net = dict(name="t", layers=[nets.gavgpool(c)], in_h=h, in_w=w, in_c=c, input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 33)
    s = Session(net, batch, ws, bs, mode=B.TUNER_MANUAL, group_last=[0], group_budget=[256], max_lds_bytes=max_lds)
    try:
        assert B.dlf_plan_group_config(s.plan, 0)["lds_bytes"] == (8192 if max_lds == 0 and c % 8 == 0 else 0)
        got = s.run_numpy(x)
        assert got.shape == (batch, 1, 1, c)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "gap %d" % c)


def test_tensor_off_the_vectors_line():
    import numpy as np
    import torch
    from oracle import oracle as o
    from paper_2011_05630_amd.runner import Session
    net = dict(name="t", layers=[nets.gavgpool(264)], in_h=7, in_w=5, in_c=264, input_dist="normal")
    x, ws, bs = gen.make_params(net, 3, 33)
    s = Session(net, 3, ws, bs)
    room = torch.zeros(x.size + 8, dtype=torch.float16, device="cuda")
    try:
        for off in (1, 4, 8):
            announce("gap, offset", off)
            xd = room[off:off + x.size].view(x.shape)
            xd.copy_(torch.from_numpy(np.ascontiguousarray(x, dtype=np.float16)))
            compare(s.run(xd).cpu().numpy(), o.run_net(net, x, ws, bs), "gap, offset %d" % off)
    finally:
        s.close()
