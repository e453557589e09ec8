"""GPU parity of the fully connected kernel in one launch, against the CPU oracle: K shorter than one wave's turn, odd numbers of
32-channel chunks, shares just above the ring's length; ragged channel groups; one image to more than two groups of 32."""
import pytest

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 32, 33, 70])
@pytest.mark.parametrize("k,cout", [(8, 1), (24, 17), (72, 33), (512, 130), (2056, 16), (4096, 47), (4136, 1000), (8200, 129)])
def test_fc(k, cout, batch):
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("fc", k, cout, batch)
    act = ("none", "relu", "relu6")[(k + batch) % 3]
    net = dict(name="t", layers=[nets.fc(k, cout, act)], in_h=1, in_w=1, in_c=k, input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 31)
    B.dlf_debug_force_config(1, 1, 0, 1, 0, 0, 32)       # K not split over workgroups
    try:
        s = Session(net, batch, ws, bs)
    finally:
        B.dlf_debug_force_config(0, 0, 0, 1, 0, 0, 32)
    try:
        cfg = B.dlf_plan_group_config(s.plan, 0)
        assert (cfg["kind"], cfg["variant"]) == (1, 2 if batch > 16 else 1 if (k + 31) // 32 * 2 > 128 else 0), cfg
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "fc")


@pytest.mark.parametrize("limit,few,many", [(131071, 0, 9), (65536, 0, 9), (36863, 4, 10), (16384, 5, 5), (8192, 6, 6), (4096, 7, 7), (2048, 8, 8)])
@pytest.mark.parametrize("k,cout,batch", [(8, 1, 1), (72, 33, 17), (520, 130, 16), (2056, 47, 33), (8200, 129, 5)])
def test_fc_under_an_lds_limit(k, cout, batch, limit, few, many):
    """The forms of a smaller LDS limit: shorter rings, fewer waves; shares longer than the ring and waves without one."""
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("fc limit", k, cout, batch, limit)
    net = dict(name="t", layers=[nets.fc(k, cout, "relu")], in_h=1, in_w=1, in_c=k, input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 43)
    B.dlf_debug_force_config(1, 1, 0, 1, 0, 0, 32)       # K not split over workgroups
    try:
        s = Session(net, batch, ws, bs, max_lds_bytes=limit)
    finally:
        B.dlf_debug_force_config(0, 0, 0, 1, 0, 0, 32)
    try:
        cfg = B.dlf_plan_group_config(s.plan, 0)
        assert (cfg["kind"], cfg["variant"]) == (1, many if batch > 16 else few) and cfg["lds_bytes"] <= limit, cfg
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "fc limit %d" % limit)


@pytest.mark.parametrize("ksplit", [2, 4, 8])
@pytest.mark.parametrize("k,cout,batch", [(2056, 72, 17), (4136, 33, 40), (8200, 129, 5)])
def test_split_k_on_ragged_k(k, cout, batch, ksplit):
    """K split over workgroups where K is no multiple of 32: the last step is half beyond K (read from a stand-in address and replaced
    by zeros), slices and waves' shares are uneven or empty; an odd number of channel blocks, two blocks of images."""
    from oracle import oracle as o
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("fc split K", k, cout, batch, ksplit)
    net = dict(name="t", layers=[nets.fc(k, cout, "none")], in_h=1, in_w=1, in_c=k, input_dist="normal")
    x, ws, bs = gen.make_params(net, batch, 47)
    B.dlf_debug_force_config(1, 1, 0, ksplit, 0, 0, 32)
    try:
        s = Session(net, batch, ws, bs)
    finally:
        B.dlf_debug_force_config(0, 0, 0, 1, 0, 0, 32)
    try:
        cfg = B.dlf_plan_group_config(s.plan, 0)
        assert (cfg["kind"], cfg["variant"]) == (1, 3), cfg
        got = s.run_numpy(x)
    finally:
        s.close()
    compare(got, o.run_net(net, x, ws, bs), "fc K in %d slices" % ksplit)
