"""dlf_run_noalloc on plans whose workspace is larger than the static one: the same layers in groups that fit it, as
long as there is such a grouping."""
import pytest
import torch

from synth import nets, gen
from gpu_util import compare, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,hw,batch", [("vgg16", 96, 16), ("mobilenet_v1", 128, 32), ("resnet50", 96, 12), ("resnet50", 96, 13)])
def test_larger_plans_run(name, hw, batch):
    from paper_2011_05630_amd import binding as B
    from paper_2011_05630_amd.runner import Session
    announce("noalloc", name, hw, batch)
    net = getattr(nets, name)(hw)
    x, ws, bs = gen.make_params(net, batch, 41)
    s = Session(net, batch, ws, bs)
    try:
        assert B.dlf_static_workspace_bytes() < B.dlf_plan_workspace_bytes(s.plan) < 2 * B.dlf_static_workspace_bytes()
        xt = torch.from_numpy(x).cuda()
        want = s.run(xt).clone()
        got = torch.full(s.out_shape, float("nan"), dtype=torch.float16, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        for _ in range(2):
            got.fill_(float("nan"))
            B.dlf_run_noalloc(s.plan, xt.data_ptr(), got.data_ptr(), stream)
            torch.cuda.synchronize()
            # (other groups round in other places, as between any two plans)
            compare(got.cpu().numpy(), want.cpu().numpy(), "%s %d batch %d" % (name, hw, batch))
        again = s.run(xt)
        torch.cuda.synchronize()
        assert torch.equal(again, want)
    finally:
        s.close()
