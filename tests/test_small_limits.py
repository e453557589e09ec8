"""Limits of the split-K kernels for outputs of few pixels (a single convolution, and a depthwise layer with the 1x1
layer behind it), as plans show them on the CPU."""
import random

import numpy as np
import pytest

from synth import nets
from paper_2011_05630_amd import binding as B

# items of a shape, pixels x channels (shape = variant - 16)
CONV_ITEM = {0: (16, 16), 1: (16, 32), 2: (16, 64), 3: (32, 64)}
PAIR_ITEM = {0: (16, 32), 1: (16, 64)}


def _plan(layers, h, w, batch, budget=256, max_lds=0):
    """-> (group configuration, pixels) of the layers as one group."""
    n = B.dlf_net_create(layers, h, w, layers[0]["cin"])
    try:
        p = B.dlf_plan(n, batch, mode=B.TUNER_MANUAL, group_last=[len(layers) - 1], group_budget=[budget], max_lds_bytes=max_lds)
        cfg = B.dlf_plan_group_config(p, 0)
        B.dlf_plan_destroy(p)
        oh, ow = B.dlf_net_layer_info(n, len(layers) - 1)[:2]
    finally:
        B.dlf_net_destroy(n)
    return cfg, batch * oh * ow


def _items_divide_exactly(m, cout, item):
    n_pg, n_cg = -(-m // item[0]), -(-cout // item[1])
    if n_cg == 1:
        return True
    items = np.arange(n_pg * n_cg, dtype=np.uint64)
    magic = np.uint64(0xFFFFFFFF // n_cg + 1)                       # the kernels' div_by
    return bool(np.all((items * magic) >> np.uint64(32) == items // np.uint64(n_cg)))


def test_items_of_many_channels_are_divided_exactly():
    """Layers of up to 2^20 output channels: a kernel that finds its pixel group by a 32-bit product is planned only
    where that product is exact for every item.  (A budget far above the chip's: the number of workgroups is no limit.)"""
    budget = 1 << 20
    rng = random.Random(7)
    cases = [(32, 905432, 44, 20), (64, 561244, 64, 16), (32, 1 << 20, 40, 24)]
    cases += [(32 * rng.randint(1, 4), 4 * rng.randint(1 << 16, 1 << 18), rng.randint(2, 48), rng.randint(2, 48)) for _ in range(20)]
    seen = 0
    for t, (cin, cout, h, w) in enumerate(cases):
        shape = 3 if t < 3 else t % 4
        B.dlf_debug_small_mode(1, shape, 0)
        try:
            cfg, m = _plan([nets.conv(cin, cout, 1, 1, 0, "relu")], h, w, 1, budget)
        except B.DlfError:
            continue
        finally:
            B.dlf_debug_small_mode(0)
        if cfg["kind"] == 10 and cfg["variant"] >= 16:
            seen += 1
            assert _items_divide_exactly(m, cout, CONV_ITEM[shape]), (cin, cout, h, w, cfg)
    for shape in (0, 1):
        B.dlf_debug_small_pair_mode(1, shape, 0)
        try:
            for c, cout, h, w in ((32, 905432, 44, 20), (32, 1 << 20, 40, 25), (64, 40000, 9, 9)):
                cfg, m = _plan([nets.dwconv(c, 3, 1, "relu"), nets.conv(c, cout, 1, 1, 0, "relu")], h, w, 1, budget)
                if cfg["kind"] == 6 and cfg["variant"] >= 16:
                    seen += 1
                    assert _items_divide_exactly(m, cout, PAIR_ITEM[shape]), (c, cout, h, w, cfg)
        finally:
            B.dlf_debug_small_pair_mode(0)
    assert seen >= 4, seen


def _split_k_groups(net, batch, **plan):
    """-> [(workgroups, budget, item shape, group configuration)] of the plan's groups on the split-K kernels."""
    h = B.dlf_net_create(net["layers"], net["in_h"], net["in_w"], net["in_c"])
    p = B.dlf_plan(h, batch, **plan)
    out = []
    for g, info in enumerate(B.dlf_plan_groups(p)):
        cfg = B.dlf_plan_group_config(p, g)
        if cfg["variant"] < 16 or cfg["kind"] not in (6, 8, 10):
            continue
        item = (PAIR_ITEM if cfg["kind"] == 6 else CONV_ITEM)[cfg["variant"] - 16]
        last = info["last"]
        if net["layers"][last]["op"] == "maxpool":
            last -= 1                                              # items count the convolution's pixels
        oh, ow, cout = B.dlf_net_layer_info(h, last)[:3]
        out.append((-(-batch * oh * ow // item[0]) * -(-cout // item[1]), info["budget"], item, cfg))
    B.dlf_plan_destroy(p)
    B.dlf_net_destroy(h)
    return out


def test_launches_keep_to_their_budget():
    """A workgroup per item, so items <= budget x occupancy (two workgroups per CU)."""
    seen = 0
    for net in (nets.resnet50(128), nets.resnet18(), nets.mobilenet_v1(), nets.vgg16(64)):
        for batch in (1, 2, 4):
            for mode, kw in ((B.TUNER_LAYERWISE, dict(fixed_budget=32)), (B.TUNER_LAYERWISE, dict(fixed_budget=64)),
                             (B.TUNER_LAYERWISE, dict(fixed_budget=128)), (B.TUNER_GREEDY, dict(fixed_budget=32)),
                             (B.TUNER_DP, {}), (B.TUNER_DP, dict(budgets=[16]))):
                for wgs, budget, item, cfg in _split_k_groups(net, batch, mode=mode, **kw):
                    seen += 1
                    assert wgs <= 2 * budget, (net["name"], batch, mode, kw, wgs, budget, cfg)
    assert seen > 100, seen


def test_launches_keep_to_the_lds_limit():
    """max_lds_bytes is the limit of every group on the split-K kernels."""
    seen = 0
    for net in (nets.resnet50(), nets.mobilenet_v1(), nets.identical_chain(64, 32, 3)):
        for limit in (4096, 16384, 65536):
            for batch in (1, 4):
                try:
                    groups = _split_k_groups(net, batch, max_lds_bytes=limit)
                except B.DlfError:
                    continue                                       # (some layer fits no kernel)
                for _, _, _, cfg in groups:
                    seen += 1
                    assert 0 < cfg["lds_bytes"] <= limit, (net["name"], batch, limit, cfg)
    # one layer, every item shape asked for: 32 x 64 outputs need 32 KiB with four waves
    for limit in (2048, 4096, 16384, 32768):
        for shape in range(4):
            B.dlf_debug_small_mode(1, shape, 0)
            try:
                cfg, _ = _plan([nets.conv(64, 64, 3, 1, 1, "relu")], 32, 32, 1, max_lds=limit)
            except B.DlfError:
                continue
            finally:
                B.dlf_debug_small_mode(0)
            seen += 1
            assert cfg["lds_bytes"] <= limit, (limit, shape, cfg)
    assert seen > 60, seen


@pytest.mark.parametrize("k,cout", [(24, 17), (2048, 1000), (25088, 4096), (25088, 96)])
@pytest.mark.parametrize("batch", [1, 16, 17, 70])
def test_fully_connected_layers_keep_to_the_lds_limit(k, cout, batch):
    """max_lds_bytes is the limit of fully connected layers too: shorter rings, then fewer waves, K split over workgroups only where its
    36 KiB fit; below 2 KiB there is none."""
    layers = [nets.fc(k, cout, "relu")]
    for limit in (0, 163840, 131071, 65536, 36864, 36863, 32768, 16384, 8192, 4096, 2048):
        cfg, _ = _plan(layers, 1, 1, batch, max_lds=limit)
        assert cfg["kind"] == 1 and 0 < cfg["lds_bytes"] <= (limit or 163840), (limit, cfg)
        want = {0: 65536, 1: 131072, 2: 131072, 3: 36864, 4: 32768, 5: 16384, 6: 8192, 7: 4096, 8: 2048,
                9: 65536, 10: 32768}[cfg["variant"]]
        assert cfg["lds_bytes"] == want and (limit > 0 or cfg["variant"] <= 3), (limit, cfg)
    n = B.dlf_net_create(layers, 1, 1, k)
    assert B.dlf_group_cost(n, batch, 0, 0, 256, 2047) is None
    B.dlf_net_destroy(n)


@pytest.mark.parametrize("c", [8, 13, 512, 2048])
def test_global_average_pools_keep_to_the_lds_limit(c):
    """max_lds_bytes is the limit of global average pools: the kernel of whole vectors, 8 KiB, only where it has them; the other takes none."""
    for limit in (0, 163840, 8192, 8191, 4096, 1):
        cfg, _ = _plan([nets.gavgpool(c)], 7, 7, 3, max_lds=limit)
        assert cfg["kind"] == 2 and cfg["lds_bytes"] == (8192 if c % 8 == 0 and (limit or 163840) >= 8192 else 0), (limit, cfg)


@pytest.mark.parametrize("layers,hw,max_lds", [
    ([nets.conv(512, 512, 1, 1, 0, "relu")], 7, 4096),           # 3.9 us with one wave, 5.4 on the pointwise kernel
    ([nets.conv(256, 256, 3, 1, 1, "relu")], 14, 4096),          # 8.9, 11.5 on the fused-group kernel
    ([nets.conv(512, 512, 3, 1, 1, "relu")], 7, 16384),          # 6.0 with four waves, 17.7
    ([nets.dwconv(256, 3, 1, "relu"), nets.conv(256, 256, 1, 1, 0, "relu")], 14, 16384)])
def test_fewer_waves_under_an_lds_limit(layers, hw, max_lds):
    """Where an LDS limit does not hold the waves a split-K launch has otherwise, it has fewer."""
    cfg, _ = _plan(layers, hw, hw, 1, max_lds=max_lds)
    assert cfg["kind"] in (6, 10) and cfg["variant"] >= 16 and 0 < cfg["lds_bytes"] <= max_lds, cfg


@pytest.mark.parametrize("layers,h,w,batch,max_lds", [
    ([nets.conv(96, 88, 3, 1, 1, "relu"), nets.maxpool(88, 2, 2, 0)], 6, 8, 2, 4096),
    ([nets.conv(256, 928, 5, 3, 4, "relu")], 33, 13, 1, 16384), ([nets.conv(352, 32, 3, 2, 1, "relu")], 37, 11, 1, 4096),
    ([nets.conv(64, 64, 3, 1, 1, "relu")], 32, 32, 7, 2048),
    ([nets.conv(3, 64, 7, 2, 3, "relu"), nets.maxpool(64, 3, 2, 1)], 64, 64, 1, 9408),
    ([nets.conv(128, 684380, 3, 1, 1, "relu")], 37, 36, 1, 0), ([nets.conv(1696, 966560, 3, 1, 1, "relu"), nets.maxpool(966560, 2, 2, 0)], 40, 22, 1, 32768)])
def test_layers_that_fit_no_tile_stay_infeasible(layers, h, w, batch, max_lds):
    """Layers that the tiled kernels refuse, for the LDS limit or their size, are refused by the library."""
    n = B.dlf_net_create(layers, h, w, layers[0]["cin"])
    assert B.dlf_group_cost(n, batch, 0, len(layers) - 1, 256, max_lds) is None
    with pytest.raises(B.DlfError) as e:
        _plan(layers, h, w, batch, max_lds=max_lds)
    assert e.value.status == B.DLF_ERR_INFEASIBLE
    B.dlf_net_destroy(n)


def test_no_layer_is_priced_below_its_bytes():
    """Whatever kernel a layer is planned on, its modelled cost covers the bytes it reads and writes once, residual operand
    and weights included, at the rate a large copy reaches (5.2 TB/s)."""
    rng = random.Random(11)
    seen = 0
    cases = [(32, 2048, 1, 58, 32, True), (32, 512, 1, 56, 40, True), (32, 256, 1, 40, 32, True), (2048, 512, 1, 7, 8, False)]
    for _ in range(150):
        k = rng.choice([1, 1, 3])
        cases.append((32 * rng.randint(1, 8), 8 * rng.randint(1, 259), k, rng.randint(1, 64 // k), rng.randint(1, 32), rng.random() < 0.5))
    for cin, cout, k, hw, batch, res in cases:
        layers = [nets.conv(cin, cin, 1, 1, 0, "relu"), nets.conv(cin, cout, 1, 1, 0, "none"),
                  nets.conv(cin, cout, k, 1, k // 2, "relu", input_from=0, residual_from=1 if res else -1)]
        n = B.dlf_net_create(layers, hw, hw, cin)
        m = batch * hw * hw
        floor_ps = (m * cin + m * cout * (2 if res else 1) + k * k * cin * cout) * 2 / 5.2
        for budget in (256, 64):
            cost = B.dlf_group_cost(n, batch, 2, 2, budget)
            seen += cost is not None
            assert cost is None or cost >= floor_ps, (cin, cout, k, hw, batch, res, budget, cost, floor_ps)
        B.dlf_net_destroy(n)
    for c, cout, stride, hw, batch in ((32, 512, 1, 40, 16), (64, 64, 1, 64, 16), (512, 512, 1, 14, 32), (1024, 1024, 1, 7, 32)):
        layers = [nets.dwconv(c, 3, stride, "relu"), nets.conv(c, cout, 1, 1, 0, "relu")]
        n = B.dlf_net_create(layers, hw, hw, c)
        B.dlf_debug_small_pair_mode(1, 1, 0)
        try:
            cost = B.dlf_group_cost(n, batch, 0, 1, 1 << 16)
        finally:
            B.dlf_debug_small_pair_mode(0)
        assert cost >= (batch * hw * hw * (c + cout) + c * cout) * 2 / 5.2, (c, cout, hw, batch, cost)
        B.dlf_net_destroy(n)
    assert seen > 250, seen


@pytest.mark.parametrize("c", range(32, 2049, 32))
def test_depthwise_pairs_pass_their_launcher(c):
    """Whatever the planner chooses for a depthwise layer and the 1x1 layer behind it, and every form of the split-K kernel that the
    testing hook names, is a launch that the kernel's launcher takes (1056 to 1376 channels: eight waves of five or six steps, 51
    to 73 KiB of LDS; wider pairs are two launches)."""
    for cout, hw, batch, stride in ((8, 7, 1, 1), (320, 14, 1, 2), (c, 7, 2, 1)):
        layers = [nets.dwconv(c, 3, stride, "relu"), nets.conv(c, cout, 1, 1, 0, "relu")]
        n = B.dlf_net_create(layers, hw, hw, c)
        one = dict(mode=B.TUNER_MANUAL, group_last=[1], group_budget=[256])
        forms = [(0, -1, 0)] + [(1, shape, waves) for shape in (0, 1) for waves in (0, 1, 2, 4, 8)]
        for mode, shape, waves in forms if c <= 1376 else forms[:1]:
            for kw in ([{}] if mode == 0 else []) + ([one] if c <= 1376 else []):
                B.dlf_debug_small_pair_mode(mode, shape, waves)
                try:
                    p = B.dlf_plan(n, batch, **kw)
                finally:
                    B.dlf_debug_small_pair_mode(0)
                B.dlf_debug_check_launches(p)
                cfg = B.dlf_plan_group_config(p, 0)
                assert mode == 0 or (cfg["kind"], cfg["variant"]) == (6, 16 + shape), (c, cout, shape, waves, cfg)
                B.dlf_plan_destroy(p)
        B.dlf_net_destroy(n)


def test_plans_pass_their_launchers():
    """Every group of the networks' plans, and of the plans under an LDS limit, is a launch that its launcher takes."""
    for net in (nets.vgg16(), nets.resnet18(173), nets.resnet50(), nets.mobilenet_v1(), nets.alexnet(), nets.identical_chain(64, 56, 4)):
        for batch in (1, 5, 32):
            for limit in (0, 65536, 16384):
                for mode in (B.TUNER_DP, B.TUNER_LAYERWISE):
                    h = B.dlf_net_create(net["layers"], net["in_h"], net["in_w"], net["in_c"])
                    try:
                        p = B.dlf_plan(h, batch, mode=mode, max_lds_bytes=limit)
                        B.dlf_debug_check_launches(p)
                        B.dlf_plan_destroy(p)
                    except B.DlfError as e:
                        assert limit > 0 and e.status == B.DLF_ERR_INFEASIBLE, (net["name"], batch, limit, e)
                    finally:
                        B.dlf_net_destroy(h)


def _default_plan(net, batch):
    h = B.dlf_net_create(net["layers"], net["in_h"], net["in_w"], net["in_c"])
    p = B.dlf_plan(h, batch)
    groups = [(g["first"], g["last"], g["model_cost"]) for g in B.dlf_plan_groups(p)]
    B.dlf_plan_destroy(p)
    return h, groups


@pytest.mark.parametrize("c,depth,hw,batch", [(32, 2, 28, 8), (32, 3, 28, 8), (32, 2, 40, 4), (32, 3, 40, 4), (32, 3, 56, 2), (64, 3, 28, 8),
                                              (64, 3, 40, 4), (64, 3, 56, 2), (64, 2, 28, 8)])
def test_small_chains_keep_their_one_launch(c, depth, hw, batch):
    """Chains that one launch of the fused-group kernel runs faster than a launch per layer (32 channels, three layers, 28 x 28, batch
    8: 12.7 us against 16.3; 64 channels: 15.6 against 18.3) are planned as one."""
    net = nets.identical_chain(c, hw, depth)
    h, groups = _default_plan(net, batch)
    assert [g[:2] for g in groups] == [(0, depth - 1)], groups
    # ... at no more than the layers one by one
    assert groups[0][2] <= sum(min(x for x in (B.dlf_group_cost(h, batch, i, i, b) for b in (32, 64, 128, 256)) if x) for i in range(depth))
    B.dlf_net_destroy(h)


def test_bottleneck_pairs_keep_their_one_launch():
    """ResNet-50's 3x3 -> 1x1 pairs of 128 channels at batch 1 - 4: 8.5 - 9.3 us in one launch, 9.4 - 13.8 in two."""
    for hw, batch in ((128, 4), (208, 4), (224, 1)):
        h, groups = _default_plan(nets.resnet50(hw), batch)
        assert {(17, 18), (20, 21), (23, 24)} <= {g[:2] for g in groups}, (hw, batch, groups)
        B.dlf_net_destroy(h)
    # ResNet-18's first blocks: 19.8 us in one launch, 22.2 in two
    h, groups = _default_plan(nets.resnet18(256), 13)
    assert {(2, 3), (4, 5)} <= {g[:2] for g in groups}, groups
    B.dlf_net_destroy(h)


@pytest.mark.parametrize("c,hw,batch,split", [(512, 9, 4, False), (512, 5, 12, False), (512, 10, 3, False), (256, 10, 8, False),
                                              (512, 9, 2, True), (512, 7, 1, True), (256, 9, 4, True), (256, 14, 1, True)])
def test_small_map_or_split_k(c, hw, batch, split):
    """3x3 layers of 256 and 512 channels go to the faster of the small-map kernel (512 at 9 x 9, batch 4: 9.6 us against 10.9; 256
    at 10 x 10, batch 8: 7.1 against 7.4) and the split-K kernel (512 at 9 x 9, batch 2: 8.4 against 9.4)."""
    cfg, _ = _plan([nets.conv(c, c, 3, 1, 1, "relu")], hw, hw, batch)
    assert cfg["kind"] == 10 and (cfg["variant"] >= 16) == split, cfg


@pytest.mark.parametrize("cin,cout,k,hw,batch,forms", [
    # short K: items of few channels (256 1x1 at 7 x 7 2.9 us, 3.6 on items of 64 channels; 32 3x3 at 14 x 14 3.2 and 3.7)
    (256, 256, 1, 7, 1, (16, 17)), (192, 192, 1, 9, 1, (16, 17)), (128, 128, 1, 14, 1, (16, 17)), (32, 32, 3, 14, 1, (16, 17)),
    # long K on items of 32 x 64: the small-map kernel (256 3x3 at 9 x 9, batch 16 7.1 us against 8.6; 512 at 20 x 20, batch 2 11.3 and 12.5)
    (256, 256, 3, 9, 16, (4,)), (512, 512, 3, 20, 2, (4,)), (512, 512, 3, 12, 4, (4,)), (2048, 512, 1, 9, 7, (12,)),
    # 1x1 layers of at most 192 such items (512 channels at 7 x 7, batch 12 5.5 us against 6.2; 1024 at batch 6 6.6 and 8.4)
    (512, 512, 1, 7, 12, (19,)), (1024, 1024, 1, 7, 6, (19,))])
def test_split_k_form_of_a_layer(cin, cout, k, hw, batch, forms):
    """Single convolutions on the faster of the split-K kernel's item shapes and the small-map kernel."""
    cfg, _ = _plan([nets.conv(cin, cout, k, 1, k // 2, "relu")], hw, hw, batch)
    assert cfg["kind"] == 10 and cfg["variant"] in forms, cfg


@pytest.mark.parametrize("c,cout,hw,batch,kinds", [
    # eight waves fill a CU: one item per CU at most (1024 channels at 7 x 7: batch 4 8.5 us against 10.2 in two launches, batch 6 15.1
    # against 13.6; 1280 at 7 x 7: batch 2 9.4 and 10.6, batch 4 16.4 and 12.5; 1376 at 10 x 10, batch 2 17.8 and 14.0)
    (1024, 1024, 7, 4, [6]), (1024, 1024, 7, 6, [5, 10]), (1024, 1024, 7, 8, [5, 10]), (1280, 1280, 7, 2, [6]), (1280, 1280, 7, 4, [5, 10]),
    (1376, 1376, 10, 2, [5, 10]),
    # four waves: a second item runs beside the first (512 channels at 14 x 14, batch 2 and 4: 6.2 and 8.8 us against 10.8 and 10.9)
    (512, 512, 14, 2, [6]), (512, 512, 14, 4, [6]),
    # the tile kernel, for at most 128 output channels
    (128, 128, 56, 1, [7]), (128, 128, 28, 3, [7]), (64, 64, 28, 6, [7]), (256, 128, 14, 12, [7]), (256, 128, 20, 6, [7]), (256, 256, 20, 3, [6])])
def test_pairs_beyond_one_item_per_cu(c, cout, hw, batch, kinds):
    """Depthwise + 1x1 pairs go to the split-K kernel only where it is the faster plan."""
    n = B.dlf_net_create([nets.dwconv(c, 3, 1, "relu"), nets.conv(c, cout, 1, 1, 0, "relu")], hw, hw, c)
    p = B.dlf_plan(n, batch)
    got = [B.dlf_plan_group_config(p, g)["kind"] for g in range(B.dlf_plan_num_groups(p))]
    B.dlf_plan_destroy(p)
    B.dlf_net_destroy(n)
    assert got == kinds


def test_first_layer_pair_is_not_priced_lower_for_more_images():
    """3 -> 64 -> 64 channels at 128 x 128 as one launch of the block kernel (forced): batches that leave half of the chip idle are all
    priced by the same rule."""
    costs = []
    n = B.dlf_net_create([nets.conv(3, 64, 3, 1, 1, "relu"), nets.conv(64, 64, 3, 1, 1, "relu")], 128, 128, 3)
    B.dlf_debug_block3x3_mode(1, 14, 14, 32)
    try:
        costs = [B.dlf_group_cost(n, b, 0, 1, 256) for b in (1, 2, 3, 4)]
    finally:
        B.dlf_debug_block3x3_mode(0)
        B.dlf_net_destroy(n)
    assert costs == sorted(costs), costs


def test_kernels_of_the_evaluated_networks():
    """The kernels that the networks' plans are known to hold, so that a silent change of the planner's choice (and with it of what
    the parity tests of these networks cover) shows."""
    def forms(net, batch):
        h = B.dlf_net_create(net["layers"], net["in_h"], net["in_w"], net["in_c"])
        p = B.dlf_plan(h, batch)
        out = [(c["kind"], c["variant"]) for c in (B.dlf_plan_group_config(p, g) for g in range(B.dlf_plan_num_groups(p)))]
        B.dlf_plan_destroy(p)
        B.dlf_net_destroy(h)
        return out
    vgg = forms(nets.vgg16(), 16)                        # register-weight kernel, with the first layer in front; small-map kernel
    assert {(4, 16), (4, 17), (4, 22)} <= set(vgg) and any(k == 10 and v < 16 for k, v in vgg) and len(vgg) <= 16, vgg
    res = forms(nets.resnet50(), 1)                      # split-K kernel, with projections; 3x3 -> 1x1 pairs; bottleneck blocks
    assert sum(k == 10 and v >= 16 for k, v in res) >= 20 and any(k == 8 and v >= 16 for k, v in res), res
    assert sum(k == 11 for k, _ in res) == 3 and any(k == 12 for k, _ in res) and len(res) <= 43, res
    mob = forms(nets.mobilenet_v1(), 1)                  # split-K depthwise pairs
    assert sum(k == 6 and v >= 16 for k, v in mob) >= 8 and len(mob) <= 14, mob


def test_depthwise_layers_have_no_step_in_their_price():
    """A streaming depthwise layer's price grows with the batch as its time does (512 channels at 14 x 14: 6.9 us at batch 1, 8.3 at 25 and
    32), and MobileNet-v1's pairs stay pairs (217 x 217, batch 25: 12.1 us a pair, 19.1 as two launches)."""
    for c, hw, measured in ((512, 14, {1: 6.9, 8: 7.4, 16: 7.6, 25: 8.3, 32: 8.3, 48: 8.7}), (256, 28, {1: 7.1, 4: 7.2, 12: 8.0, 16: 8.3, 32: 9.0}),
                            (1024, 7, {1: 4.6, 16: 5.1, 32: 5.8, 48: 6.1})):
        n = B.dlf_net_create([nets.dwconv(c, 3, 1, "relu")], hw, hw, c)
        costs = {b: B.dlf_group_cost(n, b, 0, 0, 256) / 1e6 for b in range(1, 49)}
        B.dlf_net_destroy(n)
        assert all(costs[b] <= costs[b + 1] <= costs[b] + 0.75 for b in range(1, 32)), costs  # (256 channels: a second item from 33 on)
        assert all(abs(costs[b] - us) <= 0.15 * us for b, us in measured.items()), {b: (costs[b], us) for b, us in measured.items()}
    for hw, batch in ((217, 25), (224, 16), (224, 64)):
        h, groups = _default_plan(nets.mobilenet_v1(hw), batch)
        assert {(13, 14), (15, 16), (17, 18), (19, 20), (21, 22)} <= {g[:2] for g in groups}, (hw, batch, groups)
        B.dlf_net_destroy(h)


@pytest.mark.parametrize("c,hw,batch,depth", [
    (64, 27, 8, 4),      # 19.4 us as one launch, 23.4 as four
    (64, 29, 5, 4),
    (32, 69, 1, 2),      # 9.8, 10.8
    (96, 28, 4, 3),      # 16.9, 19.4
    (96, 28, 3, 4),      # 22.9, 25.9
    (128, 28, 3, 4),     # 27.6, 29.7
    (128, 28, 4, 3),     # 19.0, 22.0
])
def test_chains_above_128_items_keep_one_launch(c, hw, batch, depth):
    h, groups = _default_plan(nets.identical_chain(c, hw, depth), batch)
    assert [g[:2] for g in groups] == [(0, depth - 1)], groups
    B.dlf_net_destroy(h)


@pytest.mark.parametrize("c,hw,batch,depth", [
    (96, 28, 4, 2),      # 13.0 us as two launches, 13.3 as one
    (128, 28, 4, 2),     # 15.0, 15.7
    (192, 28, 3, 4),     # 37.6, 47.1
    (64, 28, 3, 4),      # 17.4, 18.6
])
def test_chains_that_are_faster_layer_by_layer_are_not_fused(c, hw, batch, depth):
    h, groups = _default_plan(nets.identical_chain(c, hw, depth), batch)
    assert [g[:2] for g in groups] == [(i, i) for i in range(depth)], groups
    B.dlf_net_destroy(h)
