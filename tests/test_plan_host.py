"""What the planner chooses, on the host (no GPU): the promises of the header about which kernels a call may take."""
import random

import pytest

import paper_1805_00907_amd as glowmi
from plan_probe import Probe


@pytest.fixture(scope="module")
def probe():
    return Probe()


def _desc(n, h, w, c, k, r, st=1):
    return glowmi.ConvDesc(n, h, w, c, k, r, r, st, st, r // 2, r // 2, r // 2, r // 2, 1)


# the switches that together keep a layer on the fp32 matrix cores (glowmi.h, tuning knobs)
PIECE_SWITCHES = ("F32_P3", "F32_PATCH", "F32_FC_TILES", "F32_K3", "F32_K3C64", "F32_PW_BF16", "F32_SMALLC_BF16")
PIECE_KERNELS = {"patch", "p3", "k3", "k3c64", "short", "fc_tiles"}      # (pw and smallc have an fp32 form each)


@pytest.mark.parametrize("workspace", [0, 1 << 36], ids=["no_workspace", "workspace"])
def test_the_documented_switches_keep_every_layer_on_the_fp32_matrix_cores(probe, knobs, workspace):
    for name in PIECE_SWITCHES:
        knobs.set(name, 0)
    rng = random.Random(1)
    cases = [_desc(3, 60, 60, c, 64, 1) for c in (24, 56, 96, 160, 224)]
    for _ in range(600):
        r = rng.choice([1, 1, 3])
        cases.append(_desc(rng.choice([1, 2, 5, 16]), rng.randint(7, 80), rng.randint(7, 80), 4 * rng.randint(4, 90),
                           4 * rng.randint(4, 120), r, rng.choice([1, 1, 2])))
    for d in cases:
        for packed in (False, d.c % 8 == 0):
            plan = probe.conv(d, packed=packed, workspace=workspace)
            assert plan.kernel not in PIECE_KERNELS, ((d.n, d.h, d.w, d.c, d.k, d.r), packed, plan)


def test_planes_given_without_a_workspace_leave_a_layer_in_fp32_arithmetic(probe):
    """The header: a caller that needs non-finite values kept apart passes no workspace; of layers with their filter's planes
    given only 3x3 ones on large maps, which the 3x3 tile kernels take, run on the fp16 matrix cores then."""
    rng = random.Random(3)
    seen = set()
    for _ in range(1500):
        r = rng.choice([1, 3])
        d = _desc(rng.choice([1, 2, 5, 16]), rng.randint(7, 100), rng.randint(7, 100), 8 * rng.randint(2, 80), 8 * rng.randint(2, 140), r,
                  rng.choice([1, 1, 2]))
        with_room = probe.conv(d, packed=True, workspace=glowmi.conv2d_packed_workspace_bytes(d))
        assert with_room == probe.conv(d, packed=True), "the query covers the plan"
        plan = probe.conv(d, packed=True, workspace=0)
        assert plan.workspace == 0
        if plan.kernel in ("patch", "k3", "k3c64"):
            assert probe.conv(d, packed=True).kernel in ("patch", "k3", "k3c64")
            # (a tile of theirs, 160 pixels x 128 channels, for six in ten CUs at least)
            assert r == 3 and d.stride_h == 1 and d.n * d.h * d.w * d.k >= 3000000, ((d.n, d.h, d.w, d.c, d.k, d.r, d.stride_h), plan)
        else:
            assert plan.kernel not in ("p3", "fc_tiles"), plan
        seen.add((with_room.kernel, plan.kernel))
    assert ("patch", "tiled") in seen and ("patch", "patch") in seen


# with an offset in the filter's codes another kernel may run than without, and the query does not know which
QUERY_FC = [(627, 8004, 3204), (1024, 9216, 4096), (600, 4100, 2052), (65, 4100, 1000), (16, 2052, 1000)]


@pytest.mark.parametrize("w_offset", [0, 7, -128])
def test_the_int8_queries_cover_a_filter_with_an_offset(probe, w_offset):
    rng = random.Random(2)
    shapes = QUERY_FC + [(rng.randint(1, 1100), 4 * rng.randint(60, 2300), 4 * rng.randint(16, 1150)) for _ in range(1500)]
    for m, k, n in shapes:
        plan = probe.qfc(m, k, n, w_offset)
        assert plan.workspace <= glowmi.qfc_workspace_bytes(m, k, n), ((m, k, n), plan)
    for _ in range(1500):
        r = rng.choice([1, 3])
        d = _desc(rng.choice([1, 2, 5, 16]), rng.randint(7, 60), rng.randint(7, 60), rng.choice([4, 8, 8, 3]) * rng.randint(4, 90),
                  rng.choice([4, 8, 1]) * rng.randint(16, 120), r, rng.choice([1, 1, 2]))
        for addend in (False, True):
            plan = probe.conv(d, quantized=True, addend=addend, w_offset=w_offset)
            assert plan.workspace <= glowmi.qconv2d_workspace_bytes(d), ((d.n, d.h, d.w, d.c, d.k, d.r), plan)


def test_planes_given_do_not_move_a_layer_of_the_patch_kernel_to_the_contraction_over_planes(probe):
    """That one lies up to 1.3 times as far from 64-bit sums."""
    rng = random.Random(4)
    for _ in range(1500):
        r = rng.choice([1, 3, 3])
        d = _desc(rng.randint(1, 24), rng.randint(7, 60), rng.randint(7, 60), 8 * rng.randint(2, 90), 8 * rng.randint(2, 128), r,
                  rng.choice([1, 2]))
        if probe.conv(d).kernel == "patch":
            assert probe.conv(d, packed=True).kernel != "p3", ((d.n, d.h, d.w, d.c, d.k, d.r, d.stride_h),)


@pytest.mark.parametrize("layer,kernel", [((1, 87, 87, 232, 256, 3), "wide"), ((18, 18, 18, 216, 640, 3), "wide"),
                                          ((9, 34, 34, 240, 288, 3), "wide"), ((5, 33, 45, 72, 120, 3), "short")], ids=str)
def test_deep_int8_filters_stay_with_the_wide_kernel(probe, layer, kernel):
    assert probe.conv(_desc(*layer), quantized=True).kernel == kernel


@pytest.mark.parametrize("call,kernel", [((196, 2360, 344), "fc_small"), ((128, 1548, 132), "fc_small"), ((900, 2356, 396), "wide"),
                                         ((196, 2368, 352), "wide"), ((359, 3160, 3760), "wide")], ids=str)
def test_int8_rows_in_fours_stay_on_the_strip_kernel_within_its_traffic(probe, call, kernel):
    assert probe.qfc(*call).kernel == kernel


@pytest.mark.parametrize("layer,st,kernel", [((1, 11, 9, 352, 616, 3), 1, "small_split"), ((2, 38, 38, 368, 84, 3), 2, "small_split"),
                                             ((1, 7, 7, 512, 512, 3), 1, "small_split"), ((1, 14, 14, 256, 256, 3), 1, "few"),
                                             ((2, 11, 11, 136, 496, 3), 1, "few"), ((1, 17, 17, 512, 128, 1), 1, "few")], ids=str)
def test_deep_layers_stay_in_slices_where_those_are_the_faster_ones(probe, layer, st, kernel):
    d = _desc(*layer, st)
    assert probe.conv(d, workspace=glowmi.conv2d_workspace_bytes(d)).kernel == kernel


@pytest.mark.parametrize("layer,kernel", [((2, 32, 25, 160, 824, 1), "short"), ((4, 37, 37, 176, 200, 1), "short"), ((5, 39, 39, 288, 80, 1), "few")], ids=str)
def test_pointwise_layers_of_up_to_224_channels_take_the_faster_kernel(probe, layer, kernel):
    d = _desc(*layer)
    assert probe.conv(d, addend=True, workspace=glowmi.conv2d_workspace_bytes(d)).kernel == kernel


# layers that single-layer thresholds had on the slower kernel: 28.2 us on conv_short_i8 and 20.2 on tiles, 7.1 and 5.9 (conv_small_i8), 5.0
# on conv_small_i8 and 3.7 on conv_few_i8, 53 on tiles of 128 x 64 and 29 on conv_short_i8
@pytest.mark.parametrize("layer,st,kernel", [((26, 82, 82, 112, 87, 3), 2, "tiled"), ((5, 36, 36, 48, 376, 3), 2, "small"),
                                             ((3, 25, 32, 144, 16, 3), 1, "few"), ((13, 112, 112, 168, 32, 3), 1, "short")], ids=str)
def test_int8_layers_take_the_kernel_of_the_lowest_estimate(probe, layer, st, kernel):
    assert probe.conv(_desc(*layer, st), quantized=True).kernel == kernel


# the same in fp32: 72 us on tiles and 43 on conv_short_f32, 12.7 on the patch kernel and 9.2 on conv_short_f32, 5.3 on conv_small_f32
# and 4.1 on conv_few_f32
@pytest.mark.parametrize("layer,st,kernel", [((30, 51, 72, 32, 400, 1), 1, "short"), ((17, 39, 39, 160, 192, 1), 2, "short"),
                                             ((1, 55, 55, 144, 32, 1), 1, "few")], ids=str)
def test_fp32_layers_take_the_kernel_of_the_lowest_estimate(probe, layer, st, kernel):
    d = _desc(*layer, st)
    assert probe.conv(d, workspace=glowmi.conv2d_workspace_bytes(d)).kernel == kernel


@pytest.mark.parametrize("m,k,n,slices", [(330, 3568, 2293, 9), (314, 4088, 2219, 9), (570, 6296, 280, 16), (819, 1912, 3872, 7), (987, 1848, 1648, 7)])
def test_deeper_slabs_of_fully_connected_layers_keep_the_slices(m, k, n, slices):
    """A program that keeps a buffer of the size its calls once asked for keeps its kernel: the slices of the reduction are no more than those
    of slabs of 32; and not so few that the sums in them get longer than by a slab filled up."""
    parts = (glowmi.fc_packed_workspace_bytes(m, k, n) - 4 * m * k) / (4 * m * n)      # behind the input's planes and what goes with them
    assert 0.85 * slices <= parts < slices + 0.05, parts


@pytest.mark.parametrize("n,h,c,k,form", [(1, 14, 256, 256, ("few", 3)), (1, 10, 400, 64, ("few", 3)), (3, 8, 608, 136, ("few", 3)),
                                          (1, 20, 312, 48, ("few", 3)), (1, 28, 128, 128, ("few", 1)), (1, 7, 512, 512, ("small_split", 0)),
                                          (5, 19, 512, 16, ("small_split", 0)), (1, 16, 504, 56, ("small_split", 0))])
def test_estimates_alone_say_which_few_pixel_layers_keep_their_patch_in_lds(probe, n, h, c, k, form):
    """3x3 layers whose tiles make one round of the compute units, however deep (608 channels 15.1 us in slices, 11.7 here); against slices
    only what lies an eighth below them (504 channels 8.9 us in slices, 10.4 here)."""
    d = _desc(n, h, h, c, k, 3, 2 if h == 19 else 1)
    plan = probe.conv(d, workspace=glowmi.conv2d_workspace_bytes(d))
    assert (plan.kernel, plan.tile if plan.kernel == "few" else 0) == form, plan


@pytest.mark.parametrize("m,k,n,kernel", [(770, 2224, 4000, "fc_tiles"), (256, 4096, 4096, "fc_tiles"), (1024, 4096, 4096, "p3"),
                                          (1455, 2424, 1072, "fc_tiles")])
def test_fully_connected_calls_that_cut_their_weights_take_the_faster_kernel(probe, m, k, n, kernel):
    """Against the contraction over planes as it is: its rounds of the compute units and its slices count."""
    assert probe.fc(m, k, n).kernel == kernel


def test_fully_connected_calls_that_ask_for_next_to_no_workspace_go_on_doing_so(probe):
    """What fc_tiles_f32 takes in place of the contraction over planes by its operations alone has no scratch to ask for."""
    for m, k, n in [(838, 712, 4008), (609, 536, 4264), (881, 3200, 2264), (948, 912, 3944)]:
        assert probe.fc(m, k, n).kernel == "fc_tiles" and glowmi.fc_workspace_bytes(m, k, n) <= 256


def _drawn_3x3(seed, count):
    """3x3 layers of 48 to 1024 channels on small and middling maps, one in six with channels out of eights."""
    rng = random.Random(seed)
    for _ in range(count):
        step = rng.choice([8, 8, 8, 8, 8, 1])
        h = rng.randint(5, 60)
        yield _desc(rng.choice([1, 2, 4, 9, 20]), h, h if rng.random() < 0.6 else rng.randint(5, 60), step * rng.randint(48 // step, 1024 // step),
                    step * rng.randint(16 // step, 1024 // step), 3, rng.choice([1, 2]))


def _is(d):
    return (d.n, d.h, d.w, d.c, d.k, d.stride_h)


def test_reductions_in_parts_only_replace_kernels_of_the_same_arithmetic(probe, knobs):
    """Layers that run on fp32 operands keep them, and infinities to the outputs they reach: tiles, slices and conv_few_f32 stay."""
    layers = list(_drawn_3x3(5, 1200)) + [_desc(8, 28, 28, 256, 256, 3, 2), _desc(4, 14, 14, 512, 512, 3, 2), _desc(7, 10, 10, 632, 56, 3)]
    calls = [(d, packed, add) for d in layers for packed in (False, True) if not packed or d.c % 8 == 0 for add in (False, True)]
    plans = [probe.conv(d, packed=packed, addend=add) for d, packed, add in calls]
    knobs.set("F32_PATCH_PARTS", 1)
    whole = [probe.conv(d, packed=packed, addend=add) for d, packed, add in calls]
    taken = set()
    for (d, packed, add), plan, before in zip(calls, plans, whole):
        if plan.kernel == "patch" and plan.split_k > 1:
            taken.add(before.kernel)
            assert before.kernel in ("patch", "p3"), (_is(d), packed, add, before, plan)
        else:
            assert plan == before, (_is(d), packed, add)
    assert taken == {"patch", "p3"}


def test_planes_given_do_not_change_how_the_patch_kernel_sums(probe):
    """Bit for bit the same results where that kernel serves a layer both ways: the same form and the same parts of its reduction."""
    both = in_parts = 0
    for d in list(_drawn_3x3(6, 3000)) + [_desc(9, 41, 41, 200, 232, 3, 2), _desc(1, 50, 50, 600, 224, 3)]:
        if d.c % 8:
            continue
        plain = probe.conv(d, workspace=glowmi.conv2d_workspace_bytes(d))
        packed = probe.conv(d, packed=True, workspace=glowmi.conv2d_packed_workspace_bytes(d))
        if plain.kernel == packed.kernel == "patch":
            both += 1
            in_parts += plain.split_k > 1
            assert (plain.tile, plain.split_k) == (packed.tile, packed.split_k), (_is(d), plain, packed)
    assert both > 500 and in_parts > 50


@pytest.mark.parametrize("layer,st", [((14, 100, 100, 624, 16, 3), 1), ((25, 9, 7, 2000, 232, 3), 2), ((16, 66, 66, 544, 32, 3), 1)], ids=str)
def test_layers_beyond_those_measured_run_whole(probe, layer, st):
    """140000 and 69696 pixels; 2000 channels, 42 us on the contraction over planes and 52 in parts."""
    d = _desc(*layer, st)
    for packed in (False, True):
        plan = probe.conv(d, packed=packed)
        assert plan.kernel != "patch" or plan.split_k == 1, (packed, plan)


def test_reductions_in_parts_stay_within_the_layers_measured(probe):
    rng, taken = random.Random(8), 0
    for _ in range(4000):
        h, c, k = rng.randint(5, 110), 8 * rng.randint(4, 300), 8 * rng.randint(2, 60)
        d = _desc(rng.choice([1, 3, 10, 30]), h, h, c, k, 3, rng.choice([1, 2]))
        plan = probe.conv(d, packed=rng.random() < 0.5)
        if plan.kernel == "patch" and plan.split_k > 1:
            taken += 1
            assert 96 <= c <= 2048 and d.n * ((h - 1) // d.stride_h + 1) ** 2 <= 40000 and 36 * c * k <= 16 << 20, (_is(d), plan)
    assert taken > 100


def test_parts_of_a_reduction_are_no_longer_sums_than_without_them(probe, knobs):
    """The wavefronts that share a tile's reduction, times the parts, are no fewer than in one part, and a part has two chunks and more: what sums
    nearer to 64-bit ones need (forms: wavefronts sharing a block, channels of a chunk)."""
    sharing, chunk = (4, 2, 8, 2, 1, 2), (64, 32, 128, 32, 32, 32)
    layers = list(_drawn_3x3(7, 2500)) + [_desc(4, 56, 56, 112, 110, 3, 2), _desc(1, 29, 29, 506, 96, 3), _desc(1, 48, 48, 432, 48, 3)]
    plans = [probe.conv(d, packed=d.c % 8 == 0) for d in layers]
    knobs.set("F32_PATCH_PARTS", 1)
    compared = 0
    for d, plan in zip(layers, plans):
        if plan.kernel != "patch" or plan.split_k == 1:
            continue
        chunks = -(-d.c // chunk[plan.tile])
        assert -(-chunks // plan.split_k) >= 2, (_is(d), plan)
        whole = probe.conv(d, packed=d.c % 8 == 0)
        if whole.kernel == "patch":
            compared += 1
            assert plan.split_k * sharing[plan.tile] >= sharing[whole.tile], (_is(d), whole, plan)
    assert compared > 30


def test_layers_that_stay_whole_are_not_searched_for_parts(probe):
    """Planning a layer of conv_patch_f32 in one part costs the host what it costs with parts switched off (a search over the parts of every form
    was 1.2 times that)."""
    whole = [d for d in _drawn_3x3(9, 400) if d.c % 8 == 0 and probe.conv(d, packed=True)[:3:2] == ("patch", 1)][:60]
    assert len(whole) == 60
    off, on = (sum(ns) for ns in zip(*(probe.conv_versus(d, "F32_PATCH_PARTS", 1, packed=True) for d in whole)))
    assert on < 1.12 * off, (off, on)


def test_fully_connected_calls_that_stay_elsewhere_are_not_estimated(probe):
    """Planning a call over planes costs the host what it costs with fc_few_f32 switched off (its estimates, twice, were 1.3 times that)."""
    rng = random.Random(6)
    calls = [c for c in ((rng.randint(600, 1600), 8 * rng.randint(300, 1000), 8 * rng.randint(200, 500)) for _ in range(200)) if probe.fc(*c).kernel == "p3"][:50]
    assert len(calls) == 50
    off, on = (sum(ns) for ns in zip(*(probe.fc_versus(*c, "F32_FC_FEW", 0) for c in calls)))
    assert on < 1.12 * off, (off, on)


def test_less_room_than_the_parts_take_is_no_room_for_them(probe, knobs):
    """Whatever a call hands over below its query: what it would run if there were no parts.  Over planes that is, in 256 bytes, the same kernel in
    one part, but for the layers that parts take from the contraction over planes."""
    layers, seen = [], set()
    for d in _drawn_3x3(10, 2500):
        for packed in (False, d.c % 8 == 0):
            query = (glowmi.conv2d_packed_workspace_bytes if packed else glowmi.conv2d_workspace_bytes)(d)
            plan = probe.conv(d, packed=packed, workspace=query)
            if plan.kernel == "patch" and plan.split_k > 1:
                assert plan.workspace <= query
                rooms = (0, 16, 256, plan.workspace - 4 * plan.split_k * d.n * d.k, plan.workspace // 2, plan.workspace - 1)
                layers.append((d, packed, rooms, [probe.conv(d, packed=packed, workspace=room) for room in rooms]))
    knobs.set("F32_PATCH_PARTS", 1)
    for d, packed, rooms, plans in layers:
        whole = probe.conv(d, packed=packed).kernel
        for room, plan in zip(rooms, plans):
            assert plan == probe.conv(d, packed=packed, workspace=room), (_is(d), packed, room)
        if packed:
            assert plans[2].kernel == "patch" if whole == "patch" else plans[2].kernel not in PIECE_KERNELS, (_is(d), whole, plans[2])
        seen.add((packed, whole))
    assert seen == {(False, "patch"), (False, "p3"), (True, "patch"), (True, "p3")} and len(layers) > 60


@pytest.mark.parametrize("m,k,n,form", [(80, 176, 400, 0), (308, 112, 96, 0), (3, 134, 2736, 0), (18, 304, 1032, 1),
                                        (1, 2048, 1000, 6), (4, 2048, 1000, 4), (13, 1320, 208, 6), (44, 4007, 48, 6)])
def test_smaller_tiles_only_where_they_gain_more_than_the_estimates_miss(probe, m, k, n, form):
    """FullyConnected on tiles of 16 x 16 (forms 0 to 2): the first four calls 3.4 to 3.9 us there, 3.8 to 4.4 on smaller ones."""
    plan = probe.fc(m, k, n)
    assert plan.kernel == "fc_few" and plan.tile == form, plan
