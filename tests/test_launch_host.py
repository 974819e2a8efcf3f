"""What calls hand to the runtime (no GPU): kernels, their dynamic LDS and the limit that was set for it."""
import pytest

from launch_probe import LaunchProbe


def _block(mid, c=None):
    return [(mid, 1), (mid, 3), (c or 4 * mid, 1)]


@pytest.mark.parametrize("first", [True, False], ids=["addend_first", "addend_second"])
def test_every_block_kernel_has_its_own_lds_limit(first):
    """More dynamic LDS than 64 KB is given to a kernel only once its limit was raised: the kernel with and the one without an addend
    have the same type, and each needs it, whichever runs first."""
    with LaunchProbe() as probe:
        probe.knob("I8_BLOCK", 2)
        kernels = set()
        for add in (first, not first):
            for mid in (32, 64, 96):
                launches = probe.sequence((1, 14, 14, 4 * mid), _block(mid), add=[2] if add else [])
                assert len(launches) == 1 and "block_i8_kernel" in launches[0].kernel, launches
                kernels.add(launches[0].kernel)
                assert launches[0].limit >= launches[0].lds, launches
        assert len(kernels) == 6


@pytest.mark.parametrize("name,value", [("I8_TILE", 0), ("I8_SPLIT", 1), ("I8_SMALL_MAX_TILES", 0), ("I8_WIDE_SPLIT", 1), ("I8_WIDE_NBUF", 2),
                                        ("I8_PW_MIN_ITEMS", 1), ("I8_K3_MIN_BLOCKS", 1), ("I8_K3_WAVES", 8), ("I8_K3_GATHER", 1), ("I8_FEW", 0),
                                        ("I8_FEW_TILE", 0), ("I8_SHORT", 0), ("I8_SHORT_FORM", 0), ("I8_BLOCK", 0)])
def test_a_switch_for_single_int8_layers_keeps_them_single(name, value):
    """A sequence that runs as one launch by itself, and under a switch that asks for another kernel as three layers."""
    with LaunchProbe() as probe:
        assert len(probe.sequence((4, 28, 28, 256), _block(64), add=[2])) == 1
        probe.knob(name, value)
        launches = probe.sequence((4, 28, 28, 256), _block(64), add=[2])
        assert len(launches) >= 3 and "block_i8" not in str(launches), launches
        probe.knob("I8_BLOCK", 2)                        # asked for itself
        assert len(probe.sequence((4, 28, 28, 256), _block(64), add=[2])) == 1


def test_a_block_that_cannot_run_as_one_launch_is_not_searched_for_its_tile():
    """Fewer than 24 channels in the middle: the sequence costs the host what it costs with the one-launch form switched off (a search over
    the tiles of a 56 x 56 map was 1.4 times that)."""
    with LaunchProbe() as probe:
        assert len(probe.sequence((32, 56, 56, 64), _block(16), add=[2])) >= 3
        off, on = probe.versus("I8_BLOCK", 0)
        assert on < 1.15 * off, (off, on)


@pytest.mark.parametrize("layers,runs,launches", [
    ([(32, 1), (32, 3), (128, 1), (128, 3)], 1, 2), ([(128, 3), (32, 1), (32, 3), (128, 1)], 1, 2),
    ([(96, 1), (28, 1), (28, 3), (112, 1), (64, 1)], 1, 3), ([(64, 1), (64, 3), (256, 1), (56, 1), (56, 3), (256, 1)], 2, 2),
    ([(128, 1), (32, 1), (32, 3), (128, 1), (24, 1), (24, 3), (96, 1)], 2, 3), ([(32, 1), (32, 3)], 0, 2),
], ids=["block_layer", "layer_block", "layer_block_layer", "block_block", "layer_block_block", "two_layers"])
def test_runs_in_longer_sequences_are_found(layers, runs, launches):
    """1x1, 3x3, 1x1 anywhere in a sequence is one launch, and every other layer is launched once."""
    with LaunchProbe() as probe:
        probe.knob("I8_BLOCK", 2)
        got = probe.sequence((2, 9, 11, 64), layers)
        assert sum("block_i8" in l.kernel for l in got) == runs and len(got) == launches, got


@pytest.mark.parametrize("neighbours", [[], [(512, 1)], [(1024, 3)]], ids=["alone", "small", "large"])
@pytest.mark.parametrize("x,layer", [((16, 5, 7, 840), (248, 3)), ((5, 17, 17, 472), (64, 3)), ((1, 50, 50, 600), (224, 3))], ids=str)
def test_a_layer_of_a_sequence_is_launched_as_its_arena_was_sized(x, layer, neighbours):
    """Arenas name no room for reductions in parts, and whatever a layer finds free in one, its reduction is in one part."""
    with LaunchProbe() as probe:
        got = probe.sequence(x, [layer] + neighbours, quantized=False)
        probe.knob("F32_PATCH_PARTS", 1)
        assert got == probe.sequence(x, [layer] + neighbours, quantized=False)
