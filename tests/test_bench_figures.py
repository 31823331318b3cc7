"""What bench.py prices a launch with has to be the work of that launch."""
import bench

LAYERS = ("conv1_fwd", "conv2_fwd", "conv3_fwd")


def test_conv_launches_of_a_step_are_three_passes_in_all():
    """The launches of every form a step takes (a launch per layer, all layers in one, or the pass on s by layers beside the
    passes over s' in one, fp32 batches of 60 to 128) add up to three forward passes."""
    B, R = 96, 19
    whole = 3 * B * (bench.F_CONV1 + bench.F_CONV2 + bench.F_CONV3)
    for launches in (LAYERS, ("conv123_fwd",), LAYERS + ("conv123_fwd",)):
        fl = bench.flops_per_launch(B, R, bench.conv_passes(launches))
        assert sum(fl[k] for k in launches) == whole, launches
