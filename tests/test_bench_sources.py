"""Which files bench.py takes a fused kernel to be made from: recorded counters are quoted only while
their fingerprint is the recorded one."""
import os

import pytest


@pytest.mark.parametrize("fam,files", [
    ("k_mlp_round", ["kernels_mlp.hip", "aet_device.h", "aet_internal.h", "cluster_plan.h", "cluster_post.h"]),
    ("k_lenet_round", ["kernels_lenet.hip", "aet_device.h", "aet_internal.h", "cluster_plan.h", "cluster_post.h"]),
    ("k_softmax_round", ["kernels_softmax.hip", "aet_device.h", "aet_internal.h"]),
])
def test_every_header_counts(fam, files):
    import bench
    got = [os.path.basename(f) for f in bench.kernel_sources(fam)]
    assert got[0] == files[0] and set(files) <= set(got)


def test_layer_kernels_have_no_counters():
    import bench
    assert bench.kernel_sources("k_conv_fwd") is None
    assert bench.counter_traffic("k_conv_fwd", "cfg4_cnn32") is None
