"""Convolutions that put the gradient behind a 2 x 2 pooling layer together themselves: parity with the
CPU oracle at the edges of their tiles and for the layers that may follow.  Run with  -m gpu  on an
MI355X."""
import pytest

import workloads as W
from test_gpu_conv_split import _conv, _maps

pytestmark = pytest.mark.gpu

POOL = W.Layer(W.POOL)

CASES = {
    # 8 x 8: four samples per workgroup, the last with two
    "8x8": lambda: _maps(4, 50, (32, 8, 8), [_conv(64), _conv(64), POOL]),
    # 8 x 8 with half a block of channels on both sides
    "8x8_48": lambda: _maps(4, 51, (32, 8, 8), [_conv(48), _conv(48), POOL]),
    # 12 rows of 32: the second row block half empty; a convolution that masks behind
    "12x32": lambda: _maps(3, 48, (16, 12, 32), [_conv(32), _conv(32), POOL, W.Layer(W.CONV, 16, 3, 1, 1)]),
    # no ReLU: nothing is masked, negative winners keep their gradient
    "no_relu": lambda: _maps(4, 50, (16, 16, 16), [_conv(32), W.Layer(W.CONV, 64, 3, 1, 0), POOL]),
    # two pooling layers: the upper one hands a masked gradient down
    "two_pools": lambda: _maps(4, 50, (16, 16, 16), [_conv(32), _conv(64), POOL, POOL]),
    # a hidden dense layer behind
    "dense": lambda: _maps(4, 50, (16, 16, 16), [_conv(32), _conv(64), POOL, W.Layer(W.DENSE, 64, relu=1)]),
    # small launches, both backward kernels in one: 16 and 32 channels, 16 x 16 and 8 x 8
    "pair": lambda: _maps(2, 7, (8, 16, 16), [_conv(16), _conv(16), POOL, _conv(32), _conv(32), POOL]),
    # rows that end inside a block of them, 24 channels, no ReLU
    "pair_10x12": lambda: _maps(3, 5, (8, 10, 12), [_conv(16), W.Layer(W.CONV, 24, 3, 1, 0), POOL]),
    "pair_6x20": lambda: _maps(1, 1, (8, 6, 20), [_conv(32), _conv(32), POOL]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_parity(oracle_libs, name):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = CASES[name]()
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


def test_no_launch_of_its_own():
    """The cases above take this form: no kernel of the pooling layer runs on the way back."""
    from paper_2112_13935_amd.runner import Run
    for name in sorted(CASES):
        run = Run(CASES[name]())
        fam = run.lib.profile_family_names().index("k_pool_bwd")
        run.lib.aet_profile_enable(fam, True)
        run.run_round()
        launches, _ = run.lib.aet_profile_read(fam)
        run.close()
        # (one recursion; the upper of the two pooling layers keeps its kernel)
        assert launches == (name == "two_pools"), name
