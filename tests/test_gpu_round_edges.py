"""GPU parity of the round kernels at the sizes where their tiling can go wrong: remainders of
the unrolled recursion loops, padded tiles, the smallest and largest sizes a path takes.
Every case runs tick by tick against the CPU oracle.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need the HIP path")
    from paper_2112_13935_amd import load_library
    load_library()
    from paper_2112_13935_amd.runner import Run
    return Run


def _lockstep(gpu, wl):
    from oracle import Oracle
    from parity import lockstep
    run, orc = gpu(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


@pytest.mark.parametrize("d", [10, 600, 3072])
@pytest.mark.parametrize("s0", [0, 1, 46, 95])
def test_softmax_round_lengths(gpu, oracle_libs, d, s0):
    """Round lengths s0, s0+1, ... s0+3: every remainder of the recursions in a group of four, a
    block of 48 recursions met exactly, missed by one and passed by one, and the empty round."""
    _lockstep(gpu, W.config1(n_clients=2, n_per=40, d=d, rounds=4, a=1, b=s0))
