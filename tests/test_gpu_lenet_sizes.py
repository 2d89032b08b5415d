"""Every instantiation of the LeNet round (input side, one cluster or two, padded or not) against the CPU oracle.  Run with  -m gpu  on an MI355X."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hw,batch", [
    (2, 16, 16), (2, 20, 16), (2, 28, 16),
    (2, 16, 3), (2, 20, 5), (2, 28, 15),
    (2, 16, 18), (3, 20, 20), (2, 20, 32), (2, 28, 31),
    (65, 16, 16), (33, 20, 20),   # one client more than is resident: two launches
])
def test_lenet_sizes(oracle_libs, n, hw, batch):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = W.config3(n_clients=n, n_per=40, hw=hw, batch=batch, rounds=3 if n < 10 else 2, a=batch, b=batch)
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()
