"""Mini-batch softmax on matrix tiles: parity with the CPU oracle for every form of the round (blocks per
wave, tiles of samples, rows that are no whole number of 16-byte pieces) where its blocks, shares
and tiles end.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n, d, batch, rounds=3):
    wl = W.config5(n_clients=n, n_per=40, d=d, rounds=rounds)
    wl.model.batch = batch
    wl.a = wl.b = batch
    return wl


@pytest.mark.parametrize("n,d,batch", [
    # fewer columns than a 16-byte piece; one piece; one column into the next; a block and one more
    (2, 1, 2), (2, 3, 33), (3, 4, 16), (3, 5, 17), (2, 17, 64),
    # waves without a block; blocks that end inside a wave's share, by two and three columns
    (2, 100, 9), (3, 510, 32), (2, 511, 31),
    # one and two workgroups, all blocks there: 512 and 1,024; one more column
    (2, 512, 32), (2, 1024, 16), (2, 1025, 20), (2, 1025, 8),
    # six workgroups, all blocks there and one column short
    (2, 3072, 64), (2, 3071, 32), (2, 3071, 5),
    # eight blocks a wave: two workgroups, one; 64 samples beside them
    (60, 2048, 20), (100, 700, 8), (60, 2046, 50),
    # twelve blocks a wave: two workgroups, one, all blocks there or not
    (128, 3072, 32), (128, 2900, 18), (240, 1500, 24), (96, 2930, 16),
    # a column per lane: one and three columns, half a tile of samples, odd rows
    (260, 300, 4), (96, 3000, 8), (96, 3071, 13),
])
def test_parity(oracle_libs, n, d, batch):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = _workload(n, d, batch, rounds=3 if n < 50 else 2)
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


def test_values_that_are_not_finite_stay_in_their_client():
    """An infinite feature of one client's rows: its U is not finite, its neighbours' are, and columns
    beyond it keep the rest of the rows apart."""
    from paper_2112_13935_amd.runner import Run
    wl = _workload(3, 75, 20, rounds=1)
    wl.X[1] = wl.X[1].copy()
    wl.X[1][:, 74] = np.inf
    run = Run(wl)
    run.run_round()
    us = [run.lib.aet_get_U(c, 0) for c in range(3)]
    run.close()
    assert np.isfinite(us[0]).all() and np.isfinite(us[2]).all()
    assert not np.isfinite(us[1]).all()
