"""Mini-batch softmax on matrix tiles: parity with the CPU oracle for every form of the round (blocks per
wave, tiles of samples, rows that are no whole number of 16-byte pieces; test_softmax_batch_form.py sees to it that
these are all) where its blocks, shares and tiles end.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n, d, batch, rounds=3):
    wl = W.config5(n_clients=n, n_per=40, d=d, rounds=rounds)
    wl.model.batch = batch
    wl.a = wl.b = batch
    return wl


#: clients, columns, mini-batch, and the form that runs them: matrix tiles with up to 4 x runs blocks of 16 columns a wave
#: (one to three runs), room for so many samples, all columns there or not or fewer than four; or a column per lane
CASES = [
    # fewer columns than a 16-byte piece; one piece; one column into the next; a block and one more
    (2, 1, 2, "tiles 1x8 tiny"), (2, 3, 9, "tiles 1x16 tiny"), (2, 3, 20, "tiles 1x32 tiny"), (2, 3, 33, "tiles 1x64 tiny"),
    (3, 4, 16, "tiles 1x16 any"), (3, 5, 17, "tiles 1x32 any"), (2, 17, 64, "tiles 1x64 any"),
    # waves without a block; blocks that end inside a wave's share, by two and three columns
    (2, 100, 9, "tiles 1x16 any"), (3, 510, 32, "tiles 1x32 any"), (2, 511, 31, "tiles 1x32 any"),
    # one and two workgroups, all blocks there: 512 and 1,024; one more column
    (2, 512, 32, "tiles 1x32 full"), (2, 512, 8, "tiles 1x8 full"), (2, 1024, 16, "tiles 1x16 full"), (2, 1025, 20, "tiles 1x32 any"),
    (2, 1025, 8, "tiles 1x8 any"),
    # six workgroups, all blocks there and one column short
    (2, 3072, 64, "tiles 1x64 full"), (2, 3071, 32, "tiles 1x32 any"), (2, 3071, 5, "tiles 1x8 any"),
    # four workgroups; 64 samples
    (60, 2048, 20, "tiles 1x32 full"), (60, 2046, 50, "tiles 1x64 any"),
    # eight blocks a wave: one workgroup, two, three, all blocks there or not, with room for each number of samples
    (100, 700, 8, "tiles 2x8 any"), (41, 3072, 8, "tiles 2x8 full"), (41, 3056, 9, "tiles 2x16 any"), (41, 3072, 9, "tiles 2x16 full"),
    (130, 1600, 20, "tiles 2x32 any"), (65, 2048, 20, "tiles 2x32 full"), (65, 2046, 50, "tiles 2x64 any"), (65, 2048, 50, "tiles 2x64 full"),
    # twelve blocks a wave: two workgroups, one, all blocks there or not
    (128, 3072, 32, "tiles 3x32 full"), (128, 2900, 18, "tiles 3x32 any"), (240, 1500, 24, "tiles 3x32 any"),
    (96, 3072, 16, "tiles 3x16 full"), (96, 2928, 16, "tiles 3x16 any"),
    # a column per lane: one and three columns, half a tile of samples, odd rows
    (260, 300, 4, "lanes 1x8"), (96, 3000, 8, "lanes 3x8"), (96, 3071, 13, "lanes 3x16"), (96, 2930, 16, "lanes 3x16"),
]


@pytest.mark.parametrize("n,d,batch,form", CASES)
def test_parity(oracle_libs, n, d, batch, form):
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
