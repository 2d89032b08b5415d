"""Rows of the MLP round where they are awkward to load: input widths that end within a 16-byte piece
or within a 16-column tile, rows shorter than a piece, and rounds shorter than the number of mini-batches that
are on the way.  Against the CPU oracle, tick by tick.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hidden,batch", [
    (1, 16, 16), (2, 20, 4), (3, 32, 32),   # shorter than a piece
    (4, 16, 16), (5, 16, 5), (6, 33, 32), (7, 16, 16),   # the tail reaches back over one, two, three columns and whole pieces
    (16, 16, 16), (17, 16, 16), (30, 48, 20), (31, 16, 32),
    (255, 150, 16),      # the last tile of all eight waves; more unit groups than are fetched at a time
    (257, 70, 32),       # the first width of the larger form
    (515, 40, 32), (783, 24, 16),   # two workgroups per unit group: the tail is the second's
    (895, 256, 32),  # widest, most units
])
def test_row_widths_and_short_rounds(oracle_libs, d, hidden, batch):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    # rounds of 0, 1, 2, 3 and 4 recursions: nothing ahead, one mini-batch, two, and both register sets twice
    wl = W.config2(n_clients=2, n_total=2 * 37, d=d, hidden=hidden, batch=batch, rounds=5, a=batch, b=0)
    wl.compute_factor = np.array([1, 2], dtype=np.int32)
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


@pytest.mark.parametrize("d", [3, 21, 530])
def test_neighbouring_rows_stay_out(oracle_libs, d):
    """Rows that are never drawn hold infinities and NaN: nothing of them may reach a drawn row's piece."""
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = W.config2(n_clients=2, n_total=2 * 400, d=d, hidden=24, batch=16, rounds=2, a=0, b=32)
    probe = Oracle(wl, "f64")
    drawn = [{probe.sample_index(c, q, wl.X[c].shape[0]) for q in range(2 * 32)} for c in range(2)]
    for c in range(2):
        for k in range(wl.X[c].shape[0]):
            if k not in drawn[c]:
                wl.X[c][k] = np.nan if k % 2 else np.inf
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


@pytest.mark.parametrize("n,d,hidden,batch", [
    (2, 20, 16, 33),     # one sample in the second step
    (3, 256, 40, 64),    # both steps full, every wave has its two tiles
    (2, 3, 5, 63),       # narrow rows
    (2, 530, 100, 48),   # two workgroups per unit group, ragged columns
    (2, 784, 32, 64),    # ... whole tiles
    (9, 700, 256, 50),   # seven tiles a wave: sixteen unit groups, more clients than are resident two by two
    (5, 150, 240, 37),   # more unit groups than are fetched at a time
    (9, 688, 256, 50),   # seven tiles a wave in whole pieces
    (48, 784, 100, 64),  # ... seven unit groups, two launches
])
def test_mini_batches_in_two_steps(oracle_libs, n, d, hidden, batch):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = W.config2(n_clients=n, n_total=n * 90, d=d, hidden=hidden, batch=batch, rounds=4, a=batch, b=0)
    if n == 3:
        wl.compute_factor = np.array([1, 2, 1], dtype=np.int32)
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


@pytest.mark.parametrize("n,d,hidden,batch", [(4, 60, 40, 50), (3, 784, 100, 33), (9, 688, 256, 64)])
def test_mini_batches_in_two_steps_on_a_ring(oracle_libs, n, d, hidden, batch):
    """Peer to peer: rounds that go on from the own replica."""
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = W.config2(n_clients=n, n_total=n * 90, d=d, hidden=hidden, batch=batch, rounds=3, a=batch, b=batch)
    wl.topology = W.ring_topology(n)
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()
