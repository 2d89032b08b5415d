"""The words that the workgroups of a client exchange stay in their XCD's L2 or go through memory;
either way the same words arrive, so the models have the same bits.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _softmax(n, d, batch):
    wl = W.config1(n_clients=n, n_per=100, d=d, rounds=4, a=batch, b=batch)
    wl.model.batch = batch
    return wl


CASES = {
    "mlp_two_halves": lambda: W.config2(n_clients=3, n_total=3 * 100, rounds=4),
    "mlp_one_group": lambda: W.config2(n_clients=9, n_total=9 * 100, d=50, hidden=16, rounds=4),
    "mlp_padded_17_groups_of_7": lambda: W.config2(n_clients=17, n_total=17 * 60, hidden=100, batch=20, rounds=3, a=20, b=20),
    "mlp_16_groups": lambda: W.config2(n_clients=2, n_total=2 * 60, d=300, hidden=256, batch=16, rounds=3, a=16, b=16),
    "lenet": lambda: W.config3(n_clients=3, n_per=60, rounds=3),
    "lenet_two_clusters": lambda: W.config3(n_clients=3, n_per=60, batch=20, rounds=3, a=20, b=20),
    "softmax_cluster_of_six": lambda: _softmax(3, 3072, 20),
    "softmax_cluster_of_three_b5": lambda: _softmax(11, 1100, 5),   # records that end inside a line
    "softmax_cluster_of_two": lambda: _softmax(90, 600, 8),
    "softmax_alone": lambda: _softmax(3, 40, 8),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_same_words_through_memory(name):
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.runner import Run
    lib = load_library()
    out = []
    for mode in (0, 2):
        lib.aet_test_select_kernels(mode, 0)
        try:
            run = Run(CASES[name]())
            run.run_all()
            out.append(run.lib.aet_get_weights(-1))
            run.close()
        finally:
            lib.aet_test_select_kernels(0, 0)
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0], out[1])
