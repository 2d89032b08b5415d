"""The words that the workgroups of a client exchange stay in their XCD's L2 or go through memory, as the
workgroups find that they share an XCD or not; either way the same words arrive, so the models have the
same bits.  Run with  -m gpu  on an MI355X."""
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
    "mlp_two_steps": lambda: W.config2(n_clients=9, n_total=9 * 80, d=50, hidden=100, batch=48, rounds=3, a=48, b=48),
    "mlp_two_steps_two_halves": lambda: W.config2(n_clients=3, n_total=3 * 80, d=784, hidden=128, batch=64, rounds=3, a=64, b=64),
    "mlp_two_steps_seven_tiles": lambda: W.config2(n_clients=9, n_total=9 * 80, d=688, hidden=256, batch=50, rounds=3, a=50, b=50),
    "lenet": lambda: W.config3(n_clients=3, n_per=60, rounds=3),
    "lenet_two_clusters": lambda: W.config3(n_clients=3, n_per=60, batch=20, rounds=3, a=20, b=20),
    "softmax_cluster_of_six": lambda: _softmax(3, 3072, 20),
    "softmax_cluster_of_three_b17": lambda: _softmax(11, 1100, 17),   # records that end inside a line
    "softmax_cluster_of_two": lambda: _softmax(90, 600, 20),
    "softmax_alone_three_columns": lambda: _softmax(90, 600, 8),
    "softmax_alone": lambda: _softmax(3, 40, 8),
}


def _rounds(name, mode, variants):
    """The model after all rounds, how many clients had their words in one L2 at the end, and all clients."""
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.runner import Run
    lib = load_library()
    lib.aet_test_select_kernels(mode, 0)
    lib.aet_test_variants(variants)
    try:
        run = Run(CASES[name]())
        run.run_all()
        out = run.lib.aet_get_weights(-1), run.lib.aet_test_one_xcd_clients(), run.n
        run.close()
    finally:
        lib.aet_test_select_kernels(0, 0)
        lib.aet_test_variants(0)
    return out


@pytest.mark.parametrize("name", sorted(CASES))
def test_same_words_through_memory(name):
    """In L2, through memory without asking, and through memory because one workgroup of each client
    names another XCD."""
    model, shared, clients = _rounds(name, 0, 0)
    assert shared == (0 if name.startswith("softmax_alone") else clients)
    assert np.isfinite(model).all()
    for mode, variants in ((2, 0), (0, 1)):
        other, shared, _ = _rounds(name, mode, variants)
        assert shared == 0
        assert np.array_equal(model, other)
