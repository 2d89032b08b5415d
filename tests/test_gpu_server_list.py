"""The server's step at the lengths of an arrival list where it takes another kernel: in the arguments of the kernel that
walks the list (up to 32), of the one that sums it in groups (up to 496), and through device memory (beyond).

Every tick's new model against the old one minus sum of scale * U in 64 bits.  Tolerance: n products and n additions in
fp32, each off by at most u = 2^-24 of what it rounds: (n + 3) u (|w| + sum |scale U|).  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [31, 32, 33, 47, 255, 256, 257, 495, 496, 497, 513])
def test_model_is_the_old_one_minus_the_scaled_sums(n):
    from paper_2112_13935_amd.runner import Run
    wl = W.config1(n_clients=n, n_per=20, d=13, rounds=3, a=1, b=2)
    run = Run(wl)
    w = run.lib.aet_get_weights(-1).astype(np.float64)
    while not run.lib.aet_all_done(wl.rounds):   # the slots come back in another order each tick
        done = run.run_round()
        terms = []
        for c, k in done:
            scale = np.float32(wl.agg_scale) * np.float64(run.lib.aet_get_round_info(c, k)["eta"])
            terms.append(np.float64(np.float32(scale)) * run.lib.aet_get_U(c, k).astype(np.float64))
        applied = run.exchange()
        assert len(done) == n and len(applied) == n
        want = w - np.sum(terms, axis=0)
        got = run.lib.aet_get_weights(-1).astype(np.float64)
        bound = (n + 3) * 2.0 ** -24 * (np.abs(w) + np.sum(np.abs(terms), axis=0))
        assert (np.abs(got - want) <= bound).all()
        w = got
    run.close()
