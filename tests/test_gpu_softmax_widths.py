"""Per-sample softmax regression: the forms with fewer waves or columns give the bits of the widest one.

A row followed by columns of zeros up to the widest form's width adds zeros to every sum, in the same order, so the two
forms must agree bit for bit on the columns that are there.  Equality, no tolerance.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

WIDEST = 3072


def _run(wl, d):
    from paper_2112_13935_amd.runner import Run
    run = Run(wl)
    got = []
    while not run.lib.aet_all_done(wl.rounds):
        for c, k in run.run_round():
            got.append(("U", run.lib.aet_get_U(c, k)))
            got.append(("w", run.lib.aet_get_weights(c)))
            got.append(("loss", np.float64(run.lib.aet_get_round_info(c, k)["loss"])))
        run.exchange()
    got.append(("w", run.lib.aet_get_weights(-1)))
    run.close()
    width = wl.model.in_size()
    out = []
    for what, v in got:
        if what == "loss":
            out.append(v)
            continue
        rows = v[:10 * width].reshape(10, width)
        assert not rows[:, d:].any()
        out.append(np.concatenate([rows[:, :d].ravel(), v[10 * width:]]))
    return out


# one, two, four, eight waves; two, three, four and five columns a thread: the first and last width of each
@pytest.mark.parametrize("d", [1, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 1536, 1537, 2048, 2049, 2560, 2561])
def test_every_form_gives_the_widest_ones_bits(d):
    wl = W.config1(n_clients=3, n_per=50, d=d, rounds=4, a=21, b=3)   # up to 66 recursions: more than a block of row numbers
    wide = W.config1(n_clients=3, n_per=50, d=WIDEST, rounds=4, a=21, b=3)
    for c in range(3):
        wide.X[c] = np.zeros((wl.X[c].shape[0], WIDEST), np.float32)
        wide.X[c][:, :d] = wl.X[c]
        wide.y[c] = wl.y[c]
    assert wide.seed == wl.seed
    assert not wl.w0.any() and not wide.w0.any()
    for a, b in zip(_run(wl, d), _run(wide, d)):
        assert np.array_equal(a, b)
