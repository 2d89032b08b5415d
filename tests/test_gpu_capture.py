"""A job on a context of aet_init_static recorded into a HIP graph: every replay gives the result
of an eager run on the data that lie in the shards at that moment.  The rounds that exchange
through tagged records carry their tags into the graph, so that the records of one replay must
not pass for those of the next.  Run with  -m gpu  on an MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def softmax_batch():
    wl = W.config5(n_clients=5, n_per=40, d=1100, rounds=3)
    wl.model.batch = 20
    wl.a = wl.b = 20
    return wl


CASES = {
    "softmax": lambda: W.config1(n_clients=3, n_per=40, d=60, rounds=3, a=5, b=7),
    "softmax, mini-batch 20, clusters of 3": softmax_batch,
    "dense-ReLU-dense 50-32-10": lambda: W.config2(n_clients=4, n_total=200, d=50, hidden=32, batch=16, rounds=3, a=16, b=32),
    "padded 600-40-10": lambda: W.config2(n_clients=4, n_total=200, d=600, hidden=40, batch=20, rounds=3, a=20, b=40),
    "two steps 50-32-10": lambda: W.config2(n_clients=4, n_total=200, d=50, hidden=32, batch=40, rounds=3, a=40, b=40),
    "two steps 600-40-10": lambda: W.config2(n_clients=4, n_total=300, d=600, hidden=40, batch=64, rounds=3, a=64, b=64),
    "one round": lambda: W.config2(n_clients=4, n_total=200, d=600, hidden=40, batch=20, rounds=1, a=0, b=80),
    "LeNet 16 x 16, mini-batch 16": lambda: W.config3(n_clients=2, n_per=40, hw=16, batch=16, rounds=2, a=16, b=32),
    "LeNet 16 x 16, mini-batch 20": lambda: W.config3(n_clients=2, n_per=40, hw=16, batch=20, rounds=2, a=20, b=40),
    "small CNN": lambda: W.config4(n_clients=2, n_per=40, hw=8, width=6, fc=20, batch=4, rounds=2, a=4, b=8),
    # made with that engine asked for
    "layer engine": lambda: W.config4(n_clients=2, n_per=40, hw=8, width=6, fc=20, batch=4, rounds=2, a=4, b=8),
}


def job(wl, lib):
    lib.aet_reset()
    lib.aet_run_ticks(wl.a, wl.b, wl.rounds, wl.eta0, wl.beta, wl.power, wl.agg_scale)
    return lib.aet_get_weights_device(-1)


@pytest.mark.parametrize("name", sorted(CASES))
def test_every_replay_is_the_job_on_the_present_data(name):
    import torch
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.binding import AetSgd
    from paper_2112_13935_amd.runner import Run, upload
    wl = CASES[name]()
    wl.compute_factor = wl.is_straggler = None
    wl.delay_min = wl.delay_max = 0
    X, y = upload(wl)
    stream = torch.cuda.Stream()
    load_library().aet_test_select_kernels(1 if name == "layer engine" else 0, 0)
    try:
        eager = Run(wl, shards=(X, y))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            lib = AetSgd(wl.model, X, y, wl.w0, wl.seed, max_inflight=1, max_rounds=wl.rounds, stream=stream, static_workspace=True)
    finally:
        load_library().aet_test_select_kernels(0, 0)
    with torch.cuda.stream(stream):
        warm = job(wl, lib).clone()      # eager work of this context ahead of the recording
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out = job(wl, lib)
    first = job(wl, eager.lib)
    torch.cuda.synchronize()
    assert torch.equal(warm, first)
    rng = np.random.default_rng(7)
    results = []
    for replay in range(4):
        for c in range(wl.n_clients):    # other samples in the same shards
            X[c].copy_(torch.from_numpy(wl.X[c] * np.float32(1 + 0.1 * replay)))
            y[c].copy_(torch.from_numpy(rng.permutation(wl.y[c]).astype(np.int32)))
        want = job(wl, eager.lib).clone()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {replay}: {float((out - want).abs().max()):.2e}"
        results.append(want)
    assert not torch.equal(results[0], results[1])
    lib.aet_synchronize()
    with torch.cuda.stream(stream):      # and an eager job after the replays
        after = job(wl, lib).clone()
    torch.cuda.synchronize()
    assert torch.equal(after, results[-1])
    lib.aet_destroy()
    eager.close()
