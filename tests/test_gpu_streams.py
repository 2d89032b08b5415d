"""Several contexts on one GPU, each on a stream and in a host thread of its own, whose rounds run
in clusters of workgroups that wait for each other: their launches take turns, none gives up
waiting, and every context gets the bits it gets alone.  Run with  -m gpu  on an MI355X."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def softmax_batch(n, d, batch):
    wl = W.config5(n_clients=n, n_per=40, d=d, rounds=4)
    wl.model.batch = batch
    wl.a = wl.b = batch
    return wl


def cnn(n, hw, width, fc, batch, rounds=6):
    return W.config4(n_clients=n, n_per=60, hw=hw, width=width, fc=fc, batch=batch, rounds=rounds, a=batch, b=2 * batch)


MIXES = {
    # clusters of 32 workgroups: one of them fills an XCD
    "two padded MLPs": lambda: [W.config2(n_clients=3, n_total=180, d=784, hidden=250, batch=20, rounds=6, a=20, b=40) for _ in range(2)],
    "exact and padded MLP": lambda: [W.config2(n_clients=8, n_total=480, d=784, hidden=256, batch=16, rounds=6, a=16, b=32),
                                     W.config2(n_clients=8, n_total=480, d=784, hidden=250, batch=20, rounds=6, a=20, b=40)],
    "four engines": lambda: [W.config2(n_clients=5, n_total=300, d=784, hidden=100, batch=20, rounds=6, a=20, b=40),
                             W.config3(n_clients=9, n_per=40, hw=16, batch=20, rounds=4, a=20, b=40),
                             softmax_batch(20, 3072, 50), softmax_batch(9, 400, 20)],
    # clusters of 5 workgroups, of 1 to 25, of 16 and of 32: beside each other where there is room
    "small CNNs": lambda: [cnn(3, 12, 6, 18, 5), cnn(8, 16, 16, 64, 1), cnn(2, 8, 16, 64, 16), cnn(1, 16, 16, 64, 32)],
    "four alike": lambda: [cnn(6, 8, 16, 64, 8, 12) for _ in range(4)],
    # an XCD each
    "single clients": lambda: [cnn(1, 16, 16, 64, 32) for _ in range(3)] + [cnn(1, 8, 16, 64, 24), cnn(1, 12, 6, 18, 5)],
    # dense models: beside each other where there is room; two steps a recursion in the first four
    "dense models": lambda: [W.config2(n_clients=n, n_total=n * 70, d=d, hidden=h, batch=b, rounds=12, a=0, b=2 * b)
                             for n, d, h, b in ((1, 30, 10, 64), (4, 100, 100, 48), (1, 784, 100, 64), (8, 784, 128, 33), (3, 50, 32, 16), (9, 300, 240, 20))],
    "small CNNs and dense models": lambda: [cnn(3, 12, 6, 18, 5), cnn(1, 16, 16, 64, 32)] + [
        W.config2(n_clients=n, n_total=n * 70, d=d, hidden=40, batch=b, rounds=8, a=0, b=2 * b) for n, d, b in ((2, 60, 64), (5, 530, 33))],
    "small CNNs and an MLP": lambda: [cnn(3, 12, 6, 18, 5), cnn(9, 8, 8, 32, 4),
                                      W.config2(n_clients=8, n_total=480, d=784, hidden=256, batch=16, rounds=6, a=16, b=32)],
}


@pytest.mark.parametrize("mode,variants", [(2, 0), (0, 1)])
@pytest.mark.parametrize("make", [lambda n: cnn(n, 8, 5, 12, 5),
                                  lambda n: W.config2(n_clients=n, n_total=n * 70, d=784, hidden=100, batch=40, rounds=6, a=40, b=80)],
                         ids=["cnn", "two steps"])
def test_contexts_beside_each_other_by_the_other_ways_of_exchange(make, mode, variants):
    """Words through memory, without asking and because one workgroup of each client names another XCD, with the XCD of
    the first client given: the bits of a context that is alone."""
    import torch
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.binding import AetSgd
    from paper_2112_13935_amd.runner import upload
    lib = load_library()

    def job(ctx, wl):
        ctx.aet_reset()
        ctx.aet_run_ticks(wl.a, wl.b, wl.rounds, wl.eta0, wl.beta, wl.power, wl.agg_scale)
        return ctx.aet_get_weights_device(-1)
    jobs = []
    for n in (1, 3, 2):
        wl = make(n)
        X, y = upload(wl)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ctx = AetSgd(wl.model, X, y, wl.w0, wl.seed, max_inflight=1, max_rounds=wl.rounds, stream=stream)
            alone = None if jobs else job(ctx, wl).clone()
        torch.cuda.synchronize()
        jobs.append((ctx, wl, stream, alone))
    lib.aet_test_select_kernels(mode, 0)
    lib.aet_test_variants(variants)
    try:
        out = []
        for ctx, wl, stream, _ in jobs + jobs:
            with torch.cuda.stream(stream):
                out.append(job(ctx, wl))
        torch.cuda.synchronize()
        for ctx, *_, alone in jobs:   # (what the last round that asked found: the first context's was before)
            assert ctx.aet_test_one_xcd_clients() == (1 if mode and alone is not None else 0)
    finally:
        lib.aet_test_select_kernels(0, 0)
        lib.aet_test_variants(0)
    assert torch.equal(out[0], jobs[0][3])
    for a, b in zip(out[:3], out[3:]):
        assert torch.equal(a, b) and torch.isfinite(a).all()
    with torch.cuda.stream(jobs[0][2]):      # and as usual again
        job(jobs[0][0], jobs[0][1])
        assert jobs[0][0].aet_test_one_xcd_clients() == 1
    for ctx, *_ in jobs:
        ctx.aet_synchronize()
        ctx.aet_destroy()


@pytest.mark.parametrize("mix", sorted(MIXES))
def test_contexts_on_their_own_streams(mix):
    import torch
    from paper_2112_13935_amd.binding import AetSgd
    from paper_2112_13935_amd.runner import upload
    jobs = []
    for wl in MIXES[mix]():
        wl.compute_factor = wl.is_straggler = None
        wl.delay_min = wl.delay_max = 0
        X, y = upload(wl)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()     # the shards are there
        jobs.append((wl, AetSgd(wl.model, X, y, wl.w0, wl.seed, max_inflight=1, max_rounds=wl.rounds, stream=stream), stream))

    def job(wl, lib, stream):
        with torch.cuda.stream(stream):
            lib.aet_reset()
            lib.aet_run_ticks(wl.a, wl.b, wl.rounds, wl.eta0, wl.beta, wl.power, wl.agg_scale)
            return lib.aet_get_weights_device(-1)

    alone = []
    for j in jobs:
        w = job(*j)
        torch.cuda.synchronize()
        alone.append(w.cpu())
    # from one thread, the streams in turn, nothing waited for in between
    mixed = [[job(*j) for j in jobs] for _ in range(3)]
    torch.cuda.synchronize()
    for row in mixed:
        for a, b in zip(row, alone):
            assert torch.equal(a.cpu(), b)
    # from a thread each
    got, errors = [None] * len(jobs), []

    def work(i):
        try:
            for _ in range(6):
                got[i] = job(*jobs[i])
        except Exception as e:   # noqa: BLE001 (handed to the test's own thread)
            errors.append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for (wl, lib, stream), a, b in zip(jobs, got, alone):
        lib.aet_synchronize()    # raises if a wait had run out
        assert torch.equal(a.cpu(), b)
        assert np.isfinite(b.numpy()).all()
        lib.aet_destroy()


def test_dense_models_do_not_wait_for_each_other():
    """A short job on another stream ends while a long one of one client is under way.  (Four hardware queues serve all
    streams: one of several short ones has another queue than the long one.)"""
    import torch
    from paper_2112_13935_amd.binding import AetSgd
    from paper_2112_13935_amd.runner import upload

    def context(recursions):
        wl = W.config2(n_clients=1, n_total=200, d=100, hidden=100, batch=64, rounds=1, a=0, b=64 * recursions)
        X, y = upload(wl)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        return wl, AetSgd(wl.model, X, y, wl.w0, wl.seed, max_inflight=1, max_rounds=1, stream=stream), stream

    def job(wl, lib, stream):
        with torch.cuda.stream(stream):
            lib.aet_reset()
            lib.aet_run_ticks(wl.a, wl.b, wl.rounds, wl.eta0, wl.beta, wl.power, wl.agg_scale)
            return stream.record_event()
    long_one, short = context(20000), [context(3) for _ in range(4)]   # 170 ms and 30 us
    for j in [long_one] + short:
        job(*j).synchronize()
    end = job(*long_one)
    ends = [job(*j) for j in short]
    ahead = 0
    for e in ends:
        while not e.query():
            pass
        ahead += not end.query()
    end.synchronize()
    for _, lib, _ in [long_one] + short:
        lib.aet_synchronize()
        lib.aet_destroy()
    assert ahead >= 1
