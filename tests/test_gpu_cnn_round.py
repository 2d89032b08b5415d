"""The fused round of small convolutional networks: parity with the CPU oracle where its tiles, chunks and
shares end, the same bits by either way of exchange, and which calls take it.  Run with  -m gpu  on an
MI355X."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

POOL = W.Layer(W.POOL)


def _conv(cout, relu=1):
    return W.Layer(W.CONV, cout, 3, 1, relu)


def _cnn(n, hw, width, fc, batch, rounds=2, b=None):
    return W.config4(n_clients=n, n_per=70, hw=hw, width=width, fc=fc, batch=batch, rounds=rounds, a=batch, b=b or batch)


def _net(n, batch, shape, layers, rounds=2):
    """Maps of the given (channels, rows, columns); the layers up to the classes."""
    wl = _cnn(n, 8, 4, 8, batch, rounds)
    wl.model = W.Model(*shape, layers + [W.Layer(W.DENSE, 10)], batch)
    wl.X = [W._rng(3, c).standard_normal((70, wl.model.in_size()), dtype=np.float32) for c in range(n)]
    wl.w0 = W.init_weights(wl.model, 5)
    return wl


def _dense(n, relu=1):
    return W.Layer(W.DENSE, n, relu=relu)


CASES = {
    # channels and units that fill no tile, 6 x 6 maps
    "12x12_odd": lambda: _cnn(3, 12, 6, 18, 5),
    # gradient buffers shared by two geometries; one workgroup takes samples, others help with the update
    "16x16_one_sample": lambda: _cnn(2, 16, 16, 64, 1),
    # weights staged layer by layer; 33 samples: two turns, the last of one
    "12x12_b33": lambda: _cnn(2, 12, 16, 64, 33, 1),
    # 48 channels: a layer's weights in several chunks
    "8x8_24_chunks": lambda: _cnn(2, 8, 24, 100, 17),
    # 32 -> 64 channels, 256 units
    "8x8_32": lambda: _cnn(5, 8, 32, 256, 16, 1),
    # the smallest maps: 4 x 4, 2 x 2, one feature a channel
    "4x4": lambda: _cnn(9, 4, 5, 10, 3),
    # 1,024 pixels, two tiles of channels at most
    "32x32": lambda: _cnn(1, 32, 4, 30, 7, 1),
    # odd maps, nothing pooled: rows that end inside groups of four pixels
    "5x7_no_pool": lambda: _net(3, 5, (2, 5, 7), [_conv(9), _conv(17), _dense(33)]),
    # one convolution only: no gradient of an input anywhere
    "one_layer": lambda: _net(2, 6, (3, 10, 6), [_conv(5), POOL, _dense(20)]),
    # no ReLU at all: negative winners keep their gradient
    "no_relu": lambda: _net(2, 6, (4, 8, 8), [_conv(16, 0), POOL, _conv(18, 0), _dense(20, 0)]),
    # more classes' worth of layers: seven convolutions
    "seven_layers": lambda: _net(2, 4, (1, 8, 12), [_conv(4), _conv(8), POOL, _conv(8), _conv(12), _conv(12), _conv(8), POOL, _conv(5), _dense(40)]),
}


def _launches(run, family="k_cnn_round"):
    fam = run.lib.profile_family_names().index(family)
    run.lib.aet_profile_enable(fam, True)
    run.run_round()
    n = run.lib.aet_profile_read(fam)[0]
    run.close()
    return n


@pytest.mark.parametrize("name", sorted(CASES))
def test_parity(oracle_libs, name):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    assert _launches(Run(CASES[name]())) == 1
    wl = CASES[name]()
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


def test_parity_on_a_ring(oracle_libs):
    """Replicas that are kept from round to round, late messages."""
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = _cnn(4, 12, 6, 18, 5, rounds=3)
    wl.topology = W.ring_topology(4)
    wl.agg_scale = 1 / 3
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


@pytest.mark.parametrize("name", ["12x12_odd", "12x12_b33", "8x8_24_chunks", "16x16_one_sample"])
def test_same_words_through_memory(name):
    """In one L2, through memory without asking, and through memory because one workgroup of each client
    names another XCD: the same bits."""
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.runner import Run
    lib, out = load_library(), []
    for mode, variants in ((0, 0), (2, 0), (0, 1)):
        lib.aet_test_select_kernels(mode, 0)
        lib.aet_test_variants(variants)
        try:
            run = Run(CASES[name]())
            run.run_all()
            out.append(run.lib.aet_get_weights(-1))
            assert run.lib.aet_test_one_xcd_clients() == (0 if mode or variants else run.n)
            run.close()
        finally:
            lib.aet_test_select_kernels(0, 0)
            lib.aet_test_variants(0)
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


@pytest.mark.parametrize("n,hw,width,batch,launches", [
    (8, 16, 16, 32, 1), (9, 16, 16, 32, 0), (12, 16, 16, 32, 2), (33, 16, 16, 16, 0), (16, 16, 16, 17, 0),
    (5, 16, 16, 64, 0), (6, 16, 16, 64, 1), (2, 12, 16, 64, 1), (8, 16, 16, 64, 1), (9, 12, 6, 64, 0), (2, 16, 32, 16, 0),
])
def test_where_it_is_the_faster_engine(n, hw, width, batch, launches):
    from paper_2112_13935_amd.runner import Run
    assert _launches(Run(_cnn(n, hw, width, 16, batch, 1))) == launches


@pytest.mark.parametrize("n,channels,units,batch,launches", [
    (1, 8, 384, 1, 1), (1, 8, 400, 1, 0), (8, 16, 196, 32, 1), (8, 16, 256, 32, 0), (1, 64, 48, 8, 1), (1, 64, 1024, 8, 0),
    (4, 8, 120, 64, 1), (4, 8, 192, 64, 0),
])
def test_wide_dense_layers_keep_the_layer_engine(n, channels, units, batch, launches):
    """One convolution on 8 x 8 maps: every workgroup goes through the hidden layer's weights twice per sample."""
    from paper_2112_13935_amd.runner import Run
    assert _launches(Run(_net(n, batch, (3, 8, 8), [_conv(channels), _dense(units)], 1))) == launches


@pytest.mark.parametrize("width,launches", [(16, 2), (32, 0)])
def test_lone_workgroups_with_many_parameters_keep_the_layer_engine(width, launches):
    """More clients than compute units, mini-batch 1: one workgroup makes a client's whole update."""
    from paper_2112_13935_amd.runner import Run
    assert _launches(Run(_cnn(257, 8, width, 64, 1, 1))) == launches


def test_layer_engine_where_the_fused_round_took_over(oracle_libs):
    """A shape whose split convolutions end inside their tiles, which without asking runs fused."""
    from oracle import Oracle
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = W.config4(n_clients=8, n_per=70, hw=16, width=16, fc=16, batch=50, rounds=2, a=0, b=50)
    load_library().aet_test_select_kernels(1, 0)
    try:
        run = Run(wl)
    finally:
        load_library().aet_test_select_kernels(0, 0)
    lockstep(wl, run, Oracle(wl, "f64"))
    run.close()


@pytest.mark.parametrize("biases", [
    [-3.2e38] * 10,                              # every logit below -3e38: ten equal ones
    [-np.inf] + [0.0] * 9,                       # a class that is ruled out
    [-np.inf] * 4 + [-3.3e38] * 5 + [-np.inf],   # and no other one near zero
], ids=["lowest", "ruled_out", "both"])
def test_logits_near_the_lowest_value(biases):
    """Logits that are finite, or -inf for some classes, have a softmax: U is what the layer engine gives, and
    finite.  (The labels are classes of finite logits.)"""
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.runner import Run
    out = []
    for layers in (1, 0):
        wl = _cnn(2, 8, 5, 12, 4, rounds=1)
        wl.w0[-10:] = biases
        real = np.flatnonzero(np.isfinite(biases))
        wl.y = [real[y % real.size].astype(np.int32) for y in wl.y]
        load_library().aet_test_select_kernels(layers, 0)
        try:
            run = Run(wl)
        finally:
            load_library().aet_test_select_kernels(0, 0)
        run.run_round()
        out.append(np.stack([run.lib.aet_get_U(c, 0) for c in range(wl.n_clients)]).astype(np.float64))
        run.close()
    assert np.isfinite(out[0]).all() and np.isfinite(out[1]).all()
    # (sums in another order, as below)
    assert np.linalg.norm(out[1] - out[0]) <= 1e-5 * np.linalg.norm(out[0])


def test_small_workspace_takes_the_layer_engine(monkeypatch):
    """Its images and records are an option: without room for them the call is still accepted."""
    import re
    from paper_2112_13935_amd.binding import AetError
    from paper_2112_13935_amd.runner import Run
    make = CASES["12x12_odd"]
    run = Run(make())
    lib = run.lib.lib
    run.run_all()
    fused = run.lib.aet_get_weights(-1)
    run.close()
    size = [256]
    with monkeypatch.context() as m:
        m.setattr(lib, "aet_workspace_bytes", lambda *a: size[0])
        with pytest.raises(AetError) as err:
            Run(make())
        size[0] = int(re.search(r"(\d+) needed", str(err.value)).group(1))
        assert _launches(Run(make())) == 0
        run = Run(make())
    run.run_all()
    layers = run.lib.aet_get_weights(-1)
    run.close()
    # (sums in another order: 2e-7 seen)
    assert np.linalg.norm(fused - layers) <= 1e-5 * np.linalg.norm(layers)
