"""Convolutions whose fp32 values are split in three bf16 parts: parity with the CPU oracle where the
tiling can go wrong, precision against 64 bits, values that are not finite.  Run with  -m gpu  on
an MI355X."""
import re

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def layer_engine():
    """These are kernels of the layer engine; some of the models run in one launch per round by default."""
    from paper_2112_13935_amd import load_library
    load_library().aet_test_select_kernels(1, 0)
    yield
    load_library().aet_test_select_kernels(0, 0)


def _conv(cout):
    return W.Layer(W.CONV, cout, 3, 1, 1)


def _maps(n, batch, shape, layers, rounds=2):
    """A model on maps of the given (channels, rows, columns)."""
    wl = W.config4(n_clients=n, n_per=70, hw=8, width=4, fc=8, batch=batch, rounds=rounds, a=0, b=batch)
    wl.model = W.Model(*shape, layers + [W.Layer(W.DENSE, 10)], batch)
    wl.X = [W._rng(3, c).standard_normal((70, wl.model.in_size()), dtype=np.float32) for c in range(n)]
    wl.w0 = W.init_weights(wl.model, 5)
    return wl


# enough samples that each launch has the workgroups' worth of tiles from which this form is taken
CASES = {
    # 32 x 32 (pooled), 16 x 16 (both, pooled), two channel blocks
    "cnn32": lambda: W.config4(n_clients=4, n_per=70, batch=50, fc=16, rounds=1, a=0, b=50),
    # 8 x 8: four samples per workgroup, the last with two; 16 source channels: one chunk
    "cnn16_b50": lambda: W.config4(n_clients=8, n_per=70, hw=16, width=16, fc=16, batch=50, rounds=2, a=0, b=50),
    # 48 channels: a block of destination channels half full, three chunks
    "cnn16_48": lambda: W.config4(n_clients=5, n_per=70, hw=16, width=24, fc=16, batch=41, rounds=2, a=0, b=41),
    # 12 x 32: the second row block half empty; not pooled; the first layer has no backward-data
    "rows_12_of_32": lambda: _maps(3, 48, (16, 12, 32), [_conv(32), _conv(32), W.Layer(W.POOL)]),
    # 6 x 16: fewer rows than a workgroup has
    "rows_6_of_16": lambda: _maps(4, 60, (32, 6, 16), [_conv(32), _conv(32)]),
    # 16 x 8 and few pixels: only backward-weight takes this form, one and three samples a client
    "rows_16_of_8": lambda: _maps(4, 60, (32, 16, 8), [_conv(64), _conv(48), W.Layer(W.POOL)]),
    "one_sample": lambda: _maps(2, 1, (32, 8, 8), [_conv(64), _conv(64)]),
    "three_samples": lambda: _maps(1, 3, (48, 16, 16), [_conv(64), _conv(64)]),
    # 10 x 8: rows of 8 that are no square map
    "rows_10_of_8": lambda: _maps(4, 60, (16, 10, 8), [_conv(32), _conv(48), W.Layer(W.POOL)]),
}


def _on_the_fp32_unit(make):
    """A context none of whose convolutions, in either direction or for the weights, takes this form."""
    from paper_2112_13935_amd import load_library
    from paper_2112_13935_amd.runner import Run
    lib = load_library()
    lib.aet_test_variants(2)
    try:
        return Run(make())
    finally:
        lib.aet_test_variants(0)


def _smallest_workspace(monkeypatch, make):
    """A context without room for what is optional: forward and backward-data stay on the fp32 unit."""
    from paper_2112_13935_amd.binding import AetError
    from paper_2112_13935_amd.runner import Run
    run = Run(make())
    lib = run.lib.lib
    run.close()
    size = [256]
    with monkeypatch.context() as m:
        m.setattr(lib, "aet_workspace_bytes", lambda *a: size[0])
        with pytest.raises(AetError) as err:
            Run(make())
        size[0] = int(re.search(r"(\d+) needed", str(err.value)).group(1))
        return Run(make())


@pytest.mark.parametrize("name", sorted(CASES))
def test_parity(oracle_libs, name):
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    from parity import lockstep
    wl = CASES[name]()
    run, orc = Run(wl), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


def test_parity_in_the_smallest_workspace(oracle_libs, monkeypatch):
    from oracle import Oracle
    from parity import lockstep
    wl = CASES["cnn32"]()
    run, orc = _smallest_workspace(monkeypatch, CASES["cnn32"]), Oracle(wl, "f64")
    lockstep(wl, run, orc)
    run.close()


@pytest.mark.parametrize("n,batch,shape", [(2, 50, (16, 32, 32)), (4, 50, (32, 16, 16)), (8, 50, (64, 8, 8))])
@pytest.mark.parametrize("layers", [1, 2])
def test_no_further_from_64_bits_than_the_fp32_unit(oracle_libs, n, batch, shape, layers):
    """U of one recursion of convolutions without ReLU or pooling (no decisions that rounding could
    turn): the split products round less often (see split_bf16.h), so the error of each convolution's
    weights is the smaller one.  With one convolution its weights' gradient is a backward-weight product
    of the input rows themselves, with two the first one's went through backward-data as well."""
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run

    def make():
        return _maps(n, batch, shape, [W.Layer(W.CONV, 32 * (i + 1), 3, 1, 0) for i in range(layers)], rounds=1)
    orc = Oracle(make(), "f64")
    orc.run_round()
    us = []
    for run in (Run(make()), _on_the_fp32_unit(make)):
        run.run_round()
        us.append([run.lib.aet_get_U(c, 0).astype(np.float64) for c in range(orc.n)])
        run.close()
    ref = [orc.get_U(c, 0) for c in range(orc.n)]
    for l, s in enumerate(run.wl.model.param_slices()):
        at = slice(s[0], s[0] + s[1])
        err = [np.sqrt(sum(((x[at] - r[at]) ** 2).sum() for x, r in zip(u, ref)) / sum((r[at] ** 2).sum() for r in ref)) for u in us]
        print(f"{shape}, layer {l} of {layers + 1}: split {err[0]:.2e}, fp32 unit {err[1]:.2e}")
        if l < layers:
            assert err[0] < err[1], l


def test_infinities_stay_where_they_were():
    """One infinite pixel in one client's rows: the same entries of its model are finite, infinite and
    NaN as with the products on the fp32 unit."""
    from paper_2112_13935_amd.runner import Run

    def make():
        wl = CASES["cnn32"]()
        wl.X[1] = wl.X[1].copy()
        wl.X[1][:, 700] = np.inf
        return wl
    out = []
    for run in (Run(make()), _on_the_fp32_unit(make)):
        run.run_round()
        out.append(np.stack([run.lib.aet_get_U(c, 0) for c in range(run.n)]))
        run.close()
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(out[0]), kind(out[1]))
    assert np.isfinite(out[0][0]).all() and not np.isfinite(out[0][1]).all()


def _one_layer(scale_w, scale_dense):
    """One convolution without ReLU; its weights and the dense layer's scaled."""
    wl = _maps(4, 50, (16, 16, 16), [W.Layer(W.CONV, 32, 3, 1, 0)], rounds=1)
    s = wl.model.param_slices()
    wl.w0[s[0][0]:s[0][0] + s[0][1]] *= np.float32(scale_w)
    wl.w0[s[1][0]:s[1][0] + s[1][1]] *= np.float32(scale_dense)
    return wl


def _largest_pixel():
    """Rows with a pixel near the largest fp32 value: its outputs are about 1e7, its gradients 1e29."""
    wl = _one_layer(1e-30, 1e-7)
    for x in wl.X:
        x[:, 700] = 3.4e38
    return wl


def _largest_weight():
    wl = _one_layer(1.0, 1e-9)
    for x in wl.X:
        x *= np.float32(1e-30)
    wl.w0[1234] = -3.4e38
    return wl


@pytest.mark.parametrize("make", [_largest_pixel, _largest_weight])
def test_largest_finite_values(oracle_libs, make):
    """Finite values beyond the largest finite bf16 value (3.390e38) keep their finite products.  Bound:
    rounding of fp32 sums, 1e-5 of the tensor's norm; tensors that are below fp32's normal range (the
    weights' gradient where the weight is the large factor) are not compared."""
    from oracle import Oracle
    from paper_2112_13935_amd.runner import Run
    wl = make()
    run, orc = Run(wl), Oracle(make(), "f64")
    orc.run_round()
    run.run_round()
    for c in range(run.n):
        got, want = run.lib.aet_get_U(c, 0).astype(np.float64), orc.get_U(c, 0)
        compared = 0
        for s in [x for x in wl.model.param_slices() if x is not None]:
            for at, n in ((s[0], s[1]), (s[2], s[3])):
                g, w = got[at:at + n], want[at:at + n]
                if np.abs(w).max() < 1e-30:
                    continue
                assert np.linalg.norm(g - w) <= 1e-5 * np.linalg.norm(w), (c, at, np.isfinite(g).all())
                compared += 1
        assert compared >= 2
    run.close()


def test_splitting_of_the_weights_is_timed():
    """Once a recursion for all layers, in the family of the forward convolutions."""
    from paper_2112_13935_amd.runner import Run
    launches = []
    for run in (Run(CASES["cnn32"]()), _on_the_fp32_unit(CASES["cnn32"])):
        fam = run.lib.profile_family_names().index("k_conv_fwd")
        run.lib.aet_profile_enable(fam, True)
        run.run_round()
        launches.append(run.lib.aet_profile_read(fam)[0])
        run.close()
    assert launches == [5, 4]   # one recursion, four convolutions
