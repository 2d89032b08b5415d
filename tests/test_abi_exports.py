"""The C-ABI library loads without a GPU and exports every function include/aet_sgd.h
declares.  No compute call is made here."""
import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "aet_sgd.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(aet_[a-zA-Z0-9_]+)\s*\(", text)))


def test_header_declares_the_three_named_calls():
    names = declared_functions()
    for must in ("aet_init", "aet_run_round", "aet_server_aggregate"):
        assert must in names


def test_library_exports_every_declared_symbol():
    from paper_2112_13935_amd import build
    from paper_2112_13935_amd.binding import EXPORTS
    if build.needs_build():
        build.build(force=True)
    lib = ctypes.CDLL(build.LIB)
    names = declared_functions()
    assert names, "no declarations found"
    for name in names:
        assert hasattr(lib, name), f"{name} is declared but not exported"
    assert sorted(EXPORTS) == names, "binding and header disagree on the entry points"


def test_model_validation_runs_on_the_host():
    """aet_n_params / aet_workspace_bytes are pure host arithmetic."""
    import workloads as W
    from paper_2112_13935_amd.binding import load_library, model_desc
    lib = load_library()
    for model, want in ((W.softmax_model(784, 10), 7850), (W.mlp_model(784, 128, 10, 32), 101770),
                        (W.lenet_model(16), 44426), (W.cnn32_model(64), 1116970),
                        (W.softmax_model(3072, 10), 30730)):
        d = model_desc(model)
        assert lib.aet_n_params(ctypes.byref(d)) == want
        assert lib.aet_workspace_bytes(ctypes.byref(d), 4, 2, 10) > 4 * want * 4
    bad = model_desc(W.Model(1, 7, 7, [W.Layer(W.CONV, 2, 3, 0, 1), W.Layer(W.POOL), W.Layer(W.DENSE, 3)], 2))
    assert lib.aet_n_params(ctypes.byref(bad)) == -1          # 5x5 map cannot be pooled 2x2
    assert lib.aet_workspace_bytes(ctypes.byref(bad), 4, 1, 1) == 0
    ok = model_desc(W.softmax_model(8, 3))
    assert lib.aet_workspace_bytes(ctypes.byref(ok), 0, 1, 1) == 0


def test_room_for_split_weights_only_where_they_are_used():
    """The workspace of a model with convolutions, with and without the form that wants its weights as bf16
    parts (27,648 bytes for 16 source and 32 destination channels and a client)."""
    import workloads as W
    from paper_2112_13935_amd.binding import load_library, model_desc
    lib = load_library()

    def room(model, clients, plain=0):
        sizes = []
        for variant in (0, 2):
            lib.aet_test_select_kernels(1, plain)   # the layer engine, also for the models that do not run on it by default
            lib.aet_test_variants(variant)
            try:
                sizes.append(lib.aet_workspace_bytes(ctypes.byref(model_desc(model)), clients, 1, 10))
            finally:
                lib.aet_test_select_kernels(0, 0)
                lib.aet_test_variants(0)
        return sizes[0] - sizes[1]

    # forward and backward-data of 32 -> 32, 32 -> 64 and 64 -> 64 channels (the first layer has three)
    assert room(W.cnn32_model(64), 32) == 32 * 27648 * (2 + 2 + 4 + 4 + 8 + 8)
    assert room(W.cnn32_model(64), 32, plain=1) == 0
    # backward-data of 16 -> 32 channels has 16 destination channels, 16 -> 16 both ways: not used
    assert room(W.cnn32_model(64, hw=16, width=16), 32) == 32 * 27648 * (1 + 2 + 2)
    # too few tiles with every client at work
    assert room(W.cnn32_model(16, hw=16, width=16, fc=64), 6) == 0


def test_header_names_the_batches_that_run_in_clusters():
    """Callers of a model that runs in clusters have to know it: a precondition comes with it, and records in the workspace."""
    import workloads as W
    from paper_2112_13935_amd.binding import load_library, model_desc
    lib = load_library()
    text = re.sub(r"\n \* +", " ", open(os.path.join(ROOT, "include", "aet_sgd.h")).read())
    dense = int(re.search(r"dense-ReLU-dense models \(batch up to (\d+),", text).group(1))
    lenet = int(re.search(r"LeNet-5-style models \([^)]*batch up to (\d+)\)", text).group(1))

    def records(model):
        sizes = []
        for layers in (0, 1):
            lib.aet_test_select_kernels(layers, 0)
            try:
                sizes.append(lib.aet_workspace_bytes(ctypes.byref(model_desc(model)), 3, 1, 1))
            finally:
                lib.aet_test_select_kernels(0, 0)
        return sizes[0] > sizes[1]
    assert records(W.mlp_model(50, 20, 10, dense)) and not records(W.mlp_model(50, 20, 10, dense + 1))
    assert records(W.lenet_model(lenet, 16)) and not records(W.lenet_model(lenet + 1, 16))
