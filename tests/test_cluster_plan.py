"""Clusters per launch (csrc/cluster_plan.h): every workgroup of a launch has a place on its own
XCD, and no two clients' records share a line of memory.  The header is plain host code; a small C++ program prints its answers and the launch is
laid out here the way the round kernels number their workgroups."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_13935_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = str(d / "plan.cpp"), str(d / "plan")
    with open(src, "w") as f:
        f.write('#include "cluster_plan.h"\n#include <cstdio>\nint main() {\n'
                "    int c, x, s;\n"
                '    while (scanf("%d %d %d", &c, &x, &s) == 3)\n'
                '        if (c < -1) printf("%u\\n", c == -2 ? aet::cluster_steps(x, s) : (uint32_t)aet::tags_spent((uint32_t)x, (uint32_t)s));\n'
                '        else printf("%d\\n", c > 0 ? aet::resident_clusters(c, x, s) : c == 0 ? aet::softmax_batch_record_words(x, s)\n'
                '                                                                : aet::kWaitPolls);\n}\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", exe, src], check=True)

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]
    return ask


def most_on_one_xcd(clients, size, xcds):
    """Working workgroups per XCD: workgroup id -> (client, member) as the kernels do it."""
    on = [0] * xcds
    for block in range(8 * ((clients + 7) // 8) * size):
        client = (block & 7) + 8 * ((block >> 3) // size)
        if client < clients:
            on[block % xcds] += 1
    return max(on)


@pytest.mark.parametrize("cus,xcds", [(256, 8), (512, 8), (128, 4), (64, 2), (32, 1)])
def test_every_workgroup_of_a_launch_has_a_place(plan, cus, xcds):
    sizes = list(range(1, 33))
    for size, n in zip(sizes, plan([(cus, xcds, s) for s in sizes])):
        assert n >= xcds, f"clusters of {size} fit every XCD"
        for clients in {1, 7, 8, 9, n - 1, n} - {0}:
            if clients <= n:
                assert most_on_one_xcd(clients, size, xcds) <= cus // xcds, (size, clients)
        # and no smaller than it has to be: eight clients more overfill some XCD
        assert most_on_one_xcd(n + 8, size, xcds) > cus // xcds, size


def test_a_cluster_larger_than_an_xcd_has_no_place(plan):
    assert plan([(256, 8, 33)]) == [0]


def test_no_two_clients_share_a_line(plan):
    """A line is 16 words; a client's records are two sets of 12 words per sample and workgroup."""
    rows = [(0, hf, b) for hf in range(1, 7) for b in range(2, 65)]
    for (_, hf, b), words in zip(rows, plan(rows)):
        assert words % 16 == 0
        assert words == 0 if hf == 1 else 24 * hf * b <= words < 24 * hf * b + 16


def test_records_of_mini_batch_softmax_are_laid_out_so():
    """Workspace of n clients whose records are 3 * 5 * 24 = 360 words without the rounding, 368 with it: beside
    them a client has its model, its displacement, the layers' values and its place in the lists."""
    import ctypes
    import workloads as W
    from paper_2112_13935_amd.binding import load_library, model_desc
    lib = load_library()
    sizes = [lib.aet_workspace_bytes(ctypes.byref(model_desc(W.softmax_model(1100, 10, b))), 512, 1, 1) for b in (5, 6)]
    # per sample of 512 clients: input row, logits and their gradient, label, and the records' share
    rest = 512 * (4 * (1100 + 10 + 10) + 4)
    assert sizes[1] - sizes[0] == rest + 512 * 8 * (432 - 368)


def test_a_wait_is_no_shorter_where_polls_are_cheap(plan):
    """2^22 polls through memory took 2.2 s; a poll of the XCD's L2 takes 0.26 us (half a round trip of 1,125
    shader clocks at 2.1 GHz)."""
    assert plan([(-1, 0, 0)])[0] * 0.26e-6 >= 2.15


@pytest.mark.parametrize("kernel", ["softmax_batch", "mlp", "lenet", "cnn"])
def test_every_poll_of_a_peer_is_bounded_so(kernel):
    text = open(os.path.join(CSRC, f"kernels_{kernel}.hip")).read()
    assert "gave_up(" in text and "spins" not in text


@pytest.mark.parametrize("kernel", ["softmax_batch", "mlp", "lenet", "cnn"])
def test_the_launchers_take_their_clusters_from_the_plan(kernel):
    text = open(os.path.join(CSRC, f"kernels_{kernel}.hip")).read()
    assert "per_launch" in text and "resident_clusters(" in text


def test_steps_and_tags_of_the_longest_round(plan):
    """A round may have 2^31 - 1 recursions.  With two steps each their number, and the tags they take, just fit 32 bits
    without a sign; tags run from the next one to 2^32 - 1."""
    m = 2 ** 31 - 1
    assert plan([(-2, m, 1), (-2, m, 2), (-2, 2 ** 30, 2), (-2, 0, 2)]) == [m, 2 * m, 2 ** 31, 0]

    def signed(v):
        return v - 2 ** 32 if v >= 2 ** 31 else v
    for need in (1, 2, 7, m + 1, 2 * m + 1):
        nexts = {0, 1, 2, 3, m, 2 ** 32 - need - 1, 2 ** 32 - need, 2 ** 32 - need + 1, 2 ** 32 - 1}
        for nxt in (x for x in nexts if 0 <= x < 2 ** 32):
            fits = nxt > 0 and nxt + need - 1 <= 2 ** 32 - 1
            assert plan([(-3, signed(nxt), signed(need))]) == [0 if fits else 1], (nxt, need)


def test_the_mlp_round_counts_its_steps_so():
    text = open(os.path.join(CSRC, "kernels_mlp.hip")).read()
    assert text.count("cluster_steps(") == 2 and "tags_spent(" in text and "SUB * p.m" not in text
