"""Polls of exchange words (ClusterWords in csrc/cluster_post.h) stay where they are written.  The words are plain loads to
the compiler, of memory that other workgroups change; a kernel that looks at a word twice has to load it twice, also
where the words came in as a __restrict__ argument, and a poll loop has to hold its load.  Shown on the assembly of small kernels, compiled
here for the GPU and not run."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_13935_amd", "csrc")

KERNELS = r"""
#include "cluster_post.h"
using aet::ClusterWords;
typedef unsigned long long u64;
extern "C" __global__ void twice(u64 *QUAL words, int *QUAL out) {
    const ClusterWords w(words, 64 * blockIdx.x, 64);
    ClusterWords::look_again();
    const auto a = w.get(8 * (int)threadIdx.x, 0);
    ClusterWords::look_again();
    const auto b = w.get(8 * (int)threadIdx.x, 0);
    out[threadIdx.x] = (a[0] ^ b[0]) | (a[1] ^ b[1]);
}
extern "C" __global__ void poll(u64 *QUAL words, int *QUAL out, int tag) {
    const ClusterWords w(words, 0, 64);
    ClusterWords::look_again();
    auto v = w.get(0, 0);
    while (v[1] != tag) {
        __builtin_amdgcn_s_sleep(1);
        ClusterWords::look_again();
        v = w.get(0, 0);
    }
    out[0] = v[0];
}
"""


@pytest.fixture(scope="module", params=["", "__restrict__"])
def bodies(request, tmp_path_factory):
    from paper_2112_13935_amd import build
    d = tmp_path_factory.mktemp("words")
    src, out = str(d / "words.hip"), str(d / "words.s")
    with open(src, "w") as f:
        f.write(KERNELS)
    flags = [x for x in build.HIPCC_FLAGS if x not in ("-shared", "-Wall")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-DQUAL=" + request.param, "-I", CSRC, "--offload-device-only", "-S", "-o", out, src], check=True)
    text = open(out).read()
    return {k: text[text.index(f"\n{k}:"):text.index("s_endpgm", text.index(f"\n{k}:"))] for k in ("twice", "poll")}


def test_two_looks_are_two_loads(bodies):
    assert len(re.findall(r"buffer_load_dwordx2", bodies["twice"])) == 2


def test_a_poll_loop_holds_its_load(bodies):
    lines = bodies["poll"].splitlines()
    at = {m.group(1): i for i, s in enumerate(lines) if (m := re.match(r"(\.\w+):", s))}
    loops = [lines[at[m.group(1)]:i] for i, s in enumerate(lines)
             if (m := re.search(r"s_c?branch\w* (\.\w+)", s)) and at.get(m.group(1), i) < i]
    assert loops
    assert all(any("buffer_load" in s for s in loop) for loop in loops)
