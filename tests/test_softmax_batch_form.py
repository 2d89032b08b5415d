"""Which form of the mini-batch softmax kernels a round takes (csrc/softmax_batch_form.h): every form that the rule
names has its kernel, every kernel that is built is named by it, and the GPU tests' cases run the forms that
they say, each of them.  The header is plain host code; a C++ program prints its answers."""
import os
import re
import subprocess

import pytest

from test_gpu_softmax_tiles import CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_13935_amd", "csrc")
PROGRAM = r"""
#include "softmax_batch_form.h"
#include <cstdio>
#include <set>
#include <string>
static std::string form(int n, int D, int B, bool *fits) {
    const auto f = aet::softmax_batch_form(D, B, n, 256, 8);
    // the exchange records are made for a run of columns per workgroup
    *fits = f.workgroups * f.runs * aet::kSbRun >= D && f.workgroups <= (D + aet::kSbRun - 1) / aet::kSbRun && f.samples >= B;
    return std::string(f.lanes ? "lanes " : "tiles ") + std::to_string(f.runs) + "x" + std::to_string(f.samples) +
           (f.lanes ? "" : f.columns == 0 ? " full" : f.columns == 1 ? " any" : " tiny");
}
int main() {
    bool fits = true, all = true;
    int n, d, b;
    while (std::scanf("%d %d %d", &n, &d, &b) == 3) std::printf("%s\n", form(n, d, b, &fits).c_str());
    std::set<std::string> seen;
    for (int D = 1; D <= 3072; ++D)
        for (int B = 2; B <= 64; ++B)
            for (int c : {1, 8, 16, 40, 41, 64, 65, 96, 128, 129, 192, 256, 257, 400, 1024}) {
                seen.insert(form(c, D, B, &fits));
                all = all && fits;
            }
    std::printf("%s\n", all ? "fit" : "do not fit");
    for (const auto &s : seen) std::printf("%s\n", s.c_str());
}
"""


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    d = tmp_path_factory.mktemp("form")
    src, exe = str(d / "form.cpp"), str(d / "form")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, src], check=True)
    text = "\n".join(f"{n} {d} {b}" for n, d, b, _ in CASES)
    lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    return lines[:len(CASES)], lines[len(CASES)], set(lines[len(CASES) + 1:])


def test_cases_run_the_forms_that_they_say(answers):
    for case, got in zip(CASES, answers[0]):
        assert case[3] == got, case


def test_every_form_has_a_case(answers):
    assert answers[1] == "fit"
    assert {form for *_, form in CASES} == answers[2]


def test_every_form_has_its_kernel_and_no_other_is_built(answers):
    text = open(os.path.join(CSRC, "kernels_softmax_batch.hip")).read()
    launch = text[text.index("hipError_t launch_softmax_batch_round("):]
    built = {f"lanes {r}x{s}" for r, s in re.findall(r"k_softmax_batch_lanes<(\d), (\d+)>", launch)}
    for samples, runs, one in re.findall(r"case (\d+) \+ (\d): AET_SB(_ONE)?\(", launch):
        built |= {f"tiles {runs}x{samples} {c}" for c in ("full", "any", "tiny") if one or c != "tiny"}
    assert built == answers[2]
