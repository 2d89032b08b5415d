"""Cluster launches of several contexts on one GPU (csrc/cluster_turns.h): never two in flight on
different streams, and no event where a context is alone or the others are idle.  The header is
plain host code; a C++ program drives it with streams that only keep what they are ordered
behind."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "cluster_turns.h"
#include <cstdio>
#include <map>
#include <random>
#include <set>
#include <thread>
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (line %d)\n", #x, __LINE__); return 1; } } while (0)
using Turns = aet::ClusterTurns<int>;
int main() {
    // streams as sets of launches that are done before the next one starts
    std::map<int, std::set<int>> behind;   // stream -> launches it is ordered behind
    std::vector<int> all;
    int events = 0, launches = 0;
    Turns turns;
    Turns::Member m[4];
    const int stream[4] = {10, 20, 30, 20};   // the last shares a stream with the second
    for (int i = 0; i < 4; ++i) { m[i].stream = stream[i]; turns.join(&m[i]); }
    bool bad = false;
    auto go = [&](int i) {
        return turns.take(&m[i],
            [&](Turns::Member *o) {
                ++events;
                auto &v = behind[m[i].stream];
                const auto theirs = behind[o->stream];
                v.insert(theirs.begin(), theirs.end());
                return 0;
            },
            [&] {
                auto &v = behind[m[i].stream];
                for (int l : all) bad = bad || !v.count(l);
                v.insert(launches);
                all.push_back(launches++);
                return 0;
            });
    };
    for (int k = 0; k < 50; ++k) CHECK(go(0) == 0);
    CHECK(!bad && events == 0);              // alone: nothing to order
    CHECK(go(1) == 0 && events == 1);        // behind the first context's launches
    for (int k = 0; k < 50; ++k) CHECK(go(1) == 0);
    CHECK(!bad && events == 1);              // the first is idle since
    CHECK(go(3) == 0 && !bad);               // the same stream as the second
    std::mt19937 rng(3);
    for (int k = 0; k < 400; ++k) CHECK(go((int)(rng() % 4)) == 0);
    CHECK(!bad);
    turns.leave(&m[0]);
    const int before = events;
    for (int k = 0; k < 3; ++k) CHECK(go(2) == 0);
    CHECK(events <= before + 2 && !bad);
    // a failed order is handed on and nothing is launched
    const int n = launches;
    go(1);
    CHECK(turns.take(&m[2], [&](Turns::Member *) { return 7; }, [&] { ++launches; return 0; }) == 7);
    CHECK(launches == n + 1);
    // threads: launches never overlap
    Turns shared;
    Turns::Member t[6];
    int inside = 0, most = 0;
    std::vector<std::thread> th;
    for (int i = 0; i < 6; ++i) { t[i].stream = i; shared.join(&t[i]); }
    for (int i = 0; i < 6; ++i)
        th.emplace_back([&, i] {
            for (int k = 0; k < 500; ++k)
                shared.take(&t[i], [](Turns::Member *) { return 0; }, [&] { most = std::max(most, ++inside); --inside; return 0; });
        });
    for (auto &x : th) x.join();
    CHECK(most == 1);
    std::puts("ok");
}
"""


def test_cluster_launches_are_ordered_across_streams(tmp_path):
    src, exe = str(tmp_path / "p.cpp"), str(tmp_path / "p")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=thread", "-I",
                    os.path.join(ROOT, "paper_2112_13935_amd", "csrc"), "-o", exe, src], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr[-2000:]


def test_every_cluster_launch_takes_its_turn():
    text = open(os.path.join(ROOT, "paper_2112_13935_amd", "csrc", "aet_api.hip")).read()
    for launch in ("launch_mlp_round(", "launch_softmax_batch_round(", "launch_lenet_round("):
        at = text.index(launch)
        assert "ctx->clustered([&] {" in text[at - 120:at], launch
