"""Cluster launches of several contexts on one GPU (csrc/cluster_turns.h): never two in flight on
different streams, or as many as the compute units hold where a launch says what it needs, and no event where a context
is alone or the others are idle.  The header is
plain host code; a C++ program drives it with streams that only keep what they are ordered
behind."""
import os
import subprocess

import pytest

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


# Contexts whose launches may go beside others.  A stream is a row of launches; each knows those that are done before it
# starts, and the GPU gets on at random.
SHARED = r"""
#include "cluster_turns.h"
#include <cstdio>
#include <map>
#include <random>
#include <set>
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (line %d)\n", #x, __LINE__); return 1; } } while (0)
using Turns = aet::ClusterTurns<int>;
constexpr int kCus = 32;
using Held = Turns::Held;
struct Launch { int stream; Held held; };
struct Gpu {
    std::vector<Launch> all;
    std::map<int, std::vector<int>> row;        // stream -> its launches
    std::map<int, std::set<int>> behind;        // stream -> launches its next one is ordered behind
    std::set<int> done;
    std::map<Turns::Member *, size_t> mark;     // launches of the stream ahead of the latest mark
    bool finish(int l) {                        // if all before it are done
        for (int k : row[all[l].stream]) if (k < l && !done.count(k)) return false;
        return done.insert(l).second;
    }
};
int main() {
    int beside = 0;
    for (int seed = 1; seed <= 80; ++seed) {
        std::mt19937 rng(seed);
        Turns turns;
        Gpu gpu;
        const int N = 2 + (int)(rng() % 5);
        std::vector<Turns::Member> m(N);
        std::vector<Turns::Need> need(N);
        for (int i = 0; i < N; ++i) {
            m[i].stream = (int)(rng() % 5);
            if (rng() % 4) {
                need[i].cus = kCus;
                need[i].clients = 1 + (int)(rng() % (seed % 3 ? 8 : 30));
                need[i].least = 1 + (int)(rng() % (seed % 2 ? 16 : 4));
                need[i].most = std::max(need[i].least, kCus / ((need[i].clients + 7) / 8) - (int)(rng() % 4));
            }
            turns.join(&m[i]);
        }
        bool bad = false;
        for (int step = 0; step < 300; ++step) {
            if (!gpu.all.empty()) for (int k = (int)(rng() % (1 + seed % 4)); k > 0; --k) gpu.finish((int)(rng() % gpu.all.size()));
            if (rng() % 40 == 0 && seed % 4) for (size_t l = 0; l < gpu.all.size(); ++l) gpu.finish((int)l);
            const int i = (int)(rng() % N), s = m[i].stream, there = (need[i].clients + 7) / 8;
            const bool whole = need[i].cus == 0 || there * need[i].least > kCus;
            turns.take(&m[i], need[i],
                [&](Turns::Member *o) { for (int l : gpu.row[o->stream]) if (!gpu.done.count(l)) return false; return true; },
                [&](Turns::Member *o) { gpu.mark[o] = gpu.row[o->stream].size(); return 0; },
                [&](Turns::Member *o) {
                    const auto &r = gpu.row[o->stream];
                    for (size_t k = 0; k < gpu.mark[o]; ++k) if (!gpu.done.count(r[k])) return false;
                    return true;
                },
                [&](Turns::Member *o) {
                    auto &b = gpu.behind[s];
                    b.insert(gpu.row[o->stream].begin(), gpu.row[o->stream].end());
                    const auto theirs = gpu.behind[o->stream];
                    b.insert(theirs.begin(), theirs.end());
                    return 0;
                },
                [&](const Turns::Place &p) {
                    Held held{};
                    if (whole) held.fill(kCus);
                    else if (p.first < 0) held.fill(std::min(kCus, there * p.size));   // wherever it begins
                    else for (int c = 0; c < need[i].clients; ++c) held[(p.first + c) % 8] += p.size;
                    if (!whole) bad = bad || p.size < need[i].least || p.size > need[i].most || p.first > 7;
                    // the most that other streams may have running beside it
                    Held sum{};
                    for (const auto &r : gpu.row) {
                        Held most{};
                        if (r.first != s)
                            for (int l : r.second) if (!gpu.done.count(l) && !gpu.behind[s].count(l))
                                for (int x = 0; x < 8; ++x) most[x] = std::max(most[x], gpu.all[l].held[x]);
                        for (int x = 0; x < 8; ++x) sum[x] += most[x];
                    }
                    bool any = false;
                    for (int x = 0; x < 8; ++x) {
                        bad = bad || (sum[x] && held[x] && sum[x] + held[x] > kCus);
                        any = any || sum[x];
                    }
                    beside += any;
                    gpu.row[s].push_back((int)gpu.all.size());
                    gpu.all.push_back({s, held});
                    return 0;
                });
            CHECK(!bad);
            for (auto &x : m) CHECK(x.runs.size() <= 4);
        }
        turns.leave(&m[0]);
        for (int i = 1; i < N; ++i) for (auto &o : m[i].orders) CHECK(o.of != &m[0]);
    }
    CHECK(beside > 1000);
    std::vector<Turns::Place> places;
    int events = 0;
    bool idle_now = false;
    auto go = [&](Turns &turns, Turns::Member *me, const Turns::Need &need) {
        turns.take(me, need, [&](Turns::Member *) { return idle_now; }, [](Turns::Member *) { return 0; }, [](Turns::Member *) { return true; },
                   [&](Turns::Member *) { ++events; return 0; }, [&](const Turns::Place &p) { places.push_back(p); return 0; });
    };
    auto sizes = [&] { std::vector<int> v; for (auto &p : places) v.push_back(p.size); places.clear(); return v; };
    using V = std::vector<int>;
    {   // two on all XCDs, of 1 to 25 workgroups a cluster: the first is alone, then both have a half, without events in between
        Turns turns;
        Turns::Member a, b;
        a.stream = 1; b.stream = 2;
        turns.join(&a); turns.join(&b);
        Turns::Need need{kCus, 8, 1, 25};
        for (int k = 0; k < 4; ++k) { go(turns, &a, need); go(turns, &b, need); }
        CHECK((sizes() == V{25, 7, 16, 16, 16, 16, 16, 16}) && events == 0);
        // the other one is done: all there is again
        idle_now = true;
        for (int k = 0; k < 3; ++k) go(turns, &a, need);
        CHECK((sizes() == V{16, 25, 25}) && events == 0);
        // no room beside it: behind it, once, and so that its next launch fits
        need.least = 12;
        idle_now = false;
        for (int k = 0; k < 3; ++k) { go(turns, &b, need); go(turns, &a, need); }
        CHECK((sizes() == V{16, 16, 16, 16, 16, 16}) && events == 1);
        // what cannot share takes turns
        need.least = 20;
        for (int k = 0; k < 3; ++k) { go(turns, &b, need); go(turns, &a, need); }
        CHECK(sizes().back() == 20 && events == 7);
    }
    {   // one client each: an XCD each
        Turns turns;
        Turns::Member m[8];
        for (int i = 0; i < 8; ++i) { m[i].stream = i; turns.join(&m[i]); }
        events = 0;
        for (int k = 0; k < 3; ++k) for (auto &x : m) go(turns, &x, {kCus, 1, 32, 32});
        std::set<int> firsts;
        for (size_t k = 0; k < places.size(); ++k) {
            CHECK(places[k].size == 32 && places[k].first == places[k % 8].first);
            firsts.insert(places[k].first);
        }
        CHECK(firsts.size() == 8 && *firsts.begin() == 0 && events == 0);
    }
    {   // alone: wherever the queue begins
        Turns turns;
        Turns::Member a;
        turns.join(&a);
        places.clear();
        go(turns, &a, {kCus, 3, 5, 25});
        CHECK(places[0].first == -1 && places[0].size == 25);
    }
    std::puts("ok");
}
"""


# Contexts of dense-ReLU-dense models: clusters of one size.
DENSE = r"""
#include "cluster_plan.h"
#include "cluster_turns.h"
#include <cstdio>
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (line %d)\n", #x, __LINE__); return 1; } } while (0)
using Turns = aet::ClusterTurns<int>;
// launches of k contexts in turn, each under way while the others make theirs: how many wait for nothing once all know of each other (bad: more
// workgroups on an XCD than it holds, or another size)
int beside(int k, int groups, bool halves, int clients, bool *bad) {
    Turns turns;
    std::vector<Turns::Member> m(k);
    const int size = aet::dense_cluster_size(32, groups, halves, clients);
    Turns::Need need;
    if (size) need = {32, clients, size, size};
    int free = 0, held[8] = {};
    for (int i = 0; i < k; ++i) { m[i].stream = i; turns.join(&m[i]); }
    for (int round = 0; round < 5; ++round)
        for (int i = 0; i < k; ++i) {
            bool ordered = false;
            turns.take(&m[i], need, [](Turns::Member *) { return false; }, [](Turns::Member *) { return 0; }, [](Turns::Member *) { return true; },
                       [&](Turns::Member *) { ordered = true; return 0; },
                       [&](const Turns::Place &p) {
                           *bad = *bad || (size && p.size != size);
                           for (int x = 0; x < 8 && round == 4 && !ordered && size; ++x) {
                               for (int c = 0; c < clients; ++c) held[x] += p.first < 0 ? (c % 8 == 0) * size : ((p.first + c) % 8 == x) * size;
                               *bad = *bad || held[x] > 32;
                           }
                           return 0;
                       });
            free += round == 4 && !ordered;
        }
    return free;
}
int main() {
    bool bad = false;
    CHECK(beside(8, 1, false, 1, &bad) == 8);     // 30 -> 10
    CHECK(beside(4, 7, false, 8, &bad) == 4);     // 100 -> 100: 28 of 32 compute units
    CHECK(beside(5, 7, false, 8, &bad) < 5);
    CHECK(beside(8, 7, true, 1, &bad) == 8);      // 784 -> 100, two workgroups a unit group
    CHECK(beside(8, 16, true, 1, &bad) == 8);     // 784 -> 250: an XCD each
    CHECK(beside(4, 16, true, 2, &bad) == 4);
    CHECK(beside(5, 16, true, 2, &bad) < 5);
    CHECK(beside(2, 8, true, 8, &bad) == 2);
    CHECK(beside(2, 8, true, 16, &bad) < 2);      // the whole GPU
    CHECK(beside(2, 8, true, 17, &bad) < 2);      // unit groups have one workgroup, or two in a tick of fewer clients
    CHECK(beside(2, 16, false, 17, &bad) < 2);    // more than one launch
    CHECK(!bad);
    for (int groups = 1; groups <= 16; ++groups)
        for (int halves = 0; halves < 2; ++halves)
            for (int clients = 1; clients < 300; ++clients) {
                const int size = aet::dense_cluster_size(32, groups, halves, clients), there = (clients + 7) / 8;
                // as many as launches of these clients, or of some of them, can have on an XCD, or nothing goes beside them
                int most = 0;
                for (int now = 1; now <= clients; ++now)
                    most = std::max(most, (now + 7) / 8 * groups * (halves && now <= aet::resident_clusters(256, 8, 2 * groups) ? 2 : 1));
                CHECK(size == 0 || (there * size >= most && there * size <= 32));
                CHECK(size || most > 16);
            }
    CHECK(aet::dense_cluster_size(0, 1, false, 1) == 0);
    std::puts("ok");
}
"""


@pytest.mark.parametrize("program", ["PROGRAM", "SHARED", "DENSE"])
def test_cluster_launches_are_ordered_across_streams(tmp_path, program):
    src, exe = str(tmp_path / "p.cpp"), str(tmp_path / "p")
    with open(src, "w") as f:
        f.write(globals()[program])
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=thread", "-I",
                    os.path.join(ROOT, "paper_2112_13935_amd", "csrc"), "-o", exe, src], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr[-2000:]


def test_every_cluster_launch_takes_its_turn():
    text = open(os.path.join(ROOT, "paper_2112_13935_amd", "csrc", "aet_api.hip")).read()
    for launch in ("launch_mlp_round(", "launch_softmax_batch_round(", "launch_lenet_round("):
        at = text.index(launch)
        assert "ctx->clustered([&] {" in text[at - 120:at], launch
    assert "ctx->clustered(ctx->turn.need, [&](const ClusterTurns<hipStream_t>::Place &place) {" in text[text.index("launch_cnn_round(") - 120:text.index("launch_cnn_round(")]
