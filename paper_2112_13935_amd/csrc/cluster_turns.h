// Cluster launches of several contexts on one GPU share its compute units, or take turns.
//
// The workgroups of a cluster wait for each other, so all of them have to be resident, and the
// launchers see to that for one launch on an otherwise idle GPU.  Two such launches on two
// streams are dispatched side by side: each can get a part of its last cluster onto an XCD (two
// clusters of 32 workgroups: 16 and 16 of the 32 compute units) and wait there for the rest, which
// never comes.  So a launch goes beside others only where each XCD has a compute unit for every
// workgroup of all of them; where it has not, it is ordered after the cluster launches of other contexts that may
// be in flight, the oldest first, by events between the streams.  Nothing is needed while a context is alone.
// Host code without HIP, so that a CPU test can include it.
#pragma once
#include <algorithm>
#include <array>
#include <cstdint>
#include <mutex>
#include <vector>

namespace aet {

constexpr int kTurnXcds = 8;

template <class Stream>
class ClusterTurns {
 public:
    using Held = std::array<int, kTurnXcds>;   // compute units of each XCD
    static constexpr int kAll = 1 << 20;       // held by a launch that goes beside no other one
    // What a launch needs: compute units of an XCD, clients (a cluster each, round the XCDs), workgroups of a cluster at
    // least and at most.  (As it is: nothing beside it.)
    struct Need { int cus = 0, clients = 0, least = 0, most = 0; };
    // Workgroups of a cluster; the XCD of the first client, or below 0: wherever the queue begins (it differs
    // from queue to queue), so that every client counts on every XCD.
    struct Place { int size, first; };
    struct Member {
        Stream stream{};
        uint64_t last = 0;   // turn of its latest cluster launch; 0: none yet
        Held held{};         // by it
        int first = -1;      // its place
        // its launches that may be in flight, oldest first: a record for all in a row that hold the same, with the
        // turn of the latest
        struct Run { uint64_t last; Held held; };
        std::vector<Run> runs;
        // of another member: the turn up to which this one's stream is ordered behind it, and its
        // last turn when this one looked
        struct Order { const Member *of; uint64_t behind, seen; };
        std::vector<Order> orders;
    };
    void join(Member *m) {
        std::lock_guard<std::mutex> hold(mutex_);
        members_.push_back(m);
    }
    // the member's stream has been synchronised: nothing has to wait for it any more
    void leave(Member *m) {
        std::lock_guard<std::mutex> hold(mutex_);
        members_.erase(std::remove(members_.begin(), members_.end(), m), members_.end());
        for (Member *o : members_)
            o->orders.erase(std::remove_if(o->orders.begin(), o->orders.end(), [&](const typename Member::Order &x) { return x.of == m; }), o->orders.end());
    }
    // launch(place) puts the cluster launch into me->stream; before it, after(m) orders that stream behind
    // everything in m->stream.  Both return 0 for success.
    //   idle(m)     everything in m->stream is done (asked of members that have launched nothing since the last look)
    //   mark(me)    a mark in me->stream, ahead of the first launch that holds something else than the one before
    //   passed(m)   m->stream is past its latest mark
    template <class Idle, class Mark, class Passed, class After, class Launch>
    auto take(Member *me, const Need &need, Idle idle, Mark mark, Passed passed, After after, Launch launch) -> decltype(launch(Place())) {
        using Status = decltype(launch(Place()));
        std::lock_guard<std::mutex> hold(mutex_);
        // An XCD is shared with those that are in flight there when this one comes, or have launched there since its last one:
        // their next launches are to fit beside it.  crowd: all that were there last.
        Held shares, crowd{};
        shares.fill(1);
        bool others = false;
        for (Member *m : members_) {
            if (!other(me, m)) continue;
            others = true;
            auto &o = order(me, m);
            if (!m->runs.empty()) {
                if (m->last > o.behind && m->last == o.seen && idle(m)) m->runs.clear();
                else if (m->runs.size() > 1 && passed(m)) m->runs.erase(m->runs.begin(), m->runs.end() - 1);
                o.seen = m->last;
            }
            const bool flying = !m->runs.empty() && m->last > o.behind;
            for (int x = 0; x < kTurnXcds; ++x) {
                shares[x] += m->held[x] && (flying || m->last > me->last);
                crowd[x] += m->held[x] > 0;
            }
        }
        Place place;
        Held held;
        for (;;) {
            Held sum{};
            Member *oldest = nullptr;
            for (Member *m : members_) {
                if (!other(me, m)) continue;
                const uint64_t behind = order(me, m).behind;
                Held most{};   // of its launches that may run beside this one
                bool flying = false;
                for (const auto &r : m->runs)
                    if (r.last > behind) {
                        flying = true;
                        for (int x = 0; x < kTurnXcds; ++x) most[x] = std::max(most[x], r.held[x]);
                    }
                if (!flying) continue;
                for (int x = 0; x < kTurnXcds; ++x) sum[x] = std::min(sum[x] + most[x], (int)kAll);
                if (!oldest || m->last < oldest->last) oldest = m;
            }
            if (fits(*me, need, others, !oldest, sum, shares, crowd, &place, &held)) break;
            const Status status = after(oldest);
            if (status != Status(0)) return status;
            order(me, oldest).behind = oldest->last;
        }
        if (!me->runs.empty() && me->runs.back().held != held) {
            const Status status = mark(me);
            if (status != Status(0)) return status;
        }
        const Status status = launch(place);
        me->last = ++turn_;
        me->held = held;
        me->first = place.first;
        // (beyond a few records the two oldest become one that holds as much as either)
        if (!me->runs.empty() && me->runs.back().held == held) me->runs.back().last = me->last;
        else me->runs.push_back({me->last, held});
        if (me->runs.size() > 4) {
            for (int x = 0; x < kTurnXcds; ++x) me->runs[1].held[x] = std::max(me->runs[0].held[x], me->runs[1].held[x]);
            me->runs.erase(me->runs.begin());
        }
        return status;
    }
    // a launch that goes beside no other one
    template <class After, class Launch>
    auto take(Member *me, After after, Launch launch) -> decltype(launch()) {
        using Status = decltype(launch());
        return take(me, Need(), [](Member *) { return false; }, [](Member *) { return Status(0); }, [](Member *) { return false; }, after,
                    [&](const Place &) { return launch(); });
    }

 private:
    static bool other(const Member *me, const Member *m) { return m != me && m->stream != me->stream; }
    static typename Member::Order &order(Member *me, const Member *m) {
        for (auto &o : me->orders)
            if (o.of == m) return o;
        me->orders.push_back({m, 0, 0});
        return me->orders.back();
    }
    // The place of a launch beside those that hold `sum` (alone: none), if there is one: the largest clusters, where it was
    // before or else where the fewest are.
    static bool fits(const Member &me, const Need &need, bool others, bool alone, const Held &sum, const Held &shares, const Held &crowd,
                     Place *place, Held *held) {
        const int even = need.clients / kTurnXcds, more = need.clients % kTurnXcds, most_there = even + (more ? 1 : 0);
        if (need.cus <= 0 || need.least * most_there > need.cus) {
            *place = {need.most, -1};
            held->fill(kAll);
            return alone;
        }
        // (where all XCDs get as many clients, or nobody else is there, it does not matter which is the first)
        const int from = others && more ? 0 : -1, to = others && more ? kTurnXcds : 0;
        bool found = false, found_same = false;
        int found_crowd = 0;
        for (int f = from; f < to; ++f) {
            const auto there = [&](int x) { return f < 0 ? most_there : even + ((x - f + kTurnXcds) % kTurnXcds < more ? 1 : 0); };
            int size = need.most, crowded = 0;
            for (int x = 0; x < kTurnXcds; ++x) {
                const int n = there(x);
                if (!n) continue;
                if (shares[x] > 1) size = std::min(size, std::min(need.cus - sum[x], need.cus / shares[x]) / n);
                crowded += crowd[x];
            }
            size = std::max(size, need.least);
            Held mine;
            bool room = true;
            for (int x = 0; x < kTurnXcds; ++x) {
                mine[x] = std::min(there(x) * size, need.cus);
                room = room && (alone || !mine[x] || mine[x] + sum[x] <= need.cus);
            }
            const bool same = f == me.first;
            if (!room || (found && (size < place->size || (size == place->size && (found_same || (!same && crowded >= found_crowd)))))) continue;
            found = true;
            found_same = same;
            found_crowd = crowded;
            *place = {size, f};
            *held = mine;
        }
        return found;
    }
    std::mutex mutex_;
    std::vector<Member *> members_;
    uint64_t turn_ = 0;
};

}  // namespace aet
