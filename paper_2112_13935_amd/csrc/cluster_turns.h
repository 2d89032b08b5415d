// Cluster launches of several contexts on one GPU share its compute units, or take turns.
//
// The workgroups of a cluster wait for each other, so all of them have to be resident, and the
// launchers see to that for one launch on an otherwise idle GPU.  Two such launches on two
// streams are dispatched side by side: each can get a part of its last cluster onto an XCD (two
// clusters of 32 workgroups: 16 and 16 of the 32 compute units) and wait there for the rest, which
// never comes.  So a launch goes beside others only where each XCD has a compute unit for every
// workgroup of all of them, whichever XCD each begins with (that differs from queue to queue);
// where it has not, it is ordered after the cluster launches of other contexts that may be in flight, the
// oldest first, by events between the streams.  Nothing is needed while a context is alone.  Host code
// without HIP, so that a CPU test can include it.
#pragma once
#include <algorithm>
#include <cstdint>
#include <mutex>
#include <vector>

namespace aet {

template <class Stream>
class ClusterTurns {
 public:
    static constexpr int kAll = 1 << 20;   // held by a launch that goes beside no other one
    // What a launch needs: compute units of an XCD, its clusters there, workgroups of a cluster at least and
    // at most.  (As it is: nothing beside it.)
    struct Need { int cus = 0, clusters = 1, least = kAll, most = kAll; };
    struct Member {
        Stream stream{};
        uint64_t last = 0;   // turn of its latest cluster launch; 0: none yet
        // its launches that may be in flight, oldest first: a record for all in a row that hold as many
        // compute units of an XCD, with the turn of the latest
        struct Run { uint64_t last; int held; };
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
    // launch(size) puts the cluster launch, with clusters of `size` workgroups, into me->stream; before it,
    // after(m) orders that stream behind everything in m->stream.  Both return 0 for success.
    //   idle(m)     everything in m->stream is done (asked of members that have launched nothing since the last look)
    //   mark(me)    a mark in me->stream, ahead of the first launch that holds more or less than the one before
    //   passed(m)   m->stream is past its latest mark
    template <class Idle, class Mark, class Passed, class After, class Launch>
    auto take(Member *me, const Need &need, Idle idle, Mark mark, Passed passed, After after, Launch launch) -> decltype(launch(0)) {
        std::lock_guard<std::mutex> hold(mutex_);
        int shares = 1;
        for (Member *m : members_) {
            if (!other(me, m)) continue;
            shares += m->last > me->last;
            if (m->runs.empty()) continue;
            auto &o = order(me, m);
            if (m->last > o.behind && m->last == o.seen && idle(m)) m->runs.clear();
            else if (m->runs.size() > 1 && passed(m)) m->runs.erase(m->runs.begin(), m->runs.end() - 1);
            o.seen = m->last;
        }
        int size = need.most, held = kAll;
        for (;;) {
            int sum = 0, count = 0;
            Member *oldest = nullptr;
            for (Member *m : members_) {
                if (!other(me, m)) continue;
                const uint64_t behind = order(me, m).behind;
                int most = 0;   // of its launches that may run beside this one
                for (const auto &r : m->runs)
                    if (r.last > behind) most = std::max(most, r.held);
                if (!most) continue;
                sum = std::min(sum + most, (int)kAll);
                ++count;
                if (!oldest || m->last < oldest->last) oldest = m;
            }
            shares = std::max(shares, count + 1);
            if (need.least < kAll && need.clusters * need.least <= need.cus) {
                // What is free, but no more than an equal share where there are others: those that are in flight, were when
                // this one came, or have launched since its last one.  Their next launches are to fit beside it.
                const int room = shares > 1 ? std::min(need.cus - sum, need.cus / shares) / need.clusters : need.most;
                size = std::max(need.least, std::min(need.most, room));
                held = std::min(need.clusters * size, need.cus);
            }
            if (!count || sum + held <= need.cus) break;
            const auto status = after(oldest);
            if (status != decltype(launch(0))(0)) return status;
            order(me, oldest).behind = oldest->last;
        }
        if (!me->runs.empty() && me->runs.back().held != held) {
            const auto status = mark(me);
            if (status != decltype(launch(0))(0)) return status;
        }
        const auto status = launch(size);
        me->last = ++turn_;
        // (beyond a few records the two oldest become one that holds as much as the larger)
        if (!me->runs.empty() && me->runs.back().held == held) me->runs.back().last = me->last;
        else me->runs.push_back({me->last, held});
        if (me->runs.size() > 4) {
            me->runs[1].held = std::max(me->runs[0].held, me->runs[1].held);
            me->runs.erase(me->runs.begin());
        }
        return status;
    }
    // a launch that goes beside no other one
    template <class After, class Launch>
    auto take(Member *me, After after, Launch launch) -> decltype(launch()) {
        using Status = decltype(launch());
        return take(me, Need(), [](Member *) { return false; }, [](Member *) { return Status(0); }, [](Member *) { return false; }, after,
                    [&](int) { return launch(); });
    }

 private:
    static bool other(const Member *me, const Member *m) { return m != me && m->stream != me->stream; }
    static typename Member::Order &order(Member *me, const Member *m) {
        for (auto &o : me->orders)
            if (o.of == m) return o;
        me->orders.push_back({m, 0, 0});
        return me->orders.back();
    }
    std::mutex mutex_;
    std::vector<Member *> members_;
    uint64_t turn_ = 0;
};

}  // namespace aet
