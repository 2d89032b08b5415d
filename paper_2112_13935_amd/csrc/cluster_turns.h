// Cluster launches of several contexts on one GPU take turns.
//
// The workgroups of a cluster wait for each other, so all of them have to be resident, and the
// launchers see to that for one launch on an otherwise idle GPU.  Two such launches on two
// streams are dispatched side by side: each can get a part of its last cluster onto an XCD (two
// clusters of 32 workgroups: 16 and 16 of the 32 compute units) and wait there for the rest, which
// never comes.  So a launch is ordered after the cluster launches that other contexts on the
// GPU made since this one's last, by an event between the streams, and nothing is needed while
// a context is alone.  Host code without HIP, so that a CPU test can include it.
#pragma once
#include <algorithm>
#include <cstdint>
#include <mutex>
#include <vector>

namespace aet {

template <class Stream>
class ClusterTurns {
 public:
    struct Member {
        Stream stream{};
        uint64_t last = 0;   // turn of its latest cluster launch; 0: none yet
    };
    void join(Member *m) {
        std::lock_guard<std::mutex> hold(mutex_);
        members_.push_back(m);
    }
    // the member's stream has been synchronised: nothing has to wait for it any more
    void leave(Member *m) {
        std::lock_guard<std::mutex> hold(mutex_);
        members_.erase(std::remove(members_.begin(), members_.end(), m), members_.end());
    }
    // launch() puts the cluster launch into me->stream; before it, after(m) orders that stream
    // behind everything in m->stream.  Both return 0 for success.
    template <class After, class Launch>
    auto take(Member *me, After after, Launch launch) -> decltype(launch()) {
        std::lock_guard<std::mutex> hold(mutex_);
        for (Member *m : members_)
            if (m != me && m->stream != me->stream && m->last > me->last) {
                const auto status = after(m);
                if (status != decltype(launch())(0)) return status;
            }
        const auto status = launch();
        me->last = ++turn_;
        return status;
    }

 private:
    std::mutex mutex_;
    std::vector<Member *> members_;
    uint64_t turn_ = 0;
};

}  // namespace aet
