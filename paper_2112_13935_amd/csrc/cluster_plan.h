// How many clusters of workgroups may wait for each other in one launch.  Host arithmetic
// without HIP, so that a CPU test can include it.
//
// Consecutive workgroup ids go round the XCDs, and a cluster's workgroups have ids that are
// equal modulo 8, so all of them run on one XCD: what has to hold the cluster is an XCD, not the
// GPU.  Client a goes to XCD a mod 8 (mod the number of XCDs, where that is 4, 2 or 1).  Counted over
// the whole GPU, 42 clusters of six fit 256 compute units, but six of them fall on each of
// the first two XCDs: 36 workgroups for 32 places, and a cluster of which only a part
// is resident polls until another one has finished its round.
#pragma once
#include <stdint.h>

namespace aet {

// capacity: workgroups that are resident on the whole GPU; xcds: XCDs they are spread over
inline int resident_clusters(int capacity, int xcds, int cluster_size) {
    if (xcds < 1 || 8 % xcds != 0) xcds = 8;   // the ids' mapping knows only these
    return xcds * ((capacity / xcds) / cluster_size);
}

// Workgroups that a client of a dense-ReLU-dense context may have, for contexts on other streams to go beside it (cluster_turns.h):
// `groups`, or twice as many where a launch that has room gives every unit group two (`halves`).  0: nothing goes beside it, an XCD's `cus`
// compute units do not hold them (or, with halves, a tick of fewer clients may have twice as many of each).
inline int dense_cluster_size(int cus, int groups, bool halves, int clients) {
    const int size = halves ? 2 * groups : groups;
    return size * ((clients + 7) / 8) <= cus ? size : 0;
}

// Words that stay in an XCD's L2 are seen by that XCD alone (cluster_post.h): a line of memory that
// holds them must not hold words of a cluster that may run on another one.  So each client's records
// take whole lines.
constexpr int kLineWords = 16;   // 64-bit words of a 128-byte line
constexpr int whole_lines(int words) { return (words + kLineWords - 1) / kLineWords * kLineWords; }

// Records of one client of mini-batch softmax, in words: [step parity][workgroup][sample][12 classes]
constexpr int softmax_batch_record_words(int workgroups, int batch) {
    return workgroups > 1 ? whole_lines(2 * workgroups * batch * 12) : 0;
}

// Words of a client's workgroups about where they run: one each, and the last for their answer
constexpr int kClusterMax = 32;   // workgroups of a cluster, at most
constexpr int kPlaces = whole_lines(kClusterMax + 1);

// Steps of a round, with one tag each: a round has up to 2^31 - 1 recursions, so two steps a recursion need all of 32 bits.
constexpr uint32_t cluster_steps(int recursions, int steps_each) { return (uint32_t)recursions * (uint32_t)steps_each; }
// Whether fewer than `need` tags are left from `next` on (0, the cleared state, is none)
constexpr bool tags_spent(uint32_t next, uint32_t need) { return next == 0 || next - 1u > 0xFFFFFFFFu - need; }

// How many times a workgroup polls for a peer's word before it gives up: 2.2 s with polls of the XCD's L2
// (0.26 us), twice that with polls that go through memory.  (A count and not the clock, which goes on while
// the queue is preempted, and which cost the LeNet round with two clusters a client 1.3 %.)
constexpr int kWaitPolls = 1 << 23;

}  // namespace aet
