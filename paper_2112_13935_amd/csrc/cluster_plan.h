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

namespace aet {

// capacity: workgroups that are resident on the whole GPU; xcds: XCDs they are spread over
inline int resident_clusters(int capacity, int xcds, int cluster_size) {
    if (xcds < 1 || 8 % xcds != 0) xcds = 8;   // the ids' mapping knows only these
    return xcds * ((capacity / xcds) / cluster_size);
}

}  // namespace aet
