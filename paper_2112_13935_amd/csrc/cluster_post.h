// Exchange words of a cluster of workgroups: 64-bit {step tag, value} words that validate
// themselves, written by one workgroup and polled by its peers.
//
// What bounds an exchange is how soon a posted word can be read.  A store of agent scope is
// written through the XCD's L2 to memory; a store of workgroup scope stays in that L2 (the L1
// is written through either way), where a peer on the same XCD finds it with an agent-scope load,
// which passes the L1 by.  Ping-pong of two workgroups of one XCD, shader clocks per round trip:
// 2,065 with agent-scope stores, 1,125 with workgroup-scope stores; a peer on another XCD never
// sees the latter.  So the workgroups of a cluster first tell each other which XCD they run on
// (agent scope, once per launch, while the replica is loaded), and only where it is one and the
// same do the words stay in its L2.
//
// The memory model promises none of this: a store of workgroup scope may stay invisible to other
// workgroups.  It holds for this part (gfx950: one L2 per XCD, the L1 written through), which is the only
// one this library is built for.  Were it not so, no tagged word would be taken for another one: the
// bounded waits would expire and the error flag would say so.  Not every client of this header is that safe:
// k_cnn_round also leaves plain words in the L2 (weights, records, partial gradients; put1), and only the barrier
// behind them is tagged.  They are ordered ahead of it by s_waitcnt vmcnt(0), a store being acknowledged by the
// L2, and read past the L1; were they not visible then, a peer would go on with old values and nothing would say so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cluster_plan.h"

namespace aet {

__device__ __forceinline__ int xcc_id() {   // hardware register 20, bits 0 .. 3
    return (int)__builtin_amdgcn_s_getreg(20 | (3 << 11));
}

// places: one word per workgroup of the cluster and one for the answer, the last of kPlaces (NULL: words
// always go to memory); tag: not in any word of an earlier launch; skew: added to the first workgroup's answer (a test's: 0 otherwise)
__device__ __forceinline__ void cluster_announce(unsigned long long *places, int me, uint32_t tag, int skew) {
    if (places && threadIdx.x == 0)
        __hip_atomic_store(places + me, ((unsigned long long)tag << 32) | (unsigned)(xcc_id() + (me == 0 ? skew : 0)),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The bounded wait of a poll loop: gave_up() after every poll in vain.  Once this or another workgroup's
// wait has expired the error flag is set and the answer is yes.
struct BoundedWait {
    int polls = 0;
    __device__ __forceinline__ bool gave_up(int *errflag) {
        if ((++polls & 255) != 0) return false;
        if (polls < kWaitPolls && __hip_atomic_load(errflag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) return false;
        __hip_atomic_store(errflag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
};

// Do all n workgroups of the cluster run on one XCD?  Every wave asks for itself.  Where the wait
// expires *dead is set and the answer is no.  The first workgroup's is left behind for a test to read.
__device__ __forceinline__ bool cluster_on_one_xcd(unsigned long long *places, int me, int n, uint32_t tag, int *errflag, bool *dead) {
    if (!places) return false;
    const int lane = threadIdx.x & 63;
    unsigned long long v = 0;
    BoundedWait wait;
    for (;;) {
        v = __hip_atomic_load(places + min(lane, n - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__all((uint32_t)(v >> 32) == tag)) break;
        if (*dead) return false;
        __builtin_amdgcn_s_sleep(1);
        if (wait.gave_up(errflag)) *dead = true;
    }
    const bool yes = __all((int)(uint32_t)v == xcc_id());
    if (me == 0 && threadIdx.x == 0) __hip_atomic_store(places + kPlaces - 1, yes ? 1ull : 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return yes;
}

// one_xcd: what cluster_on_one_xcd said (the same for all lanes)
__device__ __forceinline__ void cluster_post(unsigned long long *p, uint32_t tag, float v, bool one_xcd) {
    const unsigned long long word = ((unsigned long long)tag << 32) | (unsigned long long)__float_as_uint(v);
    if (one_xcd) __hip_atomic_store(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace aet
