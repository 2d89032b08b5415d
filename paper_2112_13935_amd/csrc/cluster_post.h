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

// The same word, and a claim, where the workgroup has taken its place by the XCD that it runs on: false, for the whole
// workgroup, if another one was there before.  (Should the ids not go round the XCDs; some other place stays empty then, and the bounded waits
// say so.)  claims: as places, but never NULL; lds: a word that is free
__device__ __forceinline__ bool cluster_claim(unsigned long long *claims, int me, uint32_t tag, int skew, float *lds) {
    if (threadIdx.x == 0) {
        const unsigned long long word = ((unsigned long long)tag << 32) | (unsigned)(xcc_id() + (me == 0 ? skew : 0));
        const unsigned long long was = __hip_atomic_exchange(claims + me, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *lds = (uint32_t)(was >> 32) == tag ? 1.f : 0.f;
    }
    __syncthreads();
    const bool taken = *lds != 0.f;
    __syncthreads();
    return !taken;
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

// Dword 3 of a raw buffer descriptor for 32-bit untyped accesses, and the cache policy of agent scope: a load passes the L1
// by, a store goes through to memory.
constexpr int kBufferFlags = 0x00020000;
constexpr int kAgent = 16;

// A client's exchange words through a range-checked buffer: a word is a 32-bit offset, and what differs from record to
// record a scalar or an immediate, so that a post or a poll takes no address arithmetic.  The scopes are cluster_post's.
// A post of four words is two stores of 16 bytes.  Like the rest here it relies on more than the memory model says: that each aligned
// 8-byte half of such a store appears whole (the two need not appear together).
//
// To the compiler these are plain loads and stores, of memory that others change.  A poll loop needs look_again() in it, which
// says that memory may have changed: loads are not moved across it, nor folded with those before it.  That holds only for
// memory that the compiler cannot take for this kernel's alone, and what is reached through a __restrict__ argument it does take
// for that (two looks at a word become one, a poll loop loses its load).  So the buffer begins at a pointer whose origin
// is hidden; nothing is read or written through the argument itself.  (Without __restrict__ on the arguments instead, other
// code of the MLP round is compiled worse: 16 clients, 784 -> 128, 50 rounds 6,908 -> 7,061 us.)
struct ClusterWords {
    typedef int i2 __attribute__((ext_vector_type(2)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    __amdgpu_buffer_rsrc_t r;
    static __device__ __forceinline__ unsigned long long *hidden(unsigned long long *p) {
        asm("" : "+s"(p));
        return p;
    }
    // `words` words from all + first on.  (The argument is hidden as it is, so that the sum can be worked out again where it is needed.)
    __device__ __forceinline__ ClusterWords(unsigned long long *all, int64_t first, int words)
        : r(__builtin_amdgcn_make_buffer_rsrc(hidden(all) + first, 0, 8 * words, kBufferFlags)) {}
    static __device__ __forceinline__ void look_again() { asm volatile("" ::: "memory"); }
    // at, base: bytes; base the same for all lanes.  {value, tag}
    __device__ __forceinline__ i2 get(int at, int base) const {
        return __builtin_bit_cast(i2, __builtin_amdgcn_raw_buffer_load_b64(r, at, base, kAgent));
    }
    __device__ __forceinline__ void post(int at, int base, uint32_t tag, float v, bool one_xcd) const {
        typedef unsigned int u2 __attribute__((ext_vector_type(2)));
        const u2 word = {__float_as_uint(v), tag};
        if (one_xcd) __builtin_amdgcn_raw_buffer_store_b64(word, r, at, base, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(word, r, at, base, kAgent);
    }
    __device__ __forceinline__ void post(int at, int base, uint32_t tag, const f4 &v, bool one_xcd) const {   // four neighbours
        typedef unsigned int u4 __attribute__((ext_vector_type(4)));
        const u4 a = {__float_as_uint(v[0]), tag, __float_as_uint(v[1]), tag}, b = {__float_as_uint(v[2]), tag, __float_as_uint(v[3]), tag};
        if (one_xcd) {
            __builtin_amdgcn_raw_buffer_store_b128(a, r, at, base, 0);
            __builtin_amdgcn_raw_buffer_store_b128(b, r, at + 16, base, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b128(a, r, at, base, kAgent);
            __builtin_amdgcn_raw_buffer_store_b128(b, r, at + 16, base, kAgent);
        }
    }
};

// one_xcd: what cluster_on_one_xcd said (the same for all lanes)
__device__ __forceinline__ void cluster_post(unsigned long long *p, uint32_t tag, float v, bool one_xcd) {
    const unsigned long long word = ((unsigned long long)tag << 32) | (unsigned long long)__float_as_uint(v);
    if (one_xcd) __hip_atomic_store(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace aet
