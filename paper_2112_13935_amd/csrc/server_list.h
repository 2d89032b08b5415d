// A list of arrivals for the server that is longer than ArrivalPack and still fits the kernel arguments (4 KB): the U
// of an entry is at base + slot * stride.  (As pointers, 16 bytes an entry, 224 would fit: 300 clients of 784 columns, 20 ticks,
// 762 us with the list fetched from pinned memory, 706 this way.)
#pragma once
#include "aet_internal.h"

namespace aet {

constexpr int kArrivalList = 496;
struct ArrivalList {
    const float *base;
    int64_t stride;   // floats between two slots
    struct {
        int32_t slot;
        float scale;
    } a[kArrivalList];
};
static_assert(sizeof(ArrivalList) + 24 <= 4096, "the kernel's other arguments: a model, two lengths");

// launch_server_reduce with the list by value, kArrivalPack < n_arr <= kArrivalList
hipError_t launch_server_reduce_list(hipStream_t s, Profiler *prof, float *Wg, const ArrivalList &list, int n_arr, int64_t P);

}  // namespace aet
