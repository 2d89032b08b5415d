// Which form of the mini-batch softmax kernels runs a round (kernels_softmax_batch.hip).  Host arithmetic without
// HIP, so that a CPU test can include it.
#pragma once
#include "cluster_plan.h"

namespace aet {

constexpr int kSbRun = 512;   // columns of a run: 16 blocks of columns for each of 8 waves ... or one per thread

struct SoftmaxBatchForm {
    bool lanes;       // a column per lane, or tiles of the matrix cores
    int runs;         // runs of columns of a workgroup
    int samples;      // room for samples
    int columns;      // tiles: 0 every wave has all its blocks and all columns of them exist, 1 four columns and more, 2 fewer
    int workgroups;   // of a cluster
};

// batch: 2 .. 64; clients: of the launch; cus: one workgroup per compute unit is sure to be resident
inline SoftmaxBatchForm softmax_batch_form(int D, int batch, int clients, int cus, int xcds) {
    // How many runs of columns a workgroup takes at most: more workgroups per client have fewer blocks
    // each, fewer need no exchange and take more clients per launch.  Microseconds per recursion, with m tiles of 16
    // samples: 1 + 1.2 m for what does not depend on the columns, 0.5 for an exchange, 0.16 m per block and wave.
    const int m = batch > 32 ? 4 : batch > 16 ? 2 : 1;
    int best = 0;
    double least = 0;
    for (int runs = 1; runs <= (m == 4 ? 2 : 3); ++runs) {
        const int wgs = (D + runs * kSbRun - 1) / (runs * kSbRun), resident = resident_clusters(cus, xcds, wgs);
        const int launches = (clients + resident - 1) / resident;
        const int blocks = (((D + 15) / 16 + wgs - 1) / wgs + 7) / 8;
        const double cost = launches * (1.0 + 1.2 * m + (wgs > 1 ? 0.5 : 0.0) + 0.16 * m * blocks);
        if (best == 0 || cost < least) best = runs, least = cost;
    }
    // Mini-batches that fill no more than half of a tile's rows have no use for the matrix cores in the largest
    // form, nor where a compute unit gets several clients in turn (the lane form leaves registers for two at
    // once); nor have those of up to 16 whose rows, at odd addresses, come in twice as many pieces as 16-byte loads.
    // Tiles / lanes: mini-batch 8, 400 clients x 1,100 columns 1.31, 192 x 3,072 1.10, 400 x 500 1.14 (100 x 1,100
    // 0.94); 16, 192 x 3,071 1.09 (192 x 3,072 0.83).
    const bool odd = D % 4 != 0;
    const bool lanes = (best == 3 && (batch <= 8 || (batch <= 16 && odd))) || (batch <= 8 && (clients > cus ? D > 256 : best == 2 && odd && D > 2 * kSbRun));
    if (lanes) best = D > kSbRun ? 3 : 1;
    SoftmaxBatchForm f;
    f.lanes = lanes;
    f.runs = best;
    f.samples = batch <= 8 ? 8 : batch <= 16 ? 16 : batch <= 32 ? 32 : 64;
    f.workgroups = (D + best * kSbRun - 1) / (best * kSbRun);
    f.columns = lanes ? 0 : D == f.workgroups * kSbRun * best ? 0 : D >= 4 ? 1 : 2;
    return f;
}

}  // namespace aet
