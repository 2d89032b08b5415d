// Internal declarations shared by the host scheduler and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "per_device.h"

namespace aet {

// XCDs of the current GPU
inline hipError_t device_xcds(int *xcds) {
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    static PerDevice known;
    return known.get(dev, xcds, [dev](int *n) { return hipDeviceGetAttribute(n, hipDeviceAttributeNumberOfXccs, dev); });
}

// Is the stream under graph capture?  (An error is no answer: the default stream may not be asked
// while another stream is captured.)
inline bool stream_is_capturing(hipStream_t s) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return status == hipStreamCaptureStatusActive;
}

// Test hook: the exchange words of clusters always go through memory (see cluster_post.h).
extern bool g_posts_to_memory;
// Test hook: the first workgroup of a cluster names an XCD that is not its own.
extern int g_xcd_skew;

// Resolved geometry of one layer (activations are C,H,W per sample).
struct LayerGeom {
    int type, relu, k, pad;
    int ic, ih, iw, oc, oh, ow;
    int64_t w_off, b_off;       // offsets into the flat parameter vector
    int64_t in_size, out_size;  // floats per sample
};

// Everything a kernel needs to know about one client's round of this tick.
// One record per ACTIVE client; the array lives in device memory.
struct RoundParams {
    const float *X;      // shard rows
    const int32_t *y;    // shard labels
    float *W;            // the client's replica w_c (P floats)
    float *U;            // the slot that receives this round's gradient sum
    float *loss;         // accumulates the per-recursion mean loss
    uint64_t key;        // SplitMix64 stream key of (seed, client)
    int64_t q0;          // sample counter at the start of the round
    uint32_t n_samples;  // rows in the shard
    int32_t m;           // recursions in this round
    float eta;           // round step size
    int32_t client;
};

// One arriving message: w -= scale * U at the server, or at every neighbour of the sender.
struct Arrival {
    const float *U;
    float scale;
    int32_t sender;
};

// A short arrival list that is passed to the kernel by value.
constexpr int kArrivalPack = 32;
struct ArrivalPack {
    Arrival a[kArrivalPack];
};

// The convolutions' weights of the current recursion as bf16 parts (kernels_conv_split.hip).
struct SplitWeights {
    char *base = nullptr;          // NULL: not kept
    int64_t stride = 0;            // between clients, in 16-byte pieces
    int64_t off[16][2] = {};       // [layer][forward, backward-data], in bytes; < 0: no such form
};

// Device scratch of the layer-by-layer engine; all sized for n_clients * batch samples.
struct LayerScratch {
    float *act[17];     // act[0] = gathered inputs, act[l+1] = output of layer l
    float *del[17];     // d loss / d act[l] (l >= 1)
    uint8_t *amax[16];  // pool layers: which of the 4 window elements was the maximum
    int32_t *labels;    // [n_clients][batch]
    float *wgrad[16];   // convolutions: partial sums of the weight gradient
    bool wgrad_apart;   // ... each layer's in a place of its own (else all in the same)
    SplitWeights split;
    bool plain;         // use the plain (non matrix-core) layer kernels
    bool fp32_convolutions;   // no split ones
};

// Kernel families, for the optional per-launch timing with HIP events.
enum Family {
    F_BEGIN_ROUND = 0, F_GATHER, F_DENSE_FWD, F_DENSE_BWD_DATA, F_DENSE_BWD_WEIGHT, F_CONV_FWD,
    F_CONV_BWD_DATA, F_CONV_BWD_WEIGHT, F_POOL_FWD, F_POOL_BWD, F_SOFTMAX_CE, F_SERVER_REDUCE,
    F_SOFTMAX_ROUND, F_MLP_ROUND, F_NEIGHBOUR_APPLY, F_LENET_ROUND, F_CNN_ROUND, F_COUNT
};
const char *family_name(int fam);

// Times the launches of the enabled families with event pairs recorded on the launch
// stream; durations are summed when the pairs are drained.
struct Profiler {
    struct Pair { int fam; hipEvent_t a, b; };
    bool on[F_COUNT] = {};
    bool any = false;
    double total_ms[F_COUNT] = {};
    int64_t launches[F_COUNT] = {};
    std::vector<hipEvent_t> pool;
    std::vector<Pair> pending;
    hipEvent_t cur = nullptr;
    hipError_t status = hipSuccess;

    void before(int fam, hipStream_t s);
    void after(int fam, hipStream_t s);
    hipError_t drain(hipStream_t s);
    void clear();
    ~Profiler();
};

// ---- launchers (each returns the launch status) --------------------------------------
// Wg == NULL (here and in the fused round kernels): the clients go on from their own replicas
hipError_t launch_begin_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact,
                              const float *Wg, int64_t P);
hipError_t launch_layer_step(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u,
                             const LayerGeom *lay, int L, int B, const LayerScratch &sc);
hipError_t launch_server_reduce(hipStream_t s, Profiler *prof, float *Wg, const Arrival *darr,
                                int n_arr, int64_t P);
hipError_t launch_server_apply_small(hipStream_t s, Profiler *prof, float *Wg, const ArrivalPack &pack,
                                     int n_arr, int64_t P);
// Receive at the neighbours: replica r takes the arrivals whose sender is in nbr[nbr_off[r] ..
// nbr_off[r+1]), in list order.  The list comes by value (pack != NULL, n_arr <= kArrivalPack)
// or from device memory (darr).  W: the replicas, Ps floats apart.
hipError_t launch_apply_neighbour_U(hipStream_t s, Profiler *prof, float *W, int64_t Ps, int64_t P,
                                    int n_clients, const int32_t *nbr_off, const int32_t *nbr,
                                    const ArrivalPack *pack, const Arrival *darr, int n_arr);
// every replica (Ps floats apart, Ps a multiple of 4) <- src (Ps floats readable)
hipError_t launch_broadcast_model(hipStream_t s, float *W, int64_t Ps, int n_clients, const float *src);
hipError_t launch_debug_indices(hipStream_t s, uint64_t key, int64_t q0, int count,
                                uint32_t n_samples, int32_t *dst);
// convolution on the matrix cores (kernels_conv_mfma.hip); bwd = backward-data
bool conv_mfma_supported(const LayerGeom &L, bool bwd);
hipError_t launch_conv_mfma(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                            const LayerGeom &L, bool bwd, const float *src, float *dst,
                            const float *mask_src, uint8_t *amax = nullptr);
// the same on the bf16 matrix cores (kernels_conv_split.hip), where that is faster
// bytes per client that it wants for the layer's weights; 0: never used with so many clients
size_t conv_split_weight_bytes(const LayerGeom &L, bool bwd, int B, int n_clients);
bool conv_split_used(const LayerGeom *lay, int l, bool bwd, int B, int nact, const SplitWeights &sw);
// the weights of this recursion for every layer and direction that is used
hipError_t launch_split_weights(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, const LayerGeom *lay, int L, int B,
                                const SplitWeights &sw);
// off: of the layer's weights in this direction, in sw.  amax: forward, as for launch_conv_mfma; backward-
// data, not NULL: src is the gradient at the outputs of the 2 x 2 pooling layer behind, amax its winners
hipError_t launch_conv_split(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                             const LayerGeom &L, bool bwd, const SplitWeights &sw, int64_t off, const float *src, float *dst,
                             const float *mask_src, uint8_t *amax);
// backward-weight: slices (partial results) per client, at most cap over all; 0: no such form.  KP, OCP: columns
// and rows of a partial result
int conv_wgrad_split_slices(const LayerGeom &L, int B, int nact, int cap);
hipError_t launch_conv_wgrad_split(hipStream_t s, const RoundParams *dp, int nact, int u, int B, const LayerGeom &L, int S, int KP,
                                   int OCP, const float *in, const float *dout, const uint8_t *amax, float *partial);
// amax != NULL (forward only): dst is the output of the 2 x 2 pooling layer behind it, amax its winners
bool conv_pool_fused(const LayerGeom &L, const LayerGeom &pool);
bool conv_wgrad_mfma_supported(const LayerGeom &L, int B);
size_t conv_wgrad_partial_floats(const LayerGeom &L, int B, int n_clients);
// weight updates of convolutions that wait for the recursion's end, when one launch does them all
struct FinishList {
    alignas(8) unsigned char bytes[1024] = {};
    int blocks = 0;
};
hipError_t launch_conv_wgrad_finish(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                                    const FinishList &later);
hipError_t launch_conv_wgrad_mfma(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u,
                                  int B, const LayerGeom &L, const float *in, const float *dout,
                                  float *partial, FinishList *later, bool split_ok, const uint8_t *amax = nullptr);
// whether the backward kernels of a convolution take the gradient of the 2 x 2 pooling layer behind it and put
// their own together from it and the winners, amax (split: backward-data runs in the split form)
bool conv_bwd_unpools(const LayerGeom &L, const LayerGeom &pool, int B, int nact, bool split);
// backward-data and backward-weight of a layer in one launch where both are small; amax as above
hipError_t launch_conv_bwd_pair(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                                const LayerGeom &L, const float *dout, uint8_t *amax, float *din, const float *mask_src,
                                const float *in, float *partial, FinishList *later, bool *taken);
// dense layers on the matrix cores (kernels_dense_mfma.hip); mode 0 fwd, 1 bwd-data, 2 bwd-weight
hipError_t launch_dense_mfma(hipStream_t s, Profiler *prof, int mode, const RoundParams *dp, int nact,
                             int u, int B, int K, int O, int64_t w_off, int64_t b_off, int relu,
                             const float *x, const float *y, float *z, const float *mask_src);
// d(input) and update of a dense layer that is not the first, in one launch, where that is faster
// than two; masked: the input went through a ReLU
bool dense_bwd_pays(const LayerGeom &L, int B, int nact);
hipError_t launch_dense_bwd(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                            const LayerGeom &L, const float *in, const float *dout, float *din, bool masked);
// the whole last dense layer (logits, softmax cross-entropy, d(input), update) in one launch, where it
// fits and is faster
bool dense_head_pays(const LayerGeom &L, int B, int nact);
hipError_t launch_dense_head(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                             const LayerGeom &L, const float *in, const int32_t *labels, float *din, bool masked);
// fused round of softmax regression, per-sample SGD (kernels_softmax.hip)
bool softmax_round_supported(int D, int C, int B);
hipError_t launch_softmax_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact,
                                const float *Wg, int D, int C);
// ... with mini-batches (kernels_softmax_batch.hip)
bool softmax_batch_round_supported(int D, int C, int B);
bool softmax_batch_in_clusters(int D);   // more than one workgroup per client
size_t softmax_batch_scratch_bytes(int n_clients, int D, int B);
hipError_t launch_softmax_batch_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int max_m,
                                      const float *Wg, int D, int C, int B, void *scratch, int n_clients, uint32_t *epoch);
hipError_t softmax_batch_clear_error_flag(hipStream_t s, void *scratch, int n_clients, int D, int B);
const int *softmax_batch_error_flag_ptr(void *scratch, int n_clients, int D, int B);
// fused round of dense-ReLU-dense models (kernels_mlp.hip)
bool mlp_round_supported(int D, int H, int C, int B);
bool mlp_round_exact(int H, int B);   // no padded units or samples
bool mlp_padded_pays(int D, int H, int B, int n_clients);   // else: faster than the layer engine
size_t mlp_round_scratch_bytes(int n_clients, int B);
// hp: HOST array of the tick's round records (they are passed on in kernel arguments); first: the XCD of the first client, or below 0:
// wherever the queue begins
hipError_t launch_mlp_round(hipStream_t s, Profiler *prof, const RoundParams *hp, int nact,
                            int max_m, const float *Wg, int D, int H, int C, int B, void *scratch,
                            int n_clients, int first, uint32_t *epoch);
// Of a context's launches, for others to go beside them: compute units of an XCD (0: nothing does), clients (round the XCDs from `first`
// on; a multiple of eight, every XCD counted as the fullest, where the kernel does not take `first`) and workgroups of a client
hipError_t mlp_cluster_need(int D, int H, int B, int n_clients, int *cus, int *clients, int *size);
hipError_t mlp_clear_error_flag(hipStream_t s, void *scratch, int n_clients, int B);
const int *mlp_error_flag_ptr(void *scratch, int n_clients, int B);
// fused round of LeNet-5-style models (kernels_lenet.hip); dp: DEVICE array of round records
bool lenet_round_supported(const LayerGeom *lay, int L, int B);
bool lenet_round_exact(int B);   // no padded samples, one cluster per client
bool lenet_padded_pays(const LayerGeom &conv1, int B, int n_clients);   // else: faster than the layer engine
size_t lenet_round_scratch_bytes(int n_clients, int B);
hipError_t launch_lenet_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int max_m,
                              const float *Wg, const LayerGeom *lay, int L, int B, void *scratch,
                              int n_clients, uint32_t *epoch);
hipError_t lenet_clear_error_flag(hipStream_t s, void *scratch, int n_clients, int B);
const int *lenet_error_flag_ptr(void *scratch, int n_clients, int B);
// fused round of small convolutional networks (kernels_cnn.hip); dp: DEVICE array of round records
bool cnn_round_pays(const LayerGeom *lay, int L, int B, int n_clients);   // supported, and faster than the layer engine
size_t cnn_round_scratch_bytes(const LayerGeom *lay, int L, int n_clients, int B);
hipError_t launch_cnn_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int max_m, const float *Wg,
                            const LayerGeom *lay, int L, int B, void *scratch, int n_clients, int size, int first, uint32_t *epoch);
// Compute units of an XCD (0: there are not eight, or they are not to be shared), workgroups of a cluster: the fewest (the
// ones that take samples) and as many as help
hipError_t cnn_cluster_need(const LayerGeom *lay, int L, int B, int n_clients, int *cus, int *least, int *most);
hipError_t cnn_prepare(hipStream_t s, const LayerGeom *lay, int L, int B, void *scratch, int n_clients);   // once, ahead of the first launch
const int *cnn_error_flag_ptr(void *scratch, int n_clients);

}  // namespace aet
