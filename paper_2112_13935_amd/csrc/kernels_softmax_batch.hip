// Fused local round for softmax regression with mini-batches (one dense layer D -> 10 classes,
// 2 <= B <= 64).  One launch runs the whole round (Algorithm 2, MainComputeNode: all s_i/B
// recursions) of every active client.
//
// A client is a cluster of HF workgroups (8 waves), each owning a run of 512 * NC columns:
// thread t owns columns t, t + 512, ... of the run for every class row of W and U and, one
// recursion at a time, of the mini-batch.  All three stay in registers, so the memory traffic is
// the sampled rows.  (The form with three columns and 32 samples spills eight registers, all
// ahead of the loop over recursions; one pair of them is read back in it.)  Per recursion:
//   - partial logits: dot products over the thread's columns, two samples (20 sums) at a time
//     folded over the wave with lane swaps and DPP steps, added over the waves through LDS;
//   - HF > 1: the sums of the workgroup's columns go to the cluster's exchange record as
//     64-bit {step tag, value} words; every workgroup reads the others' and adds in cluster
//     order (two records alternate: nobody can post step u + 2 before everybody has read u);
//   - softmax and dz = p - onehot with 16 lanes per sample, dz^T to LDS.  (expf and logf as in the
//     layer engine: with __expf and __logf, 1 % faster, the entries of dz add up to more, and
//     with features of one sign models come out 1.4 times as far from 64 bits: 600 clients x 40
//     columns, mini-batch 8, 12 rounds 1.3e-5 against 1.8e-5 of the norm);
//   - g^T = sum_b x_b dz_b^T as 4 x 4 outer products on the matrix cores (see k_softmax_round:
//     the lane's own column is the B operand), then W -= eta g and U += g in place.  When a
//     column is done its registers take the next recursion's rows.
// Samples beyond the mini-batch (BC is a compile-time bound) repeat its last row with dz = 0;
// columns beyond D read the row's last column with weights of zero.
//
// What bounds it: vector instructions of the forward part (per sample and wave 10 NC
// multiply-adds and 28 for the fold), beside the rows from memory (128 clients x 32 x 12 KB:
// 8 us of a recursion at the rate of a large copy).  As separate kernels (gather, dense
// forward, softmax, weight gradient) a recursion moved the rows four times and W and U once
// more: 128 clients x 3,072 columns, mini-batch 32: 96 us, here 21 us.
//
// All workgroups of a cluster must be resident together: the launcher never puts more on an
// XCD than it has compute units (cluster_plan.h).  The wait is bounded and raises an error flag
// instead of hanging (every workgroup still runs to the end).
#include "aet_device.h"
#include "aet_internal.h"
#include "cluster_plan.h"
#include "cluster_post.h"

namespace aet {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;

constexpr int kSbWaves = 8;
constexpr int kSbThreads = 64 * kSbWaves;
constexpr int kSbClasses = 10;         // the forward part sums two samples' classes as 20 values
constexpr int kSbQ = 3;                // groups of four class rows
constexpr int kSbC = 4 * kSbQ;         // class slots
static_assert(kSbC == 12, "softmax_batch_record_words");
static_assert(2 * kSbClasses == 20 && kSbClasses <= kSbC, "five registers of four sums hold two samples' classes");
constexpr int kSbMaxHF = 6;            // workgroups of a cluster, at most
static_assert(kSbMaxHF <= kClusterMax, "a place for every workgroup");
constexpr int kSbMaxD = kSbMaxHF * kSbThreads;
constexpr int kSbMaxB = 64;
constexpr int kSbPS = 13;              // LDS stride of a sample's partial logits

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum16(float v) {
    v += dpp<0xB1>(v); v += dpp<0x4E>(v); v += dpp<0x141>(v); v += dpp<0x140>(v);
    return v;
}
__device__ __forceinline__ float max16(float v) {
    v = fmaxf(v, dpp<0xB1>(v)); v = fmaxf(v, dpp<0x4E>(v)); v = fmaxf(v, dpp<0x141>(v)); v = fmaxf(v, dpp<0x140>(v));
    return v;
}
// lane swaps of gfx950: halves, then rows of 16, of two registers; the sum of the results
// holds both folded, one per half (row)
__device__ __forceinline__ float fold32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
    return __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
}
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
    return __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
}

template <int NC, int BC>
__global__ void __launch_bounds__(kSbThreads, 1)
k_softmax_batch_round(const RoundParams *__restrict__ rp, int nhere, int rec0, const float *Wg, int D, int C,
                      int HF, int Br, int rec_words, u64 *__restrict__ xrec, u64 *__restrict__ places, int skew, uint32_t tag0, int *__restrict__ errflag) {
    constexpr int Q = kSbQ, T = kSbThreads, NW = kSbWaves;
    constexpr int GS = BC < 32 ? BC : 32;   // samples whose logits are collected before a store
    constexpr int DZ = BC + 4;              // LDS stride of a class row of dz^T
    constexpr int NE = (BC * 16 + T - 1) / T;   // (sample, class) elements per thread
    // the workgroups of a client get ids that land on one XCD
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int a = xcd + 8 * (slot / HF), h = slot % HF;
    if (a >= nhere) return;
    if (places) places += (int64_t)(rec0 + a) * kPlaces;
    if (HF > 1) cluster_announce(places, h, tag0, skew);
    const RoundParams p = rp[a];
    const gci_ptr yg = as_global(p.y);
    const gf_ptr Wc = as_global(p.W), Uc = as_global(p.U);
    const gcf_ptr W0 = as_global(Wg ? Wg : p.W);
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, l4 = lane & 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float invB = 1.0f / (float)Br;

    __shared__ float part[NW][BC * kSbPS];
    __shared__ __attribute__((aligned(16))) float dzT[kSbC * DZ];
    __shared__ float bs[16], Ubs[16];
    __shared__ int labs[BC];
    __shared__ float lred[NW];

    // own columns; one beyond D stands for the last column and keeps zero weights
    int k[NC];
    bool kok[NC];
    f4 W[NC][Q], U[NC][Q];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int kk = h * (T * NC) + tid + T * j;
        kok[j] = kk < D;
        k[j] = min(kk, D - 1);
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = 4 * q + r;
                W[j][q][r] = (o < C && kok[j]) ? W0[(int64_t)o * D + k[j]] : 0.f;
                U[j][q][r] = 0.f;
            }
    }
    if (tid < 16) {
        bs[tid] = tid < C ? W0[(int64_t)C * D + tid] : 0.f;
        Ubs[tid] = 0.f;
    }

    // row addresses and labels of a recursion: lane b for sample b
    uint32_t alo = 0, ahi = 0;
    int labn = 0;
    auto next_rows = [&](int u) {
        const uint32_t r = sample_row(p.key, (uint64_t)(p.q0 + (int64_t)min(u, p.m - 1) * Br + min(lane, Br - 1)), p.n_samples);
        const uint64_t ad = (uint64_t)p.X + (uint64_t)r * (uint64_t)D * 4u;
        alo = (uint32_t)ad;
        ahi = (uint32_t)(ad >> 32);
        labn = yg[r];
    };
    float x[BC][NC];
    auto load_col = [&](int j) {
#pragma unroll
        for (int b = 0; b < BC; ++b) {
            const uint64_t ad = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(ahi, b) << 32) | (uint32_t)__builtin_amdgcn_readlane(alo, b);
            x[b][j] = as_global(reinterpret_cast<const float *>(ad))[(uint32_t)k[j]];
            if ((b & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // few row addresses in scalar registers at a time
        }
    };
    float loss_acc = 0.f;
    u64 *rec_base = xrec + (int64_t)(rec0 + a) * rec_words;
    bool dead = false, one_xcd = false;

    if (p.m > 0) {
        next_rows(0);
#pragma unroll
        for (int j = 0; j < NC; ++j) load_col(j);
        if (wave == 0 && lane < BC) labs[lane] = labn;
        if (HF > 1) one_xcd = cluster_on_one_xcd(places, h, HF, tag0, errflag, &dead);
    }
    for (int u = 0; u < p.m; ++u) {
        int lio = li;   // compared where it is needed: 16 masks kept in scalar registers would spill
        asm volatile("" : "+v"(lio));
        // ---- partial logits of the own columns -------------------------------------------------
#pragma unroll
        for (int b0 = 0; b0 < BC; b0 += GS) {
            float res[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < GS / 2; ++c) {
                float s[2 * kSbClasses];
#pragma unroll
                for (int i = 0; i < 2 * kSbClasses; ++i) {
                    const int o = i % kSbClasses, b = b0 + 2 * c + i / kSbClasses;
                    s[i] = W[0][o >> 2][o & 3] * x[b][0];
#pragma unroll
                    for (int j = 1; j < NC; ++j) s[i] += W[j][o >> 2][o & 3] * x[b][j];
                }
                // row r of register kk ends up with the total of sum 4 kk + {0, 2, 1, 3}[r]
                float t[5];
#pragma unroll
                for (int kk = 0; kk < 5; ++kk)
                    t[kk] = fold16(fold32(s[4 * kk], s[4 * kk + 1]), fold32(s[4 * kk + 2], s[4 * kk + 3]));
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) t[kk] += dpp<0xB1>(t[kk]);
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) t[kk] += dpp<0x4E>(t[kk]);
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) t[kk] += dpp<0x141>(t[kk]);
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) t[kk] += dpp<0x140>(t[kk]);
                // lane c of every row keeps pair c
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) res[kk] = lio == c ? t[kk] : res[kk];
                __builtin_amdgcn_sched_barrier(0);
            }
            if (li < GS / 2) {
                const int row = lane >> 4, o0 = ((row & 1) << 1) | (row >> 1);
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) {
                    const int i = 4 * kk + o0, second = i >= kSbClasses ? 1 : 0;
                    part[wave][(b0 + 2 * li + second) * kSbPS + i - kSbClasses * second] = res[kk];
                }
            }
        }
        __syncthreads();
        // ---- logits: waves, then the cluster's workgroups, in order ------------------------------
        float z[NE];
        const uint32_t tag = tag0 + (uint32_t)u;
        u64 *rec = rec_base + (int64_t)(u & 1) * (rec_words >> 1);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = tid + T * e, b = i >> 4, o = i & 15;
            z[e] = 0.f;
            if (b < Br && o < C) {
#pragma unroll
                for (int w = 0; w < NW; ++w) z[e] += part[w][b * kSbPS + o];
                if (HF > 1) cluster_post(rec + ((int64_t)h * Br + b) * kSbC + o, tag, z[e], one_xcd);
            }
        }
        next_rows(u + 1);   // the hash runs while the words travel
        if (HF > 1) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int i = tid + T * e, b = i >> 4, o = i & 15;
                if (b < Br && o < C) {
                    const u64 *src = rec + (int64_t)b * kSbC + o;
                    BoundedWait wait;
                    float sum;
                    for (;;) {
                        u64 v[6];
                        bool ok = true;
#pragma unroll
                        for (int g = 0; g < 6; ++g)
                            v[g] = __hip_atomic_load(src + (int64_t)(g < HF ? g : h) * Br * kSbC, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        sum = 0.f;
#pragma unroll
                        for (int g = 0; g < 6; ++g)
                            if (g < HF) {
                                ok = ok && (g == h || (uint32_t)(v[g] >> 32) == tag);
                                sum += g == h ? z[e] : __uint_as_float((uint32_t)v[g]);
                            }
                        if (ok || dead) break;
                        __builtin_amdgcn_s_sleep(1);
                        if (wait.gave_up(errflag)) dead = true;
                    }
                    z[e] = sum;
                }
            }
        }
        // ---- softmax, dz -------------------------------------------------------------------------
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = tid + T * e, b = i >> 4, o = i & 15;
            const bool live = b < Br && o < C;
            const float zz = z[e] + bs[o];
            const float zmax = max16(live ? zz : -3.0e38f);
            const float ex = live ? expf(zz - zmax) : 0.f;
            const float lse = zmax + logf(sum16(ex));
            const int lab = labs[min(b, BC - 1)];
            if (live && o == lab) loss_acc += lse - zz;
            if (b < BC && o < kSbC) dzT[o * DZ + b] = live ? expf(zz - lse) - (o == lab ? 1.f : 0.f) : 0.f;
        }
        __syncthreads();
        if (wave == 0 && lane < BC) labs[lane] = labn;
        if (wave == 1 && lane < kSbC) {   // bias (every workgroup keeps a copy)
            float s = 0.f;
#pragma unroll
            for (int b = 0; b < BC; b += 4) {
                const f4 v = *reinterpret_cast<const f4 *>(&dzT[lane * DZ + b]);
                s += (v[0] + v[1]) + (v[2] + v[3]);
            }
            s *= invB;
            bs[lane] -= p.eta * s;
            Ubs[lane] += s;
        }
        // ---- g, update, the next recursion's rows ------------------------------------------------
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            f4 G[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) G[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < BC; b += 4) {
                f4 av[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) av[q] = *reinterpret_cast<const f4 *>(&dzT[(4 * q + l4) * DZ + b]);
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int q = 0; q < Q; ++q) G[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(av[q][r], x[b + r][j], G[q], 0, 0, 0);
            }
            if (u + 1 < p.m) load_col(j);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float gv = G[q][r] * invB;
                    W[j][q][r] = kok[j] ? W[j][q][r] - p.eta * gv : 0.f;
                    U[j][q][r] += gv;
                }
            }
        }
    }

#pragma unroll
    for (int j = 0; j < NC; ++j)
        if (kok[j]) {
#pragma unroll
            for (int o = 0; o < kSbC; ++o)
                if (o < C) {
                    Wc[(int64_t)o * D + k[j]] = W[j][o >> 2][o & 3];
                    Uc[(int64_t)o * D + k[j]] = U[j][o >> 2][o & 3];
                }
        }
    __syncthreads();   // bs, Ubs are written
    // the recursions' mean losses, added up
    float l = loss_acc;
    l = sum16(l);
    l = fold16(l, l);
    l = fold32(l, l);
    if (lane == 0) lred[wave] = l * invB;
    __syncthreads();
    if (h == 0) {
        if (tid < C) {
            Wc[(int64_t)C * D + tid] = bs[tid];
            Uc[(int64_t)C * D + tid] = Ubs[tid];
        }
        if (tid == 0) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += lred[w];
            *as_global(p.loss) = s;
        }
    }
}

__global__ void k_sb_zero(u64 *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// exchange record of one client: [step parity][workgroup][sample][class slot]
int rec_words(int D, int B) {
    return softmax_batch_record_words((D + kSbThreads - 1) / kSbThreads, B);
}
// the records of all clients, then the workgroups' places [client][kPlaces]; the error flag follows
size_t all_words(int n_clients, int D, int B) {
    const int words = rec_words(D, B);
    return words > 0 ? (size_t)n_clients * (words + kPlaces) : 0;
}

}  // namespace

bool softmax_batch_round_supported(int D, int C, int B) {
    return B >= 2 && B <= kSbMaxB && C == kSbClasses && D >= 1 && D <= kSbMaxD;
}

bool softmax_batch_in_clusters(int D) { return D > kSbThreads; }

size_t softmax_batch_scratch_bytes(int n_clients, int D, int B) {
    return all_words(n_clients, D, B) * 8 + 256;
}

const int *softmax_batch_error_flag_ptr(void *scratch, int n_clients, int D, int B) {
    return reinterpret_cast<const int *>(static_cast<u64 *>(scratch) + all_words(n_clients, D, B));
}

hipError_t softmax_batch_clear_error_flag(hipStream_t s, void *scratch, int n_clients, int D, int B) {
    k_sb_zero<<<1, 64, 0, s>>>(static_cast<u64 *>(scratch) + all_words(n_clients, D, B), 1);
    return hipGetLastError();
}

template <int NC, int BC>
static hipError_t sb_launch(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int resident, const float *Wg,
                            int D, int C, int B, int HF, int n_clients, void *scratch, uint32_t tag0) {
    u64 *xrec = static_cast<u64 *>(scratch);
    const int words = rec_words(D, B);
    u64 *places = g_posts_to_memory ? nullptr : xrec + (size_t)n_clients * words;
    int *errflag = reinterpret_cast<int *>(xrec + all_words(n_clients, D, B));
    // a cluster of one never waits: any number of clients per launch; else as many clusters as
    // are resident together
    const int per_launch = HF == 1 ? nact : resident;
    if (per_launch < 1) return hipErrorLaunchOutOfResources;
    for (int a0 = 0; a0 < nact; a0 += per_launch) {
        const int here = nact - a0 < per_launch ? nact - a0 : per_launch;
        const unsigned grid = (unsigned)(8 * ((here + 7) / 8) * HF);
        if (prof && prof->on[F_SOFTMAX_ROUND]) prof->before(F_SOFTMAX_ROUND, s);
        k_softmax_batch_round<NC, BC><<<grid, kSbThreads, 0, s>>>(dp + a0, here, a0, Wg, D, C, HF, B, words, xrec, places, g_xcd_skew, tag0, errflag);
        if (prof && prof->on[F_SOFTMAX_ROUND]) prof->after(F_SOFTMAX_ROUND, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_softmax_batch_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int max_m,
                                      const float *Wg, int D, int C, int B, void *scratch, int n_clients, uint32_t *epoch) {
    if (nact <= 0) return hipSuccess;
    const size_t words = all_words(n_clients, D, B);
    // step tags of this launch: never 0 and never one that an earlier launch may have left
    // A captured launch carries its tags into every replay, where the records still hold words
    // of the replay before with the same tags: there the records are cleared ahead of it.
    const bool spent = *epoch == 0 || *epoch > 0xFFFFFFFFu - (uint32_t)max_m - 2u;
    if (words > 0 && (spent || stream_is_capturing(s))) {
        k_sb_zero<<<(unsigned)((words + 255) / 256), 256, 0, s>>>(static_cast<u64 *>(scratch), words);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (spent) *epoch = 1;
    const uint32_t tag0 = *epoch;
    *epoch += (uint32_t)max_m + 1u;
    int dev = 0, cus = 0, xcds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = device_xcds(&xcds);
    if (e != hipSuccess) return e;
    // One column per thread (more workgroups per client) for mini-batches whose rows would not
    // fit the registers otherwise, and for mini-batches of more than 16 when all clusters are
    // resident that way; else three columns, which take more clients per launch.  21 recursions of 3,072
    // columns, one column and three: mini-batch 32, 40 clients 281 and 386 us, 8 clients 234 and
    // 356; mini-batch 17, 40 clients 269 and 381.  (Mini-batches of up to 16 could use one column
    // there as well: 16 samples, 40 clients 198 and 261 us, 784 columns, 100 clients 185 and 236.)
    const int hf1 = (D + kSbThreads - 1) / kSbThreads, hf3 = (D + 3 * kSbThreads - 1) / (3 * kSbThreads);
    // (one workgroup per compute unit is sure to be resident)
    const int r1 = resident_clusters(cus, xcds, hf1), r3 = resident_clusters(cus, xcds, hf3);
#define AET_SB(nc, bc) return sb_launch<nc, bc>(s, prof, dp, nact, nc == 1 ? r1 : r3, Wg, D, C, B, nc == 1 ? hf1 : hf3, n_clients, scratch, tag0)
    if (hf1 == 1 || B > 32 || (B > 16 && nact <= r1)) {
        if (B <= 8) AET_SB(1, 8);
        if (B <= 16) AET_SB(1, 16);
        if (B <= 32) AET_SB(1, 32);
        AET_SB(1, 64);
    }
    if (B <= 8) AET_SB(3, 8);
    if (B <= 16) AET_SB(3, 16);
    AET_SB(3, 32);
#undef AET_SB
}

}  // namespace aet
