// Fused local round for softmax regression with mini-batches (one dense layer D -> 10 classes,
// 2 <= B <= 64).  One launch runs the whole round (Algorithm 2, MainComputeNode: all s_i/B
// recursions) of every active client.
//
// A client is a cluster of HF workgroups (8 waves); the columns, in blocks of 16, are dealt over the
// workgroups and their waves.  A wave keeps its blocks of W and of the mini-batch in registers, and U
// there or, where a wave has more than four blocks, in LDS.  Per recursion:
//   - partial logits on the matrix cores (v_mfma_f32_16x16x4_f32, 16 samples by 16 classes, four columns
//     at a time): lane (li, lg) holds columns 4 lg .. 4 lg + 3 of a block for sample li and for class li,
//     so rows and weights are 16-byte loads; added over the waves through LDS;
//   - HF > 1: the sums of the workgroup's columns go to the cluster's exchange record as
//     64-bit {step tag, value} words; every workgroup reads the others' and adds in cluster
//     order (two records alternate: nobody can post step u + 2 before everybody has read u);
//   - softmax and dz = p - onehot with 16 lanes per sample, to LDS.  (expf and logf as in the
//     layer engine: with __expf and __logf, 1 % faster, the entries of dz add up to more, and
//     with features of one sign models come out 1.4 times as far from 64 bits: 600 clients x 40
//     columns, mini-batch 8, 12 rounds 1.3e-5 against 1.8e-5 of the norm);
//   - g^T = sum_b x_b dz_b^T, 16 columns by 16 classes: the accumulator's layout is that of W, so
//     W -= eta g and U += g are applied in place.  Its operand is the mini-batch's block turned round, which a
//     wave does through its own two kilobytes of LDS, without a barrier.  The block's registers then take
//     the next recursion's rows, or, where there are registers for two sets, those were asked for ahead of
//     the softmax.
// Samples beyond the mini-batch (BC is a compile-time bound) repeat its last row with dz = 0.
//
// What bounds it: with wide rows the rows from memory (128 clients x 32 x 12 KB: 10 us of a recursion at
// the rate of a large copy, 12.7 measured; 24 us per round for the first rows and the replicas), with narrow
// ones the chain logits - exchange - softmax.  The form with a column per lane below, whose dot products
// the vector unit did, took 15 us and 25.  Per recursion, before and now: 128 clients x 3,072 columns, mini-batch 32:
// 16.8 -> 14.9 us; 40 clients x 784, 32: 9.0 -> 6.2; 1 client x 16, 64: 14.3 -> 3.3; 128 clients x 3,072, 64: 67 -> 37 us.
// U in LDS: with it in registers the form with twelve blocks and 32 samples spilled, and what it
// read back waited behind the rows in flight (17.5 us).
//
// All workgroups of a cluster must be resident together: the launcher never puts more on an
// XCD than it has compute units (cluster_plan.h).  The wait is bounded and raises an error flag
// instead of hanging (every workgroup still runs to the end).
#include "aet_device.h"
#include "aet_internal.h"
#include "cluster_plan.h"
#include "cluster_post.h"
#include "softmax_batch_form.h"

namespace aet {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;

constexpr int kSbWaves = 8;
constexpr int kSbThreads = 64 * kSbWaves;
static_assert(kSbThreads == kSbRun && kSbWaves == 8, "softmax_batch_form");
constexpr int kSbClasses = 10;         // the forward part sums two samples' classes as 20 values
constexpr int kSbC = 12;               // class slots of an exchange record
static_assert(kSbClasses <= kSbC && kSbC == 12, "softmax_batch_record_words");
constexpr int kSbQ = 3;                // groups of four class rows, of the form with a column per lane
static_assert(4 * kSbQ == kSbC && 2 * kSbClasses == 20, "five registers of four sums hold two samples' classes");
constexpr int kSbLanePS = 13;          // ... and its LDS stride of a sample's partial logits
constexpr int kSbMaxHF = 6;            // workgroups of a cluster, at most
static_assert(kSbMaxHF <= kClusterMax, "a place for every workgroup");
constexpr int kSbMaxD = kSbMaxHF * kSbThreads;
constexpr int kSbMaxB = 64;
constexpr int kSbPS = 20;              // LDS stride of a sample's partial logits

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

// What the wave's lanes wrote to LDS is there for all of them afterwards, and what they read before may be
// written again.  No instruction: a wave's LDS accesses are carried out in order, this keeps the compiler's.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
}

typedef f4 __attribute__((aligned(4))) f4_any;   // four floats at any place
typedef const f4_any __attribute__((address_space(1))) *gcf4_ptr;
typedef f4_any __attribute__((address_space(1))) *gf4_ptr;

// NC: a wave has up to 4 NC blocks of 16 columns; BC: room for samples; COLS: what is known about D
enum { D_FULL, D_ANY, D_TINY };   // every wave has all its blocks, all columns of them exist; 4 and more; fewer
template <int NC, int BC, int COLS>
__global__ void __launch_bounds__(kSbThreads, 1)
k_softmax_batch_round(const RoundParams *__restrict__ rp, int nhere, int rec0, const float *Wg, int D, int C,
                      int HF, int Br, int rec_words, u64 *__restrict__ xrec, u64 *__restrict__ places, int skew, uint32_t tag0, int *__restrict__ errflag) {
    constexpr int T = kSbThreads, NW = kSbWaves;
    constexpr int NB = 4 * NC;                  // 16-column blocks per wave
    constexpr int MT = (BC + 15) / 16;          // tiles of 16 samples
    constexpr int NK = BC / 4;                  // steps of four samples
    constexpr int NE = (BC * 16 + T - 1) / T;   // (sample, class) elements per thread
    constexpr int NX = BC <= 32 ? 2 : 1;        // blocks turned round at a time
    constexpr bool DB = MT * NC <= 2;           // two sets of rows in registers
    constexpr bool ULDS = NC > 1;               // U in LDS: beside two or three runs of rows it would spill
    constexpr bool FULL = COLS == D_FULL;
    constexpr int PW = NX * BC * 16 > BC * kSbPS ? NX * BC * 16 : BC * kSbPS;
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
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float invB = 1.0f / (float)Br;

    // a wave's partial logits; between the recursions' forward parts its place to turn blocks round
    __shared__ __attribute__((aligned(16))) float part[NW][PW];
    __shared__ float dzs[BC * 16];
    __shared__ float bs[16], Ubs[16];
    __shared__ int labs[BC];
    __shared__ float lred[NW];

    __shared__ __attribute__((aligned(16))) f4 Us[ULDS ? NB * T : 1];

    // The blocks in equal shares: workgroups, then waves.  Lane (li, lg): class li, columns 4 lg .. 4 lg + 3 of
    // every block.  Where those end beyond the last column the lane takes the row's last four instead and
    // keeps zero weights for the ones that are not its own (column() and own() say which).
    const int blocks = (D + 15) >> 4, per_wg = (blocks + HF - 1) / HF, per_wave = (per_wg + NW - 1) / NW;
    const int block0 = h * per_wg + wave * per_wave;
    const int nb = FULL ? NB : max(0, min(per_wave, min(blocks, (h + 1) * per_wg) - block0));
    const int col0 = 16 * block0;
    auto column = [&](int j, int r, int last) {
        const int c = col0 + 16 * j + 4 * lg;
        return FULL ? c + r : COLS == D_ANY ? min(c, last - 4) + r : min(c + r, last - 1);
    };
    auto own = [&](int j, int r, int last) { return FULL || (column(j, r, last) >= col0 + 16 * j + 4 * lg + (COLS == D_TINY ? r : 0)); };
    f4 W[NB], U[ULDS ? 1 : NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (ULDS) Us[j * T + tid] = f4{0.f, 0.f, 0.f, 0.f};
        else U[ULDS ? 0 : j] = f4{0.f, 0.f, 0.f, 0.f};
        W[j] = f4{0.f, 0.f, 0.f, 0.f};
        if (j < nb && li < C) {
            int last = D;
            asm volatile("" : "+s"(last));
            if (COLS == D_TINY) {
#pragma unroll
                for (int r = 0; r < 4; ++r) W[j][r] = W0[(int64_t)li * D + column(j, r, last)];
            } else {
                W[j] = *(gcf4_ptr)(W0 + (int64_t)li * D + column(j, 0, last));
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) W[j][r] = own(j, r, last) ? W[j][r] : 0.f;
        }
    }
    if (tid < 16) {
        bs[tid] = tid < C ? W0[(int64_t)C * D + tid] : 0.f;
        Ubs[tid] = 0.f;
    }

    // row addresses and labels of a recursion: lane b for sample b; then, for every tile, that of sample li
    int labn = 0;
    gcf_ptr row[MT];
    auto next_rows = [&](int u) {
        const uint32_t r = sample_row(p.key, (uint64_t)(p.q0 + (int64_t)min(u, p.m - 1) * Br + min(lane, Br - 1)), p.n_samples);
        labn = yg[r];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const uint32_t rt = (uint32_t)__shfl((int)r, min(16 * t + li, BC - 1), 64);
            row[t] = as_global(p.X) + (int64_t)rt * D;
        }
    };
    // x[t][j]: sample 16 t + li, columns 4 lg .. 4 lg + 3 of block j
    f4 x[DB ? 2 : 1][MT][NB];
    auto load_block = [&](f4 (&x)[MT][NB], int j) {
        if (j >= nb) return;
        int last = D;
        if (!FULL) asm volatile("" : "+s"(last));   // where the columns are is worked out anew: kept in registers, it would spill
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            if (COLS == D_TINY) {
#pragma unroll
                for (int r = 0; r < 4; ++r) x[t][j][r] = row[t][column(j, r, last)];
            } else {
                x[t][j] = *(gcf4_ptr)(row[t] + column(j, 0, last));
            }
        }
    };
    float loss_acc = 0.f;
    u64 *rec_base = xrec + (int64_t)(rec0 + a) * rec_words;
    bool dead = false, one_xcd = false;

    if (p.m > 0) {
        next_rows(0);
#pragma unroll
        for (int j = 0; j < NB; ++j) load_block(x[0], j);
        if (wave == 0 && lane < BC) labs[lane] = labn;
        if (HF > 1) one_xcd = cluster_on_one_xcd(places, h, HF, tag0, errflag, &dead);
    }
    // x: this recursion's rows; xn: where the next one's go (the same, block by block, where there is one set)
    auto recursion = [&](int u, f4 (&x)[MT][NB], f4 (&xn)[MT][NB]) {
        // ---- partial logits of the own columns: rows samples, columns classes --------------------------
        {
            f4 acc[MT][2];
#pragma unroll
            for (int t = 0; t < MT; ++t) acc[t][0] = acc[t][1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (j < nb) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int t = 0; t < MT; ++t)
                            acc[t][r & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t][j][r], W[j][r], acc[t][r & 1], 0, 0, 0);
                }
            }
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (BC % 16 == 0 || 16 * t + 4 * lg + r < BC) part[wave][(16 * t + 4 * lg + r) * kSbPS + li] = acc[t][0][r] + acc[t][1][r];
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
        if (DB && u + 1 < p.m) {   // behind the polls, which would wait for them
#pragma unroll
            for (int j = 0; j < NB; ++j) load_block(xn, j);
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
            if (b < BC) dzs[b * 16 + o] = live ? expf(zz - lse) - (o == lab ? 1.f : 0.f) : 0.f;
        }
        __syncthreads();
        if (wave == 0 && lane < BC) labs[lane] = labn;
        if (wave == 1 && lane < kSbC) {   // bias (every workgroup keeps a copy)
            float s = 0.f;
#pragma unroll
            for (int b = 0; b < BC; b += 4)
                s += (dzs[b * 16 + lane] + dzs[(b + 1) * 16 + lane]) + (dzs[(b + 2) * 16 + lane] + dzs[(b + 3) * 16 + lane]);
            s *= invB;
            bs[lane] -= p.eta * s;
            Ubs[lane] += s;
        }
        // ---- g, update, the next recursion's rows: rows columns, columns classes ------------------------
        float dz[NK];
#pragma unroll
        for (int k = 0; k < NK; ++k) dz[k] = dzs[(4 * k + lg) * 16 + li];
        float *const turn = part[wave];
        int last = D;
        if (!FULL) asm volatile("" : "+s"(last));
#pragma unroll
        for (int j0 = 0; j0 < NB; j0 += NX) {
            if (j0 < nb) {
                f4 u_old[NX], G[NX];
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    if (ULDS) u_old[n] = Us[(j0 + n) * T + tid];
                    G[n] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < MT; ++t)
                        if (BC % 16 == 0 || li < BC) *reinterpret_cast<f4 *>(turn + n * BC * 16 + (16 * t + li) * 16 + 4 * lg) = x[t][j0 + n];
                }
                wave_lds_order();
                if (!DB && u + 1 < p.m) {
#pragma unroll
                    for (int n = 0; n < NX; ++n) load_block(x, j0 + n);
                }
#pragma unroll
                for (int k = 0; k < NK; ++k)
#pragma unroll
                    for (int n = 0; n < NX; ++n)
                        G[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(turn[n * BC * 16 + (4 * k + lg) * 16 + li], dz[k], G[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    const int j = j0 + n;
                    if (FULL || col0 + 16 * j + 16 <= last) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) W[j][r] -= p.eta * (G[n][r] * invB);
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) W[j][r] -= (j < nb && own(j, r, last) ? p.eta : 0.f) * (G[n][r] * invB);
                    }
                    if (ULDS) Us[j * T + tid] = u_old[n] + G[n] * invB;
                    else U[ULDS ? 0 : j] += G[n] * invB;
                }
            }
            wave_lds_order();   // the next block, or the next recursion's logits, go to the same place
            __builtin_amdgcn_sched_barrier(0);   // (registers: the loop does not spill)
        }
    };
    if (DB) {
        for (int u = 0; u < p.m; u += 2) {
            recursion(u, x[0], x[DB ? 1 : 0]);
            if (u + 1 < p.m) recursion(u + 1, x[DB ? 1 : 0], x[0]);
        }
    } else {
        for (int u = 0; u < p.m; ++u) recursion(u, x[0], x[0]);
    }

    if (li < C) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const f4 uj = ULDS ? Us[j * T + tid] : U[ULDS ? 0 : j];
            int last = D;
            asm volatile("" : "+s"(last));
            if (FULL || (j < nb && col0 + 16 * j + 16 <= last)) {
                const int64_t c = (int64_t)li * D + col0 + 16 * j + 4 * lg;
                *(gf4_ptr)(Wc + c) = W[j];
                *(gf4_ptr)(Uc + c) = uj;
            } else if (j < nb) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (own(j, r, last)) {
                        const int64_t c = (int64_t)li * D + column(j, r, last);
                        Wc[c] = W[j][r];
                        Uc[c] = uj[r];
                    }
            }
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

// ---- the same round with a column per lane, for mini-batches that leave most of a matrix tile empty -------
// Thread t owns columns t, t + 512, ... of the run for every class row of W and U and, one recursion at a
// time, of the mini-batch.  Partial logits: dot products over the thread's columns, two samples (20
// sums) at a time folded over the wave with lane swaps and DPP steps.  g^T = sum_b x_b dz_b^T as 4 x 4 outer
// products on the matrix cores (see k_softmax_round: the lane's own column is the B operand); when a
// column is done its registers take the next recursion's rows.  Samples beyond the mini-batch repeat its
// last row with dz = 0; columns beyond D read the row's last column with weights of zero.
template <int NC, int BC>
__global__ void __launch_bounds__(kSbThreads, 1)
k_softmax_batch_lanes(const RoundParams *__restrict__ rp, int nhere, int rec0, const float *Wg, int D, int C,
                      int HF, int Br, int rec_words, u64 *__restrict__ xrec, u64 *__restrict__ places, int skew, uint32_t tag0, int *__restrict__ errflag) {
    constexpr int Q = kSbQ, T = kSbThreads, NW = kSbWaves;
    static_assert(BC <= 32, "the samples' logits are collected before one store");
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

    __shared__ float part[NW][BC * kSbLanePS];
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
        {
            float res[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < BC / 2; ++c) {
                float s[2 * kSbClasses];
#pragma unroll
                for (int i = 0; i < 2 * kSbClasses; ++i) {
                    const int o = i % kSbClasses, b = 2 * c + i / kSbClasses;
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
            if (li < BC / 2) {
                const int row = lane >> 4, o0 = ((row & 1) << 1) | (row >> 1);
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) {
                    const int i = 4 * kk + o0, second = i >= kSbClasses ? 1 : 0;
                    part[wave][(2 * li + second) * kSbLanePS + i - kSbClasses * second] = res[kk];
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
                for (int w = 0; w < NW; ++w) z[e] += part[w][b * kSbLanePS + o];
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

template <class Kernel>
static hipError_t sb_launch(Kernel kernel, hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int resident, const float *Wg,
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
        kernel<<<grid, kSbThreads, 0, s>>>(dp + a0, here, a0, Wg, D, C, HF, B, words, xrec, places, g_xcd_skew, tag0, errflag);
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
    const SoftmaxBatchForm f = softmax_batch_form(D, B, nact, cus, xcds);
    const int resident = resident_clusters(cus, xcds, f.workgroups);
    const auto launch = [&](auto kernel) {
        return sb_launch(kernel, s, prof, dp, nact, resident, Wg, D, C, B, f.workgroups, n_clients, scratch, tag0);
    };
    if (f.lanes) return launch(f.runs == 1 ? k_softmax_batch_lanes<1, 8> : f.samples == 8 ? k_softmax_batch_lanes<3, 8> : k_softmax_batch_lanes<3, 16>);
    // (what has fewer than four columns has one run of them)
#define AET_SB(nc, bc) return launch(f.columns == D_FULL ? k_softmax_batch_round<nc, bc, D_FULL> : k_softmax_batch_round<nc, bc, D_ANY>)
#define AET_SB_ONE(bc) return launch(f.columns == D_FULL ? k_softmax_batch_round<1, bc, D_FULL> : f.columns == D_ANY ? k_softmax_batch_round<1, bc, D_ANY> : k_softmax_batch_round<1, bc, D_TINY>)
    switch (f.samples + f.runs) {
        case 8 + 1: AET_SB_ONE(8);
        case 8 + 2: AET_SB(2, 8);
        case 16 + 1: AET_SB_ONE(16);
        case 16 + 2: AET_SB(2, 16);
        case 16 + 3: AET_SB(3, 16);
        case 32 + 1: AET_SB_ONE(32);
        case 32 + 2: AET_SB(2, 32);
        case 32 + 3: AET_SB(3, 32);
        case 64 + 1: AET_SB_ONE(64);
        case 64 + 2: AET_SB(2, 64);
    }
    return hipErrorInvalidValue;
#undef AET_SB
#undef AET_SB_ONE
}

}  // namespace aet
