// Fused local round for dense-ReLU-dense models (D -> H -> C, mini-batch up to 64).
//
// One launch runs the whole round (Algorithm 2, MainComputeNode: all s_i/B recursions) of
// every active client.  A client is handled by a cluster of G = ceil(H/16) workgroups; workgroup
// g owns hidden units 16g..16g+15: its slice of the first layer (16 x D weights, 16
// biases) and of the second layer (C x 16 weights), together with the matching slices of
// U, stay in registers / LDS for the whole round, so the per-recursion traffic is the
// mini-batch rows plus one small exchange.
//
// Per recursion:
//   - each of the 8 waves owns a contiguous eighth of the input columns: it has loaded its
//     part of the B sampled rows into registers during the recursions before (two ahead
//     where the registers hold two mini-batches), in the A-operand layout of the forward product;
//   - z1 = X W1^T on the matrix cores (fp32 MFMA 16x16x4) straight from those registers,
//     partial over the wave's columns, summed over the waves through LDS; h = relu(z1 + b1);
//     the rows are then parked in LDS for the backward product (no workgroup barrier:
//     nobody else touches those columns);
//   - the partial logits of the 16 own units are written to the client's exchange record
//     as 64-bit {step tag, value} words; every workgroup polls the G records until all
//     tags show the current step, which gives the logits without a separate barrier or
//     fence (each word validates itself; two records alternate so a fast workgroup never
//     overwrites what a slow one still has to read);
//   - softmax / d logits with 16 lanes per sample; dh = (d logits W2) * 1[h > 0] and
//     dW2 = d logits^T h as small MFMA products;
//   - dW1^T = X^T dh on the matrix cores: the accumulator tile has exactly the register
//     layout the forward pass uses as its B operand, so  w <- w - eta g  and  U <- U + g
//     are applied to the register-resident slice in place (g never exists in memory).
//
// Wide inputs (more than 32 column tiles) with few enough clients take two workgroups per
// unit group: each owns half of the input columns (its half of the W1 / U1 slice, of the
// sampled rows, of the forward and of the backward product); the two add their partial
// hidden sums through a second tagged exchange and then compute the same h, logits and
// second-layer updates side by side.  16 clients x 8 unit groups then occupy all 256
// compute units instead of 128.
//
// Widths and mini-batches that do not fill the 16 x 16 tiles are padded: hidden units beyond H
// have zero weights, samples beyond the mini-batch repeat its last row with d logits of zero
// (never a row that was not drawn: it could hold a value that is not finite).  Mini-batches of
// 33 .. 64 are two steps of 32 samples, with one update: 4 clients, 784 -> 100, 64 samples 29 -> 12 us per recursion
// (five launches of the layer-by-layer engine before).
//
// What bounds it: the chain of one recursion, forward product - sum over the waves - (pair exchange) - logits -
// exchange - softmax - d(hidden) - backward product, four workgroup barriers long; the two large products are a
// third of it at 784 columns, a tenth at 60.  So the rows are on their way for a whole recursion, which row comes
// next is worked out by one wave while others have the small products, exchanges take no address arithmetic, and the
// operands of a small product that are there before its barrier are read ahead of it.  Per job, with the rows one
// recursion ahead and pieces of odd rows in up to four loads, and now: 16 clients, 784 -> 128, B = 32, 50 rounds 7.28 ->
// 6.73 ms; 12, 784 -> 100, B = 20 2.00 -> 1.83; 40, 523 -> 240, B = 32 0.75 -> 0.58; 16, 435 -> 34, B = 32 2.88 -> 1.76;
// 4, 70 -> 239, B = 32 0.48 -> 0.35; 30, 30 -> 16, B = 4 0.66 -> 0.55.  Measured and dropped: everything between the two
// large products in one wave for 16 samples, four values a lane, with two barriers instead of four: 7.68 ms (a
// single wave issues an instruction every eight clocks or so, and there are four times as many); all row loads ahead of
// the backward product: 7.55; two mini-batches ahead with seven tiles a wave: 40 clients, 896 -> 256 3.14 -> 3.47.
//
// All workgroups of a client must be resident together: the launcher never puts more
// working workgroups on an XCD than it holds (cluster_plan.h; 1 per compute unit with this
// LDS footprint).  The poll is bounded: on expiry an error flag is raised and every workgroup
// still runs to the end, so the grid always drains.
#include <type_traits>

#include "aet_device.h"
#include "aet_internal.h"
#include "cluster_plan.h"
#include "cluster_post.h"

namespace aet {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // where rows begin at any float
typedef int i2 __attribute__((ext_vector_type(2)));

constexpr int kMlpWaves = 8;         // waves per workgroup (2 per SIMD)
constexpr int kMlpThreads = 64 * kMlpWaves;
constexpr int kMlpMaxTPW = 7;        // K tiles (of 16) per wave  => D <= 16*8*7 = 896
constexpr int kMlpMaxG = 16;         // workgroups per client
constexpr int kMlpRec = 512;         // 64-bit words per exchange record (B*16 <= 512)
static_assert(kMlpRec % kLineWords == 0, "whole lines");
constexpr int kMlpPair = 512;        // 64-bit words per pair record (B*16 <= 512)
static_assert(kMlpPair % kLineWords == 0, "whole lines");
constexpr int kRowsWave = 5;         // the wave that works out which rows come next
constexpr int kMlpHalfTPW = 4;       // K tiles per wave when two workgroups share the columns

__device__ __forceinline__ f4 mfma16(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// sum / max over the 16 lanes of one sample (lanes 16k .. 16k+15 of the wave), with the
// data-parallel-primitive lane permutations inside a row: neighbours in a quad, the other
// pair of the quad, the mirrored half row, the mirrored row
#define AET_ROW_STEP(op, v, ctrl) \
    v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xF, 0xF, true)))
__device__ __forceinline__ float row16_add(float a, float b) { return a + b; }
__device__ __forceinline__ float row16_sum(float v) {
    AET_ROW_STEP(row16_add, v, 0xB1);
    AET_ROW_STEP(row16_add, v, 0x4E);
    AET_ROW_STEP(row16_add, v, 0x141);
    AET_ROW_STEP(row16_add, v, 0x140);
    return v;
}
__device__ __forceinline__ float row16_max(float v) {
    AET_ROW_STEP(fmaxf, v, 0xB1);
    AET_ROW_STEP(fmaxf, v, 0x4E);
    AET_ROW_STEP(fmaxf, v, 0x141);
    AET_ROW_STEP(fmaxf, v, 0x140);
    return v;
}
#undef AET_ROW_STEP

// sum over the 64 lanes, every lane gets it (gfx950 lane swaps: halves, then rows, then the
// in-row steps)
__device__ __forceinline__ float fold_rows(float v) {   // sum of the 4 rows, lane by lane
    const auto a = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, v), __builtin_bit_cast(int, v), false, false);
    v = __builtin_bit_cast(float, (int)a[0]) + __builtin_bit_cast(float, (int)a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, v), __builtin_bit_cast(int, v), false, false);
    return __builtin_bit_cast(float, (int)b[0]) + __builtin_bit_cast(float, (int)b[1]);
}
// column sums of a [B][16] LDS array: lane (c = lane % 16, q = lane / 16) adds the rows
// q, q + 4, ... of column c, then the four row groups are folded
template <int B>
__device__ __forceinline__ float col_sum16(const float *a, int lane) {
    float s = 0.f;
#pragma unroll
    for (int b = lane >> 4; b < B; b += 4) s += a[b * 16 + (lane & 15)];
    return fold_rows(s);
}

// FAST: D is a multiple of 16, so every row piece is one aligned 16-byte load.
// NBT: batch tiles of 16 samples; TPW: K-tile slots of a wave (a wave that owns fewer tiles
// skips the rest with scalar branches).
// The round records of one launch travel in the kernel arguments: no staging copy, no
// buffer whose reuse would have to be fenced with events.
constexpr int kMlpPack = 48;
struct MlpPack {
    RoundParams p[kMlpPack];
};

// FULL: every wave owns TPW real tiles (D = 16 * 8 * TPW): no pad tiles, loads unguarded.
// HF = 2: two workgroups per unit group, each owning one half of the input columns (its
// half of the W1 / U1 slice, of the sampled rows and of both big products); they add their
// partial hidden sums through a second tagged exchange (pair records `prec`) and from
// there on compute the same numbers side by side; half 0 posts the logits and stores the
// second layer at the end.
// PAD: the width or the mini-batch does not fill its tiles.
// SUB = 2: mini-batches of 33 .. 64 in two steps, samples 0 .. 31 and 32 .., on the same weights: the first step's
// gradient sums are kept (in registers: where the second one's products start from), the second one's update takes both.
template <int NBT, int TPW, bool FAST, bool FULL, int HF, bool PAD, int SUB>
__global__ void __launch_bounds__(kMlpThreads, 1)
k_mlp_round(const MlpPack pack, int nhere, int rec0, const float *Wg,
            int D, int H, int C, int G, int Brun, unsigned long long *__restrict__ xrec,
            unsigned long long *__restrict__ prec, unsigned long long *__restrict__ places, int skew,
            uint32_t tag0, int *__restrict__ errflag, unsigned long long *claims, int first) {
    constexpr int B = 16 * NBT;
    static_assert(SUB == 1 || (PAD && NBT == 2), "two steps of 32 samples, of which the second may be short");
    const int Br = PAD ? Brun : B;   // samples of the mini-batch
    extern __shared__ float smem[];
    // workgroup -> (client, unit group, half): consecutive workgroup ids go round the 8 XCDs,
    // so the workgroups of one client get ids that land on the same XCD and share its L2
    // for the mini-batch rows and the exchanges.  Which XCD begins differs from queue to queue: where the launch has
    // to know (others are beside it), client 0 is on XCD `first` and the workgroup asks where it is.  (The forms of
    // one step a recursion do not ask: 784 -> 100, B = 20 1,908 -> 1,972 us a job, other registers and spills in the whole kernel.)
    const int xcd = SUB == 2 ? opaque_scalar((first < 0 ? (int)blockIdx.x : xcc_id() - first) & 7) : (int)blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int a = xcd + 8 * (slot / (G * HF));  // index into this launch's records
    const int g = (slot % (G * HF)) / HF, hf = slot % HF;
    if (a >= nhere) return;
    if (places) places += (int64_t)(rec0 + a) * kPlaces;
    if (SUB == 1 || first < 0) cluster_announce(places, g * HF + hf, tag0, skew);
    else if (!cluster_claim(claims + (int64_t)(rec0 + a) * kPlaces, g * HF + hf, tag0, skew, smem)) return;
    const RoundParams p = pack.p[a];
    const gcf_ptr Xg = as_global(p.X);
    const gci_ptr yg = as_global(p.y);
    const gf_ptr Wc = as_global(p.W), Uc = as_global(p.U);

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    // the wave index as a scalar, so that everything derived from it (tile counts, column
    // offsets, branches on them) stays in scalar registers and scalar branches
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // real K tiles (of 16 columns) of this half, and the first of them
    const int KTall = (D + 15) >> 4, KH = (KTall + HF - 1) / HF;
    const int tbase = hf * KH;
    const int KT = min(KH, KTall - tbase);
    constexpr int ld = 16 * kMlpWaves * TPW + 4;  // LDS row stride: all tiles + 4 floats of skew
    constexpr int NI = NBT * TPW;             // float4 loads per lane and mini-batch
    // the KT tiles are dealt out evenly: wave w owns nt consecutive tiles from t0 on, the
    // first KT % 8 waves one more than the others (waves w and w + 4 share a SIMD and its
    // matrix core: dealt this way the four SIMDs differ by one tile at most).  A wave has
    // TPW tile slots in registers and in the staged rows; slots beyond nt are skipped.
    const int tb = KT / kMlpWaves, te = KT % kMlpWaves;
    const int nt = tb + (wave < te ? 1 : 0);
    const int t0 = wave * tb + min(wave, te);
    const int col0 = 16 * TPW * wave;         // first column of the wave's slots in the staged rows
    const int gcol0 = 16 * (tbase + t0);      // first own column in the sample / weight rows

    // the small arrays come first so that their addresses fit the 16-bit offset field of
    // the LDS instructions; the big mini-batch tile follows
    float *red = smem;                // [waves][B][16]
    float *hs = red + kMlpWaves * B * 16;  // [B][16]
    float *dhs = hs + B * 16;         // [B][16]
    float *zs = dhs + B * 16;         // [B][16]  d logits (columns >= C stay 0)
    float *W2s = zs + B * 16;         // [16][16] (o, j)
    float *U2s = W2s + 256;
    float *b1s = U2s + 256;           // [16]
    float *Ub1s = b1s + 16;
    float *b2s = Ub1s + 16;
    float *Ub2s = b2s + 16;
    float *lossb = Ub2s + 16;         // [B]
    float *lossacc = lossb + B;       // [16], entry 0: the round's loss sum; 1: not zero: the cluster spans XCDs
    int *labs = reinterpret_cast<int *>(lossacc + 16);  // [B]
    uint32_t *rows = reinterpret_cast<uint32_t *>(labs + B); // [B]  the rows of recursion u + AHEAD
    float *Xs = reinterpret_cast<float *>(rows + B); // [B][ld]

    const int64_t b1_off = (int64_t)H * D, w2_off = b1_off + H, b2_off = w2_off + (int64_t)C * H;
    const float invB = 1.0f / (float)Br;

    // The mini-batch travels global -> registers -> matrix core / LDS in the A-operand layout
    // of the forward product: lane (li, lg) holds, for batch tile bt and K tile tt, the four
    // values x[16*bt + li][col0 + 16*tt + 4*lg .. +3], one 16-byte load.  Where D is no multiple of 16
    // (not FAST) the last tile's pieces can reach beyond the row's end: such a piece is loaded as far
    // back as that takes, and put right (tail_piece) when it is used, so that a load has no branches and
    // nothing waits for it early.  (As up to four guarded 4-byte loads a piece: 40 clients, 523 -> 240, B = 32,
    // 28.4 K clocks a recursion, 15.7 K of them in the step that issues the loads.)
    const bool narrow = TPW == 2 && D < 4;        // a row is shorter than a piece: value by value
    const int tail_tt = !FAST && !narrow && (D & 15) && nt > 0 && tbase + t0 + nt == KTall ? nt - 1 : -1;
    const int tail_by = max(0, gcol0 + 16 * tail_tt + 4 * lg - (D - 4));   // columns back
    const gcf_ptr lane_src = Xg + gcol0 + 4 * lg;
    // rowp: the lane's piece of tile 0 of its row, lane_src + row * D
    auto load_piece = [&](gcf_ptr rowp, int tt, int nt, int tail_tt) -> f4 {
        f4 x = {0.f, 0.f, 0.f, 0.f};
        if (FULL || tt < nt) {
            const gcf_ptr src = rowp + 16 * tt;
            if constexpr (FAST) {
                x = *reinterpret_cast<const f4 __attribute__((address_space(1))) *>(src);
            } else if (narrow) {
#pragma unroll
                for (int r = 0; r < 3; ++r)
                    if (4 * lg + r < D) x[r] = src[r];
            } else {
                x = *reinterpret_cast<const f4u __attribute__((address_space(1))) *>(src - (tt == tail_tt ? tail_by : 0));
            }
        }
        return x;
    };
    auto tail_piece = [&](f4 &x) {
        f4 t = tail_by & 1 ? f4{x[1], x[2], x[3], 0.f} : x;
        t = tail_by & 2 ? f4{t[2], t[3], 0.f, 0.f} : t;
        x = tail_by & ~3 ? f4{0.f, 0.f, 0.f, 0.f} : t;
    };

    // ---- adopt the global model (server form) or go on from the own replica (Wg == NULL:
    // peer-to-peer form): own slice into registers / LDS; U = 0 -------------------------
    if (!Wg) Wg = p.W;
    // own unit of this lane in the first layer; the last group may have units that do not exist:
    // they carry zero weights, so h, dh and every update of theirs is zero
    const bool unit_ok = !PAD || 16 * g + li < H;
    const int unit = unit_ok ? 16 * g + li : 0;
    f4 W1r[TPW], U1r[TPW];
#pragma unroll
    for (int tt = 0; tt < TPW; ++tt) {
        f4 w = load_piece(as_global(Wg) + (int64_t)unit * D + gcol0 + 4 * lg, tt, nt, tail_tt);
        if (tt == tail_tt) tail_piece(w);
        W1r[tt] = unit_ok ? w : f4{0.f, 0.f, 0.f, 0.f};
        U1r[tt] = f4{0.f, 0.f, 0.f, 0.f};
    }
    {
        const int o = tid >> 4, j = tid & 15;  // threads 0..255 = 16 x 16
        if (tid < 256) {
            W2s[tid] = (o < C && (!PAD || 16 * g + j < H)) ? Wg[w2_off + (int64_t)o * H + 16 * g + j] : 0.f;
            U2s[tid] = 0.f;
        }
        for (int i = tid; i < B * 16; i += kMlpThreads) zs[i] = 0.f;
        if (tid < 16) {
            b1s[tid] = !PAD || 16 * g + tid < H ? Wg[b1_off + 16 * g + tid] : 0.f;
            Ub1s[tid] = 0.f;
            b2s[tid] = (tid < C) ? Wg[b2_off + tid] : 0.f;
            Ub2s[tid] = 0.f;
            lossacc[tid] = 0.f;
        }
    }
    __syncthreads();
    // Rows of the next recursions in registers, AHEAD sets that take turns (Algorithm 2, sampling step; the
    // indices are a counter hash, so they are known ahead).  The loads of a recursion are issued in its backward product, the
    // last step: with one set the next forward product, the first step, waits for them for 1 - 2 K clocks; with
    // two they have a whole recursion.
    constexpr int AHEAD = TPW <= kMlpHalfTPW ? 2 : 1;
    f4 xreg[AHEAD][NBT][TPW];
    int lab_next = 0, lab_ahead = 0;   // labels of recursions u + 1 and u + AHEAD (of the wave that sees to the rows)
    using Step = typename std::conditional<SUB == 2, uint32_t, int>::type;
    const Step steps = (Step)cluster_steps(p.m, SUB);
    auto rows_of = [&](Step u) -> uint32_t {   // of step u
        const int64_t from = SUB == 1 ? (int64_t)u * Br : (int64_t)(u >> 1) * Br;
        const int b = SUB == 1 ? lane : B * (u & 1) + lane;
        return lane < B ? sample_row(p.key, (uint64_t)(p.q0 + from + min(b, Br - 1)), p.n_samples) : 0u;
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
#pragma unroll
        for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) xreg[k][bt][tt] = f4{0.f, 0.f, 0.f, 0.f};
        if ((Step)k < steps) {
            const uint32_t rowv = rows_of(k);
            if (wave == kRowsWave && lane < B) {
                const int lab = yg[rowv];
                if (k == 0) labs[lane] = lab;
                else lab_next = lab;
            }
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) {
                const gcf_ptr rowp = lane_src + (int64_t)__shfl(rowv, 16 * bt + li) * D;
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) xreg[k][bt][tt] = load_piece(rowp, tt, nt, tail_tt);
            }
        }
    }
    // logit records [step parity][unit group][sample][class]
    const ClusterWords rec(xrec, (int64_t)(rec0 + a) * 2 * kMlpMaxG * kMlpRec, 2 * kMlpMaxG * kMlpRec);
    // pair records [client][unit group][step parity][half][B * 16]
    const ClusterWords pair(prec, ((int64_t)(rec0 + a) * kMlpMaxG + g) * 4 * kMlpPair, 4 * kMlpPair);
    int dead = 0;  // not 0: the poll expired: keep going, the host will see the flag (the same for the whole wave)
    {
        bool gone = false;
        // the same answer in all waves (one whose wait expired says no): there are barriers that hang on it
        if (!cluster_on_one_xcd(places, g * HF + hf, G * HF, tag0, errflag, &gone)) lossacc[1] = 1.f;
        dead = __any(gone);
    }
    __syncthreads();
    const bool one_xcd = __builtin_amdgcn_readfirstlane(lossacc[1] == 0.f);

    // the first of two steps' sums
    f4 Gk[SUB == 2 ? TPW : 1], dW2k = {0.f, 0.f, 0.f, 0.f};
    float db1k = 0.f, db2k = 0.f;
    // x: this step's rows; their registers take the rows of step u + AHEAD (a step is a recursion, or, SUB = 2, half
    // of one: part 0 or 1)
    auto recursion = [&](Step u, const int half, f4 (&x)[NBT][TPW], const auto same) __attribute__((always_inline)) {   // same: whether the words stay in the L2 of one XCD
        const int ntile = opaque_scalar(nt), tail = opaque_scalar(tail_tt);
        auto park_rows = [&]() {
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt)
                    if (FULL || tt < ntile)
                        *reinterpret_cast<f4 *>(Xs + (16 * bt + li) * ld + col0 + 16 * tt + 4 * lg) = x[bt][tt];
        };
        if constexpr (!FAST) {
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt)
                if (tt == tail) {
#pragma unroll
                    for (int bt = 0; bt < NBT; ++bt) tail_piece(x[bt][tt]);
                }
        }
        // ---- z1 partial sums on the matrix cores ----------------------------------------
        {
            f4 acc[NBT];
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) acc[bt] = f4{0.f, 0.f, 0.f, 0.f};
            // The rows come straight from the registers they were loaded into; empty slots are
            // skipped (us a job with the last slot skipped, and with every one: 16 clients, 784 -> 128 6,980
            // and 6,950, multiplying zeros 7,110; 16, 435 -> 34 2,000 and 1,860, 2,080; 30, 30 -> 16 625 and 598, 624).
            // Units are the product's rows and samples its columns here and in the two small products: a lane
            // has four neighbouring units or classes of one sample, one 16-byte piece.
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) {
                if (!FULL && tt >= ntile) break;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int bt = 0; bt < NBT; ++bt) acc[bt] = mfma16(W1r[tt][r], x[bt][tt][r], acc[bt]);
            }
            // the backward product needs the rows transposed: park them in LDS (this wave's
            // columns only, so no barrier; the writes drain while the logits are exchanged).
            // With two workgroups per unit group they are parked between the post and the
            // poll of the pair exchange instead.
            if constexpr (HF == 1) park_rows();
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) *reinterpret_cast<f4 *>(red + (wave * B + 16 * bt + li) * 16 + 4 * lg) = acc[bt];
        }
        __syncthreads();
        const bool more = u + AHEAD < steps, updates = SUB == 1 || half == 1;
        // ---- h = relu(z1 + b1) ----------------------------------------------------------
        const uint32_t tag = tag0 + (uint32_t)u;
        const int par = u & 1;
        // (addresses are worked out here: kept across the loop they would fill the registers)
        const int ln = opaque(lane), li = ln & 15, lg = ln >> 4, tid = 64 * wave + ln;
        const int mt = 16 * wave + li;   // waves 0 .. NBT - 1: the lane's sample in the small products
        // (threads beyond the B * 16 elements do the last one's sums and keep them to themselves)
        const int i = min(tid, B * 16 - 1);
        const bool mine_h = B * 16 >= kMlpThreads || tid < B * 16;
        float part[kMlpWaves];
#pragma unroll
        for (int w = 0; w < kMlpWaves; ++w) part[w] = red[w * B * 16 + i];
        const float bias1 = b1s[i & 15];
        f4 w2 = {0.f, 0.f, 0.f, 0.f};   // class li, units 4 lg ..
        if (wave < NBT) w2 = *reinterpret_cast<const f4 *>(W2s + 16 * li + 4 * lg);
        __builtin_amdgcn_sched_barrier(0);   // all on their way before the first is added
        if constexpr (HF == 1) {
            float s = bias1;
#pragma unroll
            for (int w = 0; w < kMlpWaves; ++w) s += part[w];
            if (mine_h) hs[i] = s > 0.f ? s : 0.f;
        } else {
            // the own half's sums go to the pair record, the other half's come from there;
            // both halves add them in the same order (half 0 + half 1), so both get the same h
            float own = 0.f;
#pragma unroll
            for (int w = 0; w < kMlpWaves; ++w) own += part[w];
            const int base = 8 * par * 2 * kMlpPair;
            if (mine_h) pair.post(8 * i, base + 8 * hf * kMlpPair, tag, own, same);
            __builtin_amdgcn_sched_barrier(0);
            park_rows();
            i2 v;
            BoundedWait wait;
            for (;;) {
                ClusterWords::look_again();
                v = pair.get(8 * i, base + 8 * (1 - hf) * kMlpPair);
                if (__all((uint32_t)v[1] == tag) || dead) break;
                __builtin_amdgcn_s_sleep(1);
                if (wait.gave_up(errflag)) dead = 1;
            }
            const int got = v[0];
            const float other = __builtin_bit_cast(float, got);
            const float s = bias1 + (hf == 0 ? own + other : other + own);
            if (mine_h) hs[i] = s > 0.f ? s : 0.f;
        }
        __syncthreads();
        // ---- partial logits of the own 16 units -> tagged exchange record ---------------
        const int recpar = 8 * par * kMlpMaxG * kMlpRec;
        f4 h = {0.f, 0.f, 0.f, 0.f};   // sample mt, units 4 lg ..
        if (wave < NBT) {
            h = *reinterpret_cast<const f4 *>(hs + 16 * mt + 4 * lg);
            if (hf == 0) {
                f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s) acc = mfma16(w2[s], h[s], acc);
                if (4 * lg < C) rec.post(8 * (16 * mt + 4 * lg), recpar + 8 * g * kMlpRec, tag, acc, same);
            }
        }
        // ---- logits, softmax, d logits: thread (b, o) = (tid / 16, tid % 16) ------------
        // Every thread polls the G tagged words of its own element (b, o): with the
        // words in the XCD's L2 an exchange is then one trip.  Polls through memory slow the peers'
        // stores down (they meet in the same memory channels): there, while the peers are still
        // computing, only wave 0 looks, and only at one word per record and batch tile (the last one
        // its owner stores).  The element tags are still checked, and the fetch repeated if one is
        // stale.  (A separate flag word per poster, stored after the logits, overtakes them on the
        // way.)  16 clients, 784 -> 128, 50 rounds: in L2 7.61 ms with the watch, 7.47 without;
        // through memory 8.9 and 12.1.
        if (!same) {
            if (wave == 0) {
                // lane -> (record, batch tile); the word of sample 16*bt+15, class C-1
                const int gg = lane % G, bt = lane / G;
                const int at = 8 * (gg * kMlpRec + (16 * min(bt, NBT - 1) + 15) * 16 + (C - 1));
                BoundedWait wait;
                for (;;) {
                    ClusterWords::look_again();
                    const bool ok = bt >= NBT || (uint32_t)rec.get(at, recpar)[1] == tag;
                    if (__all(ok) || dead) break;
                    __builtin_amdgcn_s_sleep(2);
                    if (wait.gave_up(errflag)) dead = 1;
                }
            }
            __syncthreads();
        }
        float w2t[4];   // unit li, classes 4 lg ..
        if (wave < 4 * NBT) {
            const int b = tid >> 4, o = tid & 15;
            const int at = 8 * (16 * b + min(o, C - 1));
            const float bias2 = b2s[o];
            const int lab = labs[b];
            if (wave < NBT) {
#pragma unroll
                for (int s = 0; s < 4; ++s) w2t[s] = W2s[(4 * lg + s) * 16 + li];
            }
            float z;
            BoundedWait wait;
            const int Gn = opaque_scalar(G);
            // all records at once, as many as there are at most; those beyond the last stand for it
            auto fetch = [&](auto most) __attribute__((always_inline)) {
                constexpr int GC = decltype(most)::value;
                i2 v[GC];
                ClusterWords::look_again();
#pragma unroll
                for (int gg = 0; gg < GC; ++gg) v[gg] = rec.get(at, recpar + 8 * min(gg, Gn - 1) * kMlpRec);
                __builtin_amdgcn_sched_barrier(0);
                uint32_t stale = 0;
                z = bias2;
#pragma unroll
                for (int gg = 0; gg < GC; ++gg) {
                    const int bits = v[gg][0];
                    stale |= (uint32_t)v[gg][1] ^ tag;
                    if (gg < Gn) z += __builtin_bit_cast(float, bits);
                }
                return __all(stale == 0);
            };
            for (;;) {
                if (Gn <= 4 ? fetch(std::integral_constant<int, 4>{}) : Gn <= 8 ? fetch(std::integral_constant<int, 8>{}) : fetch(std::integral_constant<int, kMlpMaxG>{})) break;
                if (dead) break;
                if (!same) __builtin_amdgcn_s_sleep(2);
                if (wait.gave_up(errflag)) dead = 1;
            }
            const float zmax = row16_max(o < C ? z : -3.0e38f);
            // PAD: expf and logf as in the layer engine, where these models run otherwise
            const auto exp_of = [](float v) { return PAD ? expf(v) : __expf(v); };
            const float ex = o < C ? exp_of(z - zmax) : 0.f;
            const float sum = row16_sum(ex), lse = zmax + (PAD ? logf(sum) : __logf(sum));
            if (o == lab) lossb[b] = lse - z;
            zs[b * 16 + o] = o < C && (SUB == 1 ? b : B * half + b) < Br ? exp_of(z - lse) - (o == lab ? 1.f : 0.f) : 0.f;
        }
        __syncthreads();
        // ---- small products on the matrix cores -----------------------------------------
        f4 dW2acc = SUB == 2 && updates ? dW2k : f4{0.f, 0.f, 0.f, 0.f};
        if (wave < NBT) {
            // dh = (dz W2) * 1[h > 0] for samples 16*wave .. 16*wave+15
            const f4 dz = *reinterpret_cast<const f4 *>(zs + 16 * mt + 4 * lg);
            f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = mfma16(w2t[s], dz[s], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = h[r] > 0.f ? acc[r] : 0.f;
            *reinterpret_cast<f4 *>(dhs + 16 * mt + 4 * lg) = acc;
        } else if (wave == 2) {
            // dW2[o][j] = sum_b dz[b][o] h[b][j]; applied after the barrier (W2 is still read)
            float za[4 * NBT], hb[4 * NBT];
#pragma unroll
            for (int s = 0; s < 4 * NBT; ++s) {
                za[s] = zs[(4 * s + lg) * 16 + li];
                hb[s] = hs[(4 * s + lg) * 16 + li];
            }
#pragma unroll
            for (int s = 0; s < 4 * NBT; ++s) dW2acc = mfma16(za[s], hb[s], dW2acc);
            if (!updates) dW2k = dW2acc;
        } else if (wave == 3) {
            // second-layer bias: column sums of dz
            float s = col_sum16<B>(zs, lane);
            if (SUB == 2) s = updates ? db2k + s : (db2k = s);
            s *= invB;
            if (updates && lane < C) {
                b2s[lane] -= p.eta * s;
                Ub2s[lane] += s;
            }
        } else if (wave == 4) {
            // the recursion's mean loss
            const float s = row16_sum(fold_rows((SUB == 1 ? lane : B * half + lane) < Br && lane < B ? lossb[min(lane, B - 1)] : 0.f));
            if (lane == 0) lossacc[0] += s * invB;
        } else if (wave == kRowsWave && more) {
            // the rows that recursion u + AHEAD samples, for all waves, and their labels
            const uint32_t row = rows_of(u + AHEAD);
            if (lane < B) {
                rows[lane] = row;
                lab_ahead = yg[row];
            }
        }
        __syncthreads();
        // The row loads are issued a few at a time between the first tiles of the backward product, so that a wave
        // that has to wait for room in the memory pipeline leaves the matrix core to the SIMD's other
        // wave.  They go into the registers the forward product has finished with.  (Loads of one wave return in
        // order, so nothing is issued before the exchange polls.)
        gcf_ptr myrow[NBT];
        if (more) {
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) myrow[bt] = lane_src + (int64_t)rows[16 * bt + li] * D;
        }
        constexpr int PFT = TPW > 4 ? 4 : TPW;   // tiles of the backward product that carry loads
        auto prefetch_load = [&](int j) {        // j = tt * NBT + bt: in the order the forward product uses them
            // (beyond the last recursion zeros: the rows at work end here on every way, which frees their registers before)
            f4 piece = {0.f, 0.f, 0.f, 0.f};
            if (more) piece = load_piece(myrow[j % NBT], j / NBT, ntile, tail);
            x[j % NBT][j / NBT] = piece;
        };
        // ---- second layer and first-layer bias: w <- w - eta g, U <- U + g ---------------
        if (wave == 2 && updates) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = (4 * lg + r) * 16 + li;  // (o, j)
                const float gv = dW2acc[r] * invB;
                W2s[e] -= p.eta * gv;
                U2s[e] += gv;
            }
        } else if (wave == 3) {
            // first-layer bias: column sums of dh
            float s = col_sum16<B>(dhs, lane);
            if (SUB == 2) s = updates ? db1k + s : (db1k = s);
            s *= invB;
            if (updates && lane < 16) {
                b1s[lane] -= p.eta * s;
                Ub1s[lane] += s;
            }
        }
        // ---- first layer: dW1^T = X^T dh on the matrix cores, update in registers -------
        {
            // contraction step s of lane group lg takes sample 16*(s/4) + (s%4) + 4*lg: with
            // rows 4*lg apart the four lane groups read LDS banks 16 apart (ld = 4 mod 32)
            float dhb[4 * NBT];
#pragma unroll
            for (int s = 0; s < 4 * NBT; ++s) dhb[s] = dhs[(16 * (s >> 2) + (s & 3) + 4 * lg) * 16 + li];
            float xb[2][4 * NBT];
            const float *xcol = Xs + opaque(4 * lg * ld + col0 + li);
            if (FULL || ntile > 0) {
#pragma unroll
                for (int s = 0; s < 4 * NBT; ++s) xb[0][s] = xcol[(16 * (s >> 2) + (s & 3)) * ld];
            }
            const float eb = p.eta * invB;
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) {
                if (tt + 1 < TPW && (FULL || tt + 1 < ntile)) {
#pragma unroll
                    for (int s = 0; s < 4 * NBT; ++s) xb[(tt + 1) & 1][s] = xcol[(16 * (s >> 2) + (s & 3)) * ld + 16 * (tt + 1)];
                }
                __builtin_amdgcn_sched_barrier(0);   // the next tile's operands are on their way before the products
                if (FULL || tt < ntile) {
                    // two independent accumulation chains per tile
                    // (the first product of each chain takes the constant zero as its addend)
                    f4 acc0 = mfma16(xb[tt & 1][0], dhb[0], SUB == 2 && updates ? Gk[tt] : f4{0.f, 0.f, 0.f, 0.f});
                    f4 acc1 = mfma16(xb[tt & 1][1], dhb[1], f4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                    for (int s = 2; s < 4 * NBT; s += 2) {
                        acc0 = mfma16(xb[tt & 1][s], dhb[s], acc0);
                        acc1 = mfma16(xb[tt & 1][s + 1], dhb[s + 1], acc1);
                    }
                    if (!updates) Gk[tt] = acc0 + acc1;
#pragma unroll
                    for (int r = 0; r < 4 && updates; ++r) {
                        const float gsum = acc0[r] + acc1[r];
                        W1r[tt][r] -= eb * gsum;
                        U1r[tt][r] += invB * gsum;
                    }
                }
                // this tile's share of the row loads
#pragma unroll
                for (int j = tt * NI / PFT; j < (tt + 1) * NI / PFT && j < NI; ++j) prefetch_load(j);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // ---- the next recursion's labels ----------------------------------------------------
        if (AHEAD == 1) lab_next = lab_ahead;
        if (wave == kRowsWave && lane < B && u + 1 < steps) labs[lane] = lab_next;
        lab_next = lab_ahead;
    };
    auto recursions = [&](const auto same) __attribute__((always_inline)) {
        for (Step u = 0; u < steps; ++u) {
            recursion(u, AHEAD == 2 ? 0 : u & 1, xreg[0], same);
            if constexpr (AHEAD == 2) {
                if (++u == steps) break;
                recursion(u, 1, xreg[1], same);
            }
        }
    };
    // Written out for either answer, or with a test in one loop where two are no faster.  One loop / two, words in L2, ms
    // a job: 16 clients, 784 -> 128, B = 32 6.99 / 6.73; 13, 256 -> 128 0.516 / 0.501; 48, 784 -> 128, B = 16 2.06 / 2.03; 40, 896 -> 256,
    // B = 32 (two batch tiles with seven column tiles) 3.14 / 3.29.
    if (NBT * TPW > 2 * kMlpHalfTPW) recursions(one_xcd);
    else if (one_xcd) recursions(std::true_type());
    else recursions(std::false_type());

    // ---- end of round: the replica and the message payload go to HBM ---------------------
#pragma unroll
    for (int tt = 0; tt < TPW; ++tt) {
        if (tt < nt && unit_ok) {
            const int64_t base = (int64_t)unit * D + gcol0 + 16 * tt + 4 * lg;
            if constexpr (FAST) {
                *reinterpret_cast<f4 __attribute__((address_space(1))) *>(Wc + base) = W1r[tt];
                *reinterpret_cast<f4 __attribute__((address_space(1))) *>(Uc + base) = U1r[tt];
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (gcol0 + 16 * tt + 4 * lg + r < D) {
                        Wc[base + r] = W1r[tt][r];
                        Uc[base + r] = U1r[tt][r];
                    }
            }
        }
    }
    __syncthreads();
    if (hf == 0) {
        const int o = tid >> 4, j = tid & 15;
        if (tid < 256 && o < C && (!PAD || 16 * g + j < H)) {
            Wc[w2_off + (int64_t)o * H + 16 * g + j] = W2s[tid];
            Uc[w2_off + (int64_t)o * H + 16 * g + j] = U2s[tid];
        }
        if (tid < 16) {
            if (!PAD || 16 * g + tid < H) {
                Wc[b1_off + 16 * g + tid] = b1s[tid];
                Uc[b1_off + 16 * g + tid] = Ub1s[tid];
            }
            if (g == 0 && tid < C) {
                Wc[b2_off + tid] = b2s[tid];
                Uc[b2_off + tid] = Ub2s[tid];
            }
        }
    }
    // the loss was accumulated by wave 4, lane 0 of unit group 0
    if (g == 0 && hf == 0 && wave == 4 && lane == 0) *as_global(p.loss) = lossacc[0];
}

__global__ void k_zero_words(unsigned long long *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

static int mlp_tpw(int D) { return (D + 15) / 16 <= 2 * kMlpWaves ? 2 : kMlpMaxTPW; }
// whether launch_mlp_round gives a unit group two workgroups where there is room
static bool mlp_halves(int D) { return mlp_tpw(D) != 2 && ((D + 15) / 16 + 1) / 2 <= kMlpWaves * kMlpHalfTPW; }

static size_t mlp_lds_bytes_tpw(int tpw, int B) {
    const int ld = 16 * kMlpWaves * tpw + 4;
    return sizeof(float) * ((size_t)B * ld + kMlpWaves * B * 16 + 3 * B * 16 + 512 + 64 + B + 16) + sizeof(int) * 2 * B;
}
static size_t mlp_lds_bytes(int D, int B) { return mlp_lds_bytes_tpw(mlp_tpw(D), B); }

bool mlp_round_supported(int D, int H, int C, int B) {
    if (B < 1 || B > 64) return false;
    if (H < 1 || H > 16 * kMlpMaxG || C < 1 || C > 16) return false;
    if (D < 1 || (D + 15) / 16 > kMlpWaves * kMlpMaxTPW) return false;
    return mlp_lds_bytes(D, B <= 16 ? 16 : 32) <= 160 * 1024;
}

bool mlp_round_exact(int H, int B) { return (B == 16 || B == 32) && H % 16 == 0; }

// (The ratios are those of the form that had one mini-batch ahead; the present one is 1.05 to 1.6 times as fast, so the line could lie
// further out.  It stays because models beyond it would get other bits.)
// The layer engine's launches take all clients, these as many as are resident (at most kMlpPack)
// and follow one another, so it catches up with many clients, the sooner the smaller the
// model.  Time here / there per recursion at mini-batches of 1 to 31, launches in brackets:
//              30 inputs              100                    300                    784
//   10 units   96 (2)  0.43 .. 0.48   0.51 .. 0.56           0.64 .. 0.76
//             192 (4)  0.74 .. 0.86   0.86 .. 0.93           1.03 .. 1.13
//             256 (6)  1.03 .. 1.25   1.20 .. 1.27           1.37 .. 1.48           0.88 .. 0.99
//   100 units 128 (4)  0.63 .. 0.75   0.67 .. 0.70           0.75 .. 0.78
//             256 (8)  0.99 .. 1.26   0.76 .. 0.88           0.65 .. 0.77           0.30 .. 0.36
//   130 units 256 (11) 1.28 .. 1.65   1.05 .. 1.15           0.83 .. 0.96
//   250 units  96 (6)  0.87 .. 1.09   0.95 .. 0.99           0.91 .. 0.96
//             256 (16) 1.76 .. 2.10   1.29 .. 1.42           0.93 .. 1.10           0.37 .. 0.46
// (256 inputs, 250 units, 256 clients: 0.82 .. 0.89; 400: 0.67 .. 0.79.)
// Mini-batches of 33 .. 64 take two steps a recursion here and the same launches there, where the time grows with the mini-batch,
// so that the table above does not hold for them.  Here a recursion takes a time per launch that depends on a wave's column tiles and the
// unit groups, however few clients the last launch has; there 28 us and what the products take.  Both in us, fitted to 2,040 shapes of 30 .. 896
// inputs, 1 .. 256 units and 17 .. 256 clients (the first that needs one launch more, for each number of launches) at 33, 48, 56 and 64
// samples.  Time here / there, lowest and highest over the inputs, at 33 samples:
//   units        launches: 3   4          5          6          8          16
//     1           .66 1.08     1.20 1.22  1.28 1.28  1.34 1.40
//    17           .66 1.01     .80 1.11   .95 1.20   1.06 1.26
//    33           .63 .93      .74 .99    .86 1.02   .95 1.14
//    97           .59 .80      .71 .84    .77 .87    .80 .93    .81 1.03
//   161           .67 .95      .81 .98    .97 1.09   1.01 1.16  1.08 1.33  .77 1.23   (16 clients a launch: 11 of 16 compute units at work)
//   250           .62 .77      .72 .91    .74 .92    .68 .96    .79 1.06   .62 1.00
// (at 56 samples 0.8 - 0.9 of that; two launches .41 - .96.)  With the line 3 % below the layer engine's time, 10 of the 1,600 that come here
// are slower, by up to 6 %, and 69 of the others would be more than 8 % faster, by up to 1.4 times (130 to 170 units, over 176 clients).
static bool mlp_two_steps_pay(int D, int H, int B, int n_clients, int G, int launches) {
    const int tiles = ((D + 15) / 16 + kMlpWaves - 1) / kMlpWaves;
    const double here = launches * (5.4 + (D > 256 ? 1.15 : 0) + 1.5 * tiles + (G > 4 ? 0.65 : 0) + (G > 8 ? 1.1 : 0));
    const double there = 28.2 + n_clients * (5.9e-6 * H * D + 4.1e-6 * B * D + 1.8e-5 * B * H);
    return launches <= 2 || here <= 0.97 * there;
}
bool mlp_padded_pays(int D, int H, int B, int n_clients) {
    const int G = (H + 15) / 16, fit = resident_clusters(256, 8, G), per = fit < kMlpPack ? fit : kMlpPack;
    const int launches = (n_clients + per - 1) / per;
    if (B > 32 && !mlp_two_steps_pay(D, H, B, n_clients, G, launches)) return false;
    if (launches <= 3 || D >= 768) return true;
    return G > 1 && (launches <= 5 || D >= 384 || (D >= 256 && launches <= 12) || (D >= 100 && launches <= 8));
}

// exchange records [client][2][kMlpMaxG][kMlpRec] 64-bit words, the pair records
// [client][kMlpMaxG][2][2][kMlpPair], the workgroups' places [client][kPlaces], then the error flag
static size_t mlp_rec_words(int n_clients) { return (size_t)n_clients * 2 * kMlpMaxG * kMlpRec; }
static size_t mlp_pair_words(int n_clients) { return (size_t)n_clients * kMlpMaxG * 4 * kMlpPair; }
static size_t mlp_all_words(int n_clients) { return mlp_rec_words(n_clients) + mlp_pair_words(n_clients) + (size_t)n_clients * kPlaces; }
static_assert(2 * kMlpMaxG <= kClusterMax, "a place for every workgroup");

size_t mlp_round_scratch_bytes(int n_clients, int B) {
    (void)B;
    return mlp_all_words(n_clients) * 8 + 256;
}

template <int NBT, int TPW, bool FAST, bool FULL, int HF, bool PAD, int SUB = 1>
static hipError_t mlp_capacity(size_t lds, int *cap) {   // resident workgroups
    int dev = 0;
    const hipError_t e0 = hipGetDevice(&dev);
    if (e0 != hipSuccess) return e0;
    static PerDevice capacity;   // of this instantiation
    return capacity.get(dev, cap, [lds, dev](int *found) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_mlp_round<NBT, TPW, FAST, FULL, HF, PAD, SUB>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        int cus = 0, per_cu = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_round<NBT, TPW, FAST, FULL, HF, PAD, SUB>, kMlpThreads, lds);
        *found = cus * per_cu;
        return e;
    });
}

// HF = 2 (two workgroups per unit group) is taken only when all active clients fit one
// launch that way; otherwise *declined is set and nothing is launched.
template <int NBT, int TPW, bool FAST, bool FULL, int HF, bool PAD, int SUB = 1>
static hipError_t mlp_launch(hipStream_t s, Profiler *prof, const RoundParams *hp, int nact, int max_m,
                             const float *Wg, int D, int H, int C, int Br, void *scratch, int n_clients,
                             int first, uint32_t *epoch, bool *declined = nullptr) {
    constexpr int B = 16 * NBT;
    const int G = (H + 15) / 16;
    const size_t lds = mlp_lds_bytes_tpw(TPW, B);
    int cap = 0, xcds = 0;
    hipError_t e = mlp_capacity<NBT, TPW, FAST, FULL, HF, PAD, SUB>(lds, &cap);
    if (e == hipSuccess) e = device_xcds(&xcds);
    if (e != hipSuccess) return e;
    // Clusters per launch: every workgroup that polls must be resident together with its
    // peers.  Workgroups of unused slots exit at once and free their compute unit, so only
    // the working ones count.
    const int fit = resident_clusters(cap, xcds, G * HF);
    const int per_launch = fit < kMlpPack ? fit : kMlpPack;
    if (HF == 2 && per_launch < nact) {
        *declined = true;
        return hipSuccess;
    }
    if (per_launch < 1) return hipErrorLaunchOutOfResources;
    unsigned long long *xrec = static_cast<unsigned long long *>(scratch);
    unsigned long long *prec = xrec + mlp_rec_words(n_clients), *claims = prec + mlp_pair_words(n_clients), *places = g_posts_to_memory ? nullptr : claims;
    int *errflag = reinterpret_cast<int *>(xrec + mlp_all_words(n_clients));
    // step tags of this launch: never 0 (the cleared state) and never a tag that an
    // earlier launch may have left in the records
    // A captured launch carries its tags into every replay, where the records still hold words
    // of the replay before with the same tags: there the records are cleared ahead of it.
    const uint32_t need = cluster_steps(max_m, SUB) + 1u;
    const bool spent = tags_spent(*epoch, need);
    if (spent || stream_is_capturing(s)) {
        k_zero_words<<<(unsigned)((mlp_all_words(n_clients) + 255) / 256), 256, 0, s>>>(xrec, mlp_all_words(n_clients));
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (spent) *epoch = 1;
    const uint32_t tag0 = *epoch;
    *epoch += need;
    for (int a0 = 0; a0 < nact; a0 += per_launch) {
        const int here = (nact - a0 < per_launch) ? nact - a0 : per_launch;
        const int groups = (here + 7) / 8;  // clients per XCD in this launch
        const unsigned grid = (unsigned)(8 * groups * G * HF);
        MlpPack pack;
        for (int j = 0; j < here; ++j) pack.p[j] = hp[a0 + j];
        if (prof && prof->on[F_MLP_ROUND]) prof->before(F_MLP_ROUND, s);
        k_mlp_round<NBT, TPW, FAST, FULL, HF, PAD, SUB><<<grid, kMlpThreads, lds, s>>>(pack, here, a0, Wg, D, H, C, G, Br, xrec, prec, places, g_xcd_skew, tag0, errflag, claims, first);
        if (prof && prof->on[F_MLP_ROUND]) prof->after(F_MLP_ROUND, s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_mlp_round(hipStream_t s, Profiler *prof, const RoundParams *hp, int nact, int max_m,
                            const float *Wg, int D, int H, int C, int B, void *scratch,
                            int n_clients, int first, uint32_t *epoch) {
    if (nact <= 0) return hipSuccess;
    if (first > 7 || (first >= 0 && B <= 32)) return hipErrorInvalidValue;
    const bool small = mlp_tpw(D) == 2;  // at most 2 K tiles per wave
    const bool fast = (D & 15) == 0;
    const bool full = D == 16 * kMlpWaves * mlp_tpw(D);   // no pad tiles
    // wide inputs: two workgroups per unit group, half of the columns each, when every active
    // client gets its 2 G workgroups resident in one launch
    const bool pad = !mlp_round_exact(H, B), half = mlp_halves(D);
    if (B > 32) {
#define AET_MLP_TWO(tpw, fast_, hf, ...) mlp_launch<2, tpw, fast_, false, hf, true, 2>(s, prof, hp, nact, max_m, Wg, D, H, C, B, scratch, n_clients, first, epoch, ##__VA_ARGS__)
        if (half) {
            bool declined = false;
            const hipError_t e = fast ? AET_MLP_TWO(kMlpHalfTPW, true, 2, &declined) : AET_MLP_TWO(kMlpHalfTPW, false, 2, &declined);
            if (e != hipSuccess || !declined) return e;
        }
        if (small) return fast ? AET_MLP_TWO(2, true, 1) : AET_MLP_TWO(2, false, 1);
        return fast ? AET_MLP_TWO(kMlpMaxTPW, true, 1) : AET_MLP_TWO(kMlpMaxTPW, false, 1);
#undef AET_MLP_TWO
    }
#define AET_MLP(nbt, tpw, fast_, full_, hf, ...)                                                                            \
    (pad ? mlp_launch<nbt, tpw, fast_, full_, hf, true>(s, prof, hp, nact, max_m, Wg, D, H, C, B, scratch, n_clients, first, epoch, ##__VA_ARGS__)   \
         : mlp_launch<nbt, tpw, fast_, full_, hf, false>(s, prof, hp, nact, max_m, Wg, D, H, C, B, scratch, n_clients, first, epoch, ##__VA_ARGS__))
    if (half) {
        bool declined = false;
        hipError_t e;
        if (B <= 16) e = fast ? AET_MLP(1, kMlpHalfTPW, true, false, 2, &declined) : AET_MLP(1, kMlpHalfTPW, false, false, 2, &declined);
        else e = fast ? AET_MLP(2, kMlpHalfTPW, true, false, 2, &declined) : AET_MLP(2, kMlpHalfTPW, false, false, 2, &declined);
        if (e != hipSuccess || !declined) return e;
    }
#define AET_MLP_CASE(nbt, tpw)                                        \
    do {                                                              \
        if (full) return AET_MLP(nbt, tpw, true, true, 1);            \
        if (fast) return AET_MLP(nbt, tpw, true, false, 1);           \
        return AET_MLP(nbt, tpw, false, false, 1);                    \
    } while (0)
    if (B <= 16) {
        if (small) AET_MLP_CASE(1, 2);
        AET_MLP_CASE(1, kMlpMaxTPW);
    }
    if (small) AET_MLP_CASE(2, 2);
    AET_MLP_CASE(2, kMlpMaxTPW);
#undef AET_MLP_CASE
#undef AET_MLP
}

hipError_t mlp_cluster_need(int D, int H, int B, int n_clients, int *cus, int *clients, int *size) {
    int dev = 0, all = 0, xcds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&all, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = device_xcds(&xcds);
    if (e != hipSuccess) return e;
    *size = dense_cluster_size(xcds == 8 ? all / xcds : 0, (H + 15) / 16, mlp_halves(D), n_clients);
    *cus = *size ? all / xcds : 0;
    *clients = B > 32 ? n_clients : (n_clients + 7) / 8 * 8;
    return hipSuccess;
}

hipError_t mlp_clear_error_flag(hipStream_t s, void *scratch, int n_clients, int B) {
    (void)B;
    unsigned long long *xrec = static_cast<unsigned long long *>(scratch);
    k_zero_words<<<1, 64, 0, s>>>(xrec + mlp_all_words(n_clients), 1);
    return hipGetLastError();
}

const int *mlp_error_flag_ptr(void *scratch, int n_clients, int B) {
    (void)B;
    unsigned long long *xrec = static_cast<unsigned long long *>(scratch);
    return reinterpret_cast<const int *>(xrec + mlp_all_words(n_clients));
}

}  // namespace aet
