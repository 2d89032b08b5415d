// 3 x 3 convolutions of the layer-by-layer engine with padding 1 on the bf16 matrix cores, fp32
// values split in three bf16 parts (split_bf16.h), as implicit GEMMs over tiles staged in LDS.
//
// Forward and backward-data are the same kernel (as in kernels_conv_mfma.hip):
//   dst[dc][y][x] = sum_{sc,ky,kx} src[sc][y+ky-1][x+kx-1] * Wt[dc][sc][ky][kx]
//   forward:        Wt[dc][sc][ky][kx] = W[dc][sc][ky][kx], then bias and ReLU (and pooling);
//   backward-data:  Wt[dc][sc][ky][kx] = W[sc][dc][2-ky][2-kx], then the ReLU mask of the layer below.
// GEMM view: M = 32 destination channels, N = pixels in tiles of 32 (whole rows of 8, 16 or 32),
// K = (tap, sc) in chunks of 16 source channels.  A workgroup owns 256 pixels (rows of one sample, or
// several samples of 8 x 8) and 32 destination channels; each of its 4 waves owns two pixel tiles.
//
// What bounds it: in launches of all 32 clients of the CNN on 32 x 32 the matrix cores are busy 52 to 55 % of
// the time in forward, 47 % in backward-data at 16 x 16 and 38 % at 32 x 32, where it moves 0.72 GB in about
// 0.25 ms; the rest is the staging between two barriers and the LDS (9 reads of 16 bytes for 12 products, and
// 17 % of a compute unit's cycles in bank conflicts on maps of 16).  The clock meanwhile is 2.1 GHz of 2.4: cards
// differ by 5 % after what their power limit leaves.  Unlike the fp32 matrix instructions these leave the
// vector ALU free for the splitting.  CNN on 32 x 32, 32 clients, 4 rounds: forward and backward-data
// together 24 -> 16 ms, the job 48.9 -> 40.1.
#include <type_traits>

#include "aet_device.h"
#include "aet_internal.h"
#include "split_bf16.h"

namespace aet {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));

// dword 3 of a raw buffer descriptor for 32-bit untyped accesses on this part
constexpr int kBufferFlags = 0x00020000;
constexpr uint32_t kNowhere = 0x80000000u;   // a byte offset no buffer here reaches: reads as zero

typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef const u4 __attribute__((address_space(1))) *gu4_ptr;

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

struct SplitDir {
    int SC, DC;          // source / destination channels
    int H;               // rows of the maps (both sides; the width is the template's)
    int lgRW;            // R W = 2^lgRW
    int R, NS;           // rows and samples per workgroup: R * W * NS = 128 MT pixels (NS > 1: R = H)
    int rblocks;         // row blocks per sample
    int64_t w_off, b_off;
    int ic, oc;          // the layer's own channel counts (weight layout W[oc][ic][3][3])
    int relu, pool;
};

// LDS, in 16-byte pieces (8 channels of one bf16 part): the source tile [part][octet][position],
// the weights [part][tap][octet][32]
template <int LGW, int MT>
struct SplitTile {
    static constexpr int W = 1 << LGW, PX = 128 * MT, ROWS = PX / W;   // rows over all samples
    static constexpr int SMALL = W;                                    // square maps of several samples: H = W
    // positions of the padded tile: NS (R + 2) (W + 2); NS = 1: R = ROWS; else R = W, NS = ROWS / W
    static constexpr int NSMAX = ROWS / SMALL > 1 ? ROWS / SMALL : 1;
    static constexpr int POS1 = (ROWS + 2) * (W + 2), POSN = NSMAX > 1 ? NSMAX * (SMALL + 2) * (W + 2) : 0;
    static constexpr int POS = (POS1 > POSN ? POS1 : POSN) | 1;        // odd: see the staging
    static constexpr int LDS = (6 * POS + 6 * 9 * 32) * 16;            // bytes
};

// UNPOOL (backward-data only): src is the gradient at the outputs of the 2 x 2 pooling layer behind the
// convolution, amax that layer's winners; the gradient at the convolution's own outputs, a value at
// each window's winner and zeros, is put together while it is staged: five bytes a window are read where
// a kernel of the pooling layer wrote sixteen and this one read them again.  32 clients (compute factors
// 1, 2, 4) x 64 samples, us per launch: 32 -> 32 channels at 32 x 32 129 -> 125, its backward-weight 126
// -> 128; 64 -> 64 at 16 x 16 92 -> 99 (the selections, in both blocks of channels) and 124 -> 124; the
// pooling kernels' 26 each are gone: the job of 4 rounds 37.0 -> 35.7 ms.
template <int LGW, int MT, bool BWD, bool UNPOOL>
__global__ void __launch_bounds__(256, 2)
k_conv_split(const RoundParams *__restrict__ rp, int u, int B, SplitDir g, const u4 *__restrict__ wsplit, int64_t wstride,
             const float *__restrict__ src, float *__restrict__ dst, const float *__restrict__ mask_src, uint8_t *__restrict__ amax) {
    static_assert(BWD || !UNPOOL, "the forward pass reads whole maps");
    typedef SplitTile<LGW, MT> T;
    constexpr int W = T::W, POS = T::POS, WT = W + 2;
    const RoundParams p = rp[blockIdx.z];
    if (u >= p.m) return;
    extern __shared__ __attribute__((aligned(16))) bf8 sm[];
    bf8 *const As = sm;                 // [3][2][POS]
    bf8 *const Bs = sm + 6 * POS;       // [3][9][2][32]
    __shared__ __attribute__((aligned(16))) float bs[32];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dc0 = 32 * (int)blockIdx.x;
    const int HW = g.H * W;
    const int y0 = (int)blockIdx.y % g.rblocks * g.R, s0 = (int)blockIdx.y / g.rblocks * g.NS;   // row; sample of the mini-batch
    const int ns = min(g.NS, B - s0);   // samples that exist
    const int64_t sample0 = (int64_t)blockIdx.z * B + s0;
    constexpr int UN = UNPOOL ? 2 : 1;
    const int SHW = HW / (UN * UN);     // a channel of src
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(src) + sample0 * g.SC * SHW, 0, 4 * g.SC * SHW * ns, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        UNPOOL ? amax + sample0 * g.SC * SHW : nullptr, 0, UNPOOL ? g.SC * SHW * ns : 0, kBufferFlags);

    // ---- staging: what this thread moves ----------------------------------------------------
    // source: four pixels of one tile row, 8 channels (an octet of the chunk's two).  Threads in the
    // order (four quarters of a row, octet, row, rest of the row): with POS odd the 16 lanes that
    // write to LDS together then meet 16 different places.
    constexpr int XL = W / 4 < 4 ? W / 4 : 4;
    const int rowsT = g.R + 2, rows = g.NS * rowsT;
    const int ao = (tid / XL) & 1, at = tid / (2 * XL), atr = at % rows, axq = tid % XL + XL * (at / rows);
    const int as = atr / rowsT, ay = atr - as * rowsT - 1;
    const int alds = axq < W / 4 ? ao * POS + atr * WT + 1 + 4 * axq : -1;
    // (samples beyond the last lie beyond the buffer)
    const uint32_t aoff = alds >= 0 && (unsigned)(y0 + ay) < (unsigned)g.H
                              ? (uint32_t)(4 * ((as * g.SC + 8 * ao) * SHW + (y0 + ay) / UN * (W / UN) + 4 / UN * axq)) : kNowhere;
    const int awin = 2 * ((y0 + ay) & 1);        // UNPOOL: the row's first element of a window
    // weights: split and in order already
    constexpr int WP = 6 * 9 * 32, WTURNS = (WP + 255) / 256;
    const gu4_ptr wsrc = (gu4_ptr)(wsplit + blockIdx.z * wstride + (int64_t)blockIdx.x * WP);
    const int wchunk = WP * (int)gridDim.x;
    const int astep = 4 * SHW;                   // bytes per source channel
    f4 av[8];                                    // UNPOOL: the first two: the gradients of two windows
    uint32_t aw[8];                              // UNPOOL: their winners
    u4 wv[WTURNS];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (UNPOOL) {
                const f2v d = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)aoff, (c0 + c) * astep, 0));
                av[c][0] = d[0];
                av[c][1] = d[1];
                aw[c] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)(aoff >> 2), (c0 + c) * SHW, 0);
            } else {
                av[c] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)aoff, (c0 + c) * astep, 0));
            }
        }
        const gu4_ptr w = wsrc + (c0 >> 4) * wchunk;
#pragma unroll
        for (int i = 0; i < WTURNS; ++i) wv[i] = w[min(tid + 256 * i, WP - 1)];
    };
    auto stash_source = [&](auto clamp, uint32_t &seen) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                x[c] = !UNPOOL ? av[c][e] : ((aw[c] >> (8 * (e >> 1))) & 0xffu) == (uint32_t)(awin + (e & 1)) ? av[c][e >> 1] : 0.f;
            const Split8 s = split8<decltype(clamp)::value>(x);
            split_watch(seen, s);
#pragma unroll
            for (int q = 0; q < 3; ++q) As[q * 2 * POS + alds + e] = s.p[q];
        }
    };
    auto stash = [&]() {
        if (alds >= 0) {
            uint32_t seen = 0;
            stash_source(std::false_type(), seen);
            if (split_over(seen)) stash_source(std::true_type(), seen);
        }
#pragma unroll
        for (int i = 0; i < WTURNS; ++i)
            if (256 * (i + 1) <= WP || tid + 256 * i < WP) Bs[tid + 256 * i] = __builtin_bit_cast(bf8, wv[i]);
    };
    if (!BWD && tid < 32) bs[tid] = dc0 + tid < g.DC ? as_global((const float *)p.W)[g.b_off + dc0 + tid] : 0.f;
    // the halo columns stay zero
    for (int e = tid; e < 6 * rows * 2; e += 256) {
        const int side = e & 1, r = (e >> 1) % rows, po = (e >> 1) / rows;
        bf8 z;
#pragma unroll
        for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.f;
        As[po * POS + r * WT + side * (W + 1)] = z;
    }

    // ---- the wave's pixel tiles ---------------------------------------------------------------
    int abase[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int px = 32 * (MT * wave + m) + li;
        const int s = px >> g.lgRW, r = px & ((1 << g.lgRW) - 1);
        abase[m] = lh * POS + (s * rowsT + (r >> LGW)) * WT + (r & (W - 1));
    }
    const int bbase = lh * 32 + li;
    f16v main[MT], corr[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) main[m][r] = corr[m][r] = 0.f;

    // ---- epilogue: lane has pixel li of the tile, register r channel dc0 + 8 (r / 4) + 4 lh + r % 4:
    // every access is 128 contiguous bytes of a channel (with the channels over the lanes, 16 bytes
    // each, the requests to L2 took longer than the products)
    auto value = [&](int m, int r, float bias) {
        float v = split_sum(main[m][r], corr[m][r]);
        if (!BWD) v += bias;
        if (!BWD && g.relu && !(v > 0.f)) v = 0.f;
        return v;
    };
    auto store = [&]() {
        if (!BWD && g.pool) {
            constexpr int LGPW = LGW - 1;
            const int PHW = (g.H / 2) << LGPW;
            const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(dst + sample0 * g.DC * PHW, 0, 4 * g.DC * PHW * ns, kBufferFlags);
            const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(amax + sample0 * g.DC * PHW, 0, g.DC * PHW * ns, kBufferFlags);
            const bool odd = li & 1, low = LGW == 4 ? (li & 16) != 0 : (li & 8) != 0;   // column, row of the window
#pragma unroll
            for (int m = 0; m < MT; m += (LGW == 5 ? 2 : 1)) {
                // the four lanes of a window (two, where its rows are in two tiles) look after a channel each
                const int px = 32 * (MT * wave + m) + li, s = px >> g.lgRW, q = px & ((1 << g.lgRW) - 1);
                const int y = y0 + (q >> LGW), x = q & (W - 1);
                const int ch = dc0 + 4 * lh + (odd ? 1 : 0) + (LGW != 5 && low ? 2 : 0);
                const uint32_t o = y < g.H ? (uint32_t)((s * g.DC + ch) * PHW + ((y >> 1) << LGPW) + (x >> 1)) : kNowhere / 4;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (dc0 + 8 * i >= g.DC) break;
                    const f4 bias = *reinterpret_cast<const f4 *>(&bs[8 * i + 4 * lh]);
                    // [channel pair][row of the window, where that is a tile] -> left and right value of the own channel
                    float left[2][2], right[2][2];
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int t = 0; t < (LGW == 5 ? 2 : 1); ++t) {
                            const int mm = m + t < MT ? m + t : MT - 1;
                            const float v0 = value(mm, 4 * i + 2 * c, bias[2 * c]), v1 = value(mm, 4 * i + 2 * c + 1, bias[2 * c + 1]);
                            const float own = odd ? v1 : v0, other = dpp_mov<0xB1>(odd ? v0 : v1);
                            left[c][t] = odd ? other : own;
                            right[c][t] = odd ? own : other;
                        }
#pragma unroll
                    for (int c = 0; c < (LGW == 5 ? 2 : 1); ++c) {
                        float k[4];
                        if (LGW == 5) {
                            k[0] = left[c][0]; k[1] = right[c][0]; k[2] = left[c][1]; k[3] = right[c][1];
                        } else if (LGW == 4) {
                            const auto l = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, left[0][0]), __builtin_bit_cast(int, left[1][0]), false, false);
                            const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, right[0][0]), __builtin_bit_cast(int, right[1][0]), false, false);
                            k[0] = __builtin_bit_cast(float, (int)l[0]); k[2] = __builtin_bit_cast(float, (int)l[1]);
                            k[1] = __builtin_bit_cast(float, (int)r[0]); k[3] = __builtin_bit_cast(float, (int)r[1]);
                        } else {
                            const float lo = low ? left[1][0] : left[0][0], lx = dpp_mov<0x128>(low ? left[0][0] : left[1][0]);
                            const float ro = low ? right[1][0] : right[0][0], rx = dpp_mov<0x128>(low ? right[0][0] : right[1][0]);
                            k[0] = low ? lx : lo; k[2] = low ? lo : lx;
                            k[1] = low ? rx : ro; k[3] = low ? ro : rx;
                        }
                        float best = k[0];
                        int which = 0;
#pragma unroll
                        for (int j = 1; j < 4; ++j)   // row-major: the first maximum wins
                            if (k[j] > best) { best = k[j]; which = j; }
                        const int so = (8 * i + 2 * c) * PHW;
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, best), rd, (int)(4 * o), 4 * so, 0);
                        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)which, ra, (int)o, so, 0);
                    }
                }
            }
            return;
        }
        const int bytes = 4 * g.DC * HW * ns;
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(dst + sample0 * g.DC * HW, 0, bytes, kBufferFlags);
        const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(BWD && mask_src ? mask_src : dst) + sample0 * g.DC * HW, 0, bytes, kBufferFlags);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int px = 32 * (MT * wave + m) + li, s = px >> g.lgRW, q = px & ((1 << g.lgRW) - 1);
            const int y = y0 + (q >> LGW);
            const uint32_t o = y < g.H ? 4u * (uint32_t)((s * g.DC + dc0 + 4 * lh) * HW + y0 * W + q) : kNowhere;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (dc0 + 8 * i >= g.DC) break;
                float k[4];
                f4 bias = {0.f, 0.f, 0.f, 0.f};
                if (BWD && mask_src) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        k[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, (int)o, 4 * (8 * i + e) * HW, 0));
                }
                if (!BWD) bias = *reinterpret_cast<const f4 *>(&bs[8 * i + 4 * lh]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = value(m, 4 * i + e, bias[e]);
                    if (BWD && mask_src && !(k[e] > 0.f)) v = 0.f;
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), rd, (int)o, 4 * (8 * i + e) * HW, 0);
                }
            }
        }
    };

    // (the next chunk is on its way while the products run; a workgroup that went on to further tiles
    // and fetched those ahead as well was no faster: 42.4 ms a job against 40.1)
    fetch(0);
    for (int c0 = 0; c0 < g.SC; c0 += 16) {
        __syncthreads();
        stash();
        __syncthreads();
        if (c0 + 16 < g.SC) fetch(c0 + 16);
        __builtin_amdgcn_sched_barrier(0);
        bf8 a[2][MT][3], b[2][3];
        auto operands = [&](int tap, int set) {
            const int off = (tap / 3) * WT + tap % 3;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                b[set][q] = Bs[bbase + (q * 9 + tap) * 64];
#pragma unroll
                for (int m = 0; m < MT; ++m) a[set][m][q] = As[abase[m] + q * 2 * POS + off];
            }
        };
        operands(0, 0);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            if (tap + 1 < 9) operands(tap + 1, (tap + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);   // the next tap's operands are on their way before the products
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int m = 0; m < MT; ++m) split_mfma(i, b[tap & 1], a[tap & 1][m], main[m], corr[m]);
        }
    }
    store();
}

// ---- backward-weight ----------------------------------------------------------------------------
// g[oc][ci][ky][kx] = sum over samples and pixels of dout[oc][y][x] in[ci][y+ky-1][x+kx-1]
// M = 32 output channels, N = 32 input channels for each of the nine taps, K = pixels in steps of 16 (a
// lane's eight elements are neighbours in a row).  A workgroup accumulates its slice of the client's
// pixels for one (oc, ci) block and writes one partial result, in the layout and for the finish
// kernel of kernels_conv_mfma.hip.  Its six waves are the three filter rows, twice: the two halves
// take turns at the steps and are added at the end.  The three taps of a filter row read the same
// pixels, shifted: the shifted operands are put together from aligned ones, not read.
//
// What bounds it: the staging between two barriers, which only the compute unit's second workgroup
// covers (no registers are left to fetch the next tile ahead: 96 accumulators of 168): the matrix cores are
// busy 36 to 38 % of the time in launches of all 32 clients.  64 -> 64 channels at 16 x 16, 32 clients x 64 samples: 378
// -> 260 us; 32 -> 32 at 32 x 32: 389 -> 278 us.
struct SplitWgrad {
    int IC, OC, H;
    int items;           // tiles of R rows per sample
    int units, U, S;     // 32-pixel units of a client, per slice; slices
    int KP, OCP;         // the partial result's columns and rows
    int cblocks;         // blocks of 32 input channels
};

template <int LGW>
struct SplitWgradTile {
    static constexpr int W = 1 << LGW, R = W == 32 ? 4 : 8, PX = R * W;
    static constexpr int UNITS = PX / 32;                       // of a tile
    static constexpr int RS = W + 8, ROWST = R + 2;             // a row: 8 elements of zeros (x = -1 is the last of them), the pixels
    // 16-byte pieces of a channel, one part; the zeros behind the last row; odd, so that 16 lanes of
    // an operand read meet 16 different places
    static constexpr int IN = (ROWST * RS + 8) / 8 | 1, DO = PX / 8 | 1;
    static constexpr int LDS = 3 * 32 * (IN + DO) * 16;
    static constexpr int OUT = 32 * 288 * 4;                    // the partial result takes the tiles' place
    static_assert(OUT <= LDS || W == 8, "room for the result");
    static constexpr int BYTES = LDS > OUT ? LDS : OUT;
};

constexpr int kWgThreads = 384;

// UNPOOL: as above, dout is the gradient at the outputs of the pooling layer
template <int LGW, bool UNPOOL>
__global__ void __launch_bounds__(kWgThreads, 3)
k_conv_wgrad_split(const RoundParams *__restrict__ rp, int u, int B, SplitWgrad g, const float *__restrict__ in,
                   const float *__restrict__ dout, const uint8_t *__restrict__ amax, float *__restrict__ partial) {
    typedef SplitWgradTile<LGW> T;
    constexpr int W = T::W, R = T::R, IN = T::IN, DO = T::DO, W8 = W / 8;
    if (u >= rp[blockIdx.z].m) return;
    extern __shared__ __attribute__((aligned(16))) bf8 sm[];
    bf8 *const Is = sm;                   // [3][32][IN]
    bf8 *const Ds = sm + 3 * 32 * IN;     // [3][32][DO]
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ky = wave % 3, half = wave / 3;
    const int oc0 = 32 * ((int)blockIdx.y / g.cblocks), ci0 = 32 * ((int)blockIdx.y % g.cblocks);
    const int HW = g.H * W;

    __shared__ bool again;
    if (tid == 0) again = false;
    // zeros around the rows: never written again
    for (int e = tid; e < 3 * 32 * (T::ROWST + 1); e += kWgThreads) {
        bf8 z;
#pragma unroll
        for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.f;
        Is[e / (T::ROWST + 1) * IN + e % (T::ROWST + 1) * (T::RS / 8)] = z;
    }
    // staging: octets of pixels, [channel][row][octet]
    constexpr int ITASKS = 32 * T::ROWST * W8, ITURNS = (ITASKS + kWgThreads - 1) / kWgThreads;
    constexpr int DTASKS = 32 * R * W8, DTURNS = (DTASKS + kWgThreads - 1) / kWgThreads;
    float bsum[DTURNS];
    constexpr int UN = UNPOOL ? 2 : 1, DL = UNPOOL ? 1 : 2;
    const int SHW = HW / (UN * UN);          // a channel of dout
    f4 iv[ITURNS][2], dv[DTURNS][DL];
    uint32_t dw[DTURNS];                     // UNPOOL: the winners of the octet's four windows
    auto fetch = [&](int it) {
        const int b = it / g.items, y0 = (it - b * g.items) * R;
        const int64_t sample = (int64_t)blockIdx.z * B + b;
        const __amdgpu_buffer_rsrc_t ri = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(in) + (sample * g.IC + ci0) * HW, 0, 4 * (g.IC - ci0) * HW, kBufferFlags);
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(dout) + (sample * g.OC + oc0) * SHW, 0, 4 * (g.OC - oc0) * SHW, kBufferFlags);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
            UNPOOL ? const_cast<uint8_t *>(amax) + (sample * g.OC + oc0) * SHW : nullptr, 0, UNPOOL ? (g.OC - oc0) * SHW : 0, kBufferFlags);
#pragma unroll
        for (int i = 0; i < ITURNS; ++i) {
            const int t = tid + kWgThreads * i, x8 = t % W8, row = t / W8 % T::ROWST, c = t / (W8 * T::ROWST);
            const int y = y0 + row - 1;
            const bool ok = t < ITASKS && (unsigned)y < (unsigned)g.H;
            const uint32_t off = ok ? 4u * (uint32_t)(c * HW + y * W + 8 * x8) : kNowhere;
#pragma unroll
            for (int q = 0; q < 2; ++q) iv[i][q] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(ri, (int)off, 16 * q, 0));
        }
#pragma unroll
        for (int i = 0; i < DTURNS; ++i) {
            const int t = tid + kWgThreads * i, o = t % (R * W8), c = t / (R * W8);
            const uint32_t off = t >= DTASKS ? kNowhere
                                 : UNPOOL ? 4u * (uint32_t)(c * SHW + (y0 + o / W8) / 2 * (W / 2) + 4 * (o % W8))
                                          : 4u * (uint32_t)(c * HW + y0 * W + 8 * o);
            if (UNPOOL) dw[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rw, (int)(off >> 2), 0, 0);
#pragma unroll
            for (int q = 0; q < DL; ++q) dv[i][q] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rd, (int)off, 16 * q, 0));
        }
    };
    // A value whose first part became infinite makes the corrections NaN: then all again, with the first parts
    // kept finite.  (A watch in the staging as above costs this kernel 1 to 2 %, this 0.5 %.)
    bool clamp = false;
    // o_lo, o_hi: the pixels of the tile that are this slice's own, in octets (for the bias)
    auto stash = [&](int o_lo, int o_hi) {
#pragma unroll
        for (int i = 0; i < ITURNS; ++i) {
            const int t = tid + kWgThreads * i, x8 = t % W8, row = t / W8 % T::ROWST, c = t / (W8 * T::ROWST);
            if (t < ITASKS) {
                const float x[8] = {iv[i][0][0], iv[i][0][1], iv[i][0][2], iv[i][0][3], iv[i][1][0], iv[i][1][1], iv[i][1][2], iv[i][1][3]};
                Split8 s = split8<false>(x);
                if (__builtin_expect(clamp, 0)) s = split8<true>(x);
#pragma unroll
                for (int q = 0; q < 3; ++q) Is[(q * 32 + c) * IN + row * (T::RS / 8) + 1 + x8] = s.p[q];
            }
        }
#pragma unroll
        for (int i = 0; i < DTURNS; ++i) {
            const int t = tid + kWgThreads * i, o = t % (R * W8), c = t / (R * W8);
            if (t < DTASKS) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)   // (tiles begin in even rows)
                    x[e] = !UNPOOL ? dv[i][e / 4 % DL][e % 4]
                           : ((dw[i] >> (8 * (e / 2))) & 0xffu) == (uint32_t)(2 * (o / W8 & 1) + (e & 1)) ? dv[i][0][e / 2] : 0.f;
                Split8 s = split8<false>(x);
                if (__builtin_expect(clamp, 0)) s = split8<true>(x);
#pragma unroll
                for (int q = 0; q < 3; ++q) Ds[(q * 32 + c) * DO + o] = s.p[q];
                if (o >= o_lo && o < o_hi) bsum[i] += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
            }
        }
    };

    f16v main[3], corr[3];
    const int u0 = (int)blockIdx.x * g.U, u1 = min(u0 + g.U, g.units);
    const uint32_t *const Iw = reinterpret_cast<const uint32_t *>(Is);
    for (;;) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) main[k][r] = corr[k][r] = 0.f;
#pragma unroll
        for (int i = 0; i < DTURNS; ++i) bsum[i] = 0.f;
        for (int it = u0 / T::UNITS; it * T::UNITS < u1; ++it) {
            fetch(it);
            const int lo = max(u0 - it * T::UNITS, 0), hi = min(u1 - it * T::UNITS, T::UNITS);
            __syncthreads();   // the products of the previous tile are done with the tiles
            stash(4 * lo, 4 * hi);
            __syncthreads();
            for (int un = lo; un < hi; ++un) {
                const int o = 4 * un + 2 * half + lh;      // the lane's octet of the tile
                const int row = o / W8 + ky, x8 = o % W8;
                bf8 a[3], b[3][3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    a[q] = Ds[(q * 32 + li) * DO + o];
                    const int at = (q * 32 + li) * IN + row * (T::RS / 8) + 1 + x8;
                    const u4 c = __builtin_bit_cast(u4, Is[at]);
                    const uint32_t l = Iw[4 * at - 1], r = Iw[4 * at + 4];
                    const uint32_t m1 = __builtin_amdgcn_alignbit(c[1], c[0], 16), m2 = __builtin_amdgcn_alignbit(c[2], c[1], 16),
                                   m3 = __builtin_amdgcn_alignbit(c[3], c[2], 16);
                    b[0][q] = __builtin_bit_cast(bf8, u4{(uint32_t)__builtin_amdgcn_alignbit(c[0], l, 16), m1, m2, m3});
                    b[1][q] = __builtin_bit_cast(bf8, c);
                    b[2][q] = __builtin_bit_cast(bf8, u4{m1, m2, m3, (uint32_t)__builtin_amdgcn_alignbit(r, c[3], 16)});
                }
#pragma unroll
                for (int i = 0; i < 6; ++i)
#pragma unroll
                    for (int k = 0; k < 3; ++k) split_mfma(i, a, b[k], main[k], corr[k]);
            }
        }
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += corr[k][r];
        if (sum != sum) again = true;
        __syncthreads();   // (the products are done with the tiles too)
        if (clamp || !again) break;
        clamp = true;
    }

    // ---- partial[client][slice][oc][k], k = ci * 9 + tap: the halves are added in LDS ----------------
    float *const out = reinterpret_cast<float *>(sm);     // [32][288]
    const gf_ptr pg = as_global(partial) + ((int64_t)blockIdx.z * g.S + blockIdx.x) * g.OCP * g.KP;
    if (ci0 == 0) {   // the bias column: the threads of a channel are neighbours in a row of 16 lanes (of 8)
#pragma unroll
        for (int i = 0; i < DTURNS; ++i) {
            float v = bsum[i];
            v += dpp_mov<0xB1>(v);
            v += dpp_mov<0x4E>(v);
            v += dpp_mov<0x141>(v);
            if (R * W8 == 16) v += dpp_mov<0x140>(v);
            const int t = tid + kWgThreads * i, c = t / (R * W8);
            if (t < DTASKS && t % (R * W8) == 0 && oc0 + c < g.OC) pg[(int64_t)(oc0 + c) * g.KP + 9 * g.IC] = v;
        }
    }
#pragma unroll
    for (int h = 1; h >= 0; --h) {
        if (half == h) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float *p = out + (8 * (r / 4) + 4 * lh + r % 4) * 288 + li * 9 + 3 * ky + k;
                    const float v = split_sum(main[k][r], corr[k][r]);
                    *p = h == 1 ? v : v + *p;
                }
        }
        __syncthreads();
    }
    const int cols4 = min(32, g.IC - ci0) * 9 / 4, rows = min(32, g.OC - oc0);   // IC is a multiple of 16
    for (int e = tid; e < rows * cols4; e += kWgThreads) {
        const int r = e / cols4, c = e - r * cols4;
        *reinterpret_cast<f4 __attribute__((address_space(1))) *>(pg + (int64_t)(oc0 + r) * g.KP + 9 * ci0 + 4 * c) =
            *reinterpret_cast<const f4 *>(out + r * 288 + 4 * c);
    }
}

// ---- the weights of a recursion, split ------------------------------------------------------
// A layer's weights in one direction are pieces of 16 source and 32 destination channels, each as the
// LDS holds it: [part][tap][octet][32][8], [chunk of source channels][block of destination channels].
// Splitting them in the convolution's own staging, once per workgroup, took 132 of its 819 vector
// instructions and wrote LDS with up to nine lanes to a bank.
constexpr int kSplitPiece = 6 * 9 * 32 * 16;   // bytes
constexpr int kSplitJobs = 32;   // 16 layers, both directions
struct SplitJob {
    char *dst;
    int64_t w_off;
    int ic, oc, bwd, nblk, piece0;
};
struct SplitJobs {
    SplitJob j[kSplitJobs];
    int n;
};

__global__ void __launch_bounds__(192)
k_split_weights(const RoundParams *__restrict__ rp, int u, SplitJobs jobs, int64_t stride) {
    const RoundParams p = rp[blockIdx.z];
    if (u >= p.m) return;
    int ji = 0;
    while (ji + 1 < jobs.n && (int)blockIdx.x >= jobs.j[ji + 1].piece0) ++ji;
    const SplitJob j = jobs.j[ji];
    const int piece = (int)blockIdx.x - j.piece0, c0 = 16 * (piece / j.nblk), d0 = 32 * (piece % j.nblk);
    const gcf_ptr W = as_global((const float *)p.W) + j.w_off;
    u4 *dst = reinterpret_cast<u4 *>(j.dst + blockIdx.z * stride * 16) + (int64_t)piece * (kSplitPiece / 16);
    const int lim = j.bwd ? j.ic : j.oc;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int t = (int)threadIdx.x + 192 * i;            // (tap, octet, destination channel)
        const int tap = t >> 6, o = (t >> 5) & 1, d = d0 + (t & 31), c = c0 + 8 * o;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            x[e] = d >= lim ? 0.f : j.bwd ? W[((int64_t)(c + e) * j.ic + d) * 9 + 8 - tap] : W[((int64_t)d * j.ic + c + e) * 9 + tap];
        const Split8 s = split8<true>(x);
#pragma unroll
        for (int q = 0; q < 3; ++q) dst[q * 576 + t] = __builtin_bit_cast(u4, s.p[q]);
    }
}

// both maps are the same size: 3 x 3, padding 1; MT: pixel tiles per wave
bool split_dir(const LayerGeom &L, bool bwd, int MT, SplitDir *d) {
    if (L.type != 0 || L.k != 3 || L.pad != 1 || L.ic % 16 != 0 || L.oc % 16 != 0) return false;
    const int W = L.iw, PX = 128 * MT;
    if (W != 8 && W != 16 && W != 32) return false;
    d->ic = L.ic; d->oc = L.oc; d->relu = L.relu; d->pool = 0;
    d->SC = bwd ? L.oc : L.ic; d->DC = bwd ? L.ic : L.oc;
    d->H = L.ih;
    d->w_off = L.w_off; d->b_off = L.b_off;
    if (L.ih == W && L.ih * W < PX) {          // several samples per workgroup
        d->R = L.ih; d->NS = PX / (L.ih * W); d->rblocks = 1;
    } else {
        d->R = PX / W; d->NS = 1; d->rblocks = (L.ih + d->R - 1) / d->R;
    }
    d->lgRW = 0;
    while (1 << d->lgRW < d->R * W) ++d->lgRW;
    // 32-bit byte offsets
    return (int64_t)L.in_size * d->NS < (int64_t)1 << 28 && (int64_t)L.out_size * d->NS < (int64_t)1 << 28 &&
           (int64_t)L.oc * L.ic * 9 < (int64_t)1 << 28;
}

constexpr int kSplitResident = 512;   // workgroups of a launch that are resident together: two per compute unit

template <int LGW, int MT, bool BWD, bool UNPOOL>
hipError_t split_launch(hipStream_t s, dim3 grid, const RoundParams *dp, int u, int B, const SplitDir &d, const u4 *w,
                        int64_t wstride, const float *src, float *dst, const float *mask_src, uint8_t *amax) {
    constexpr int lds = SplitTile<LGW, MT>::LDS;
    if (lds > 64 * 1024) {
        int dev = 0, done = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        static PerDevice allowed;
        e = allowed.get(dev, &done, [](int *v) {
            *v = 1;
            return hipFuncSetAttribute(reinterpret_cast<const void *>(k_conv_split<LGW, MT, BWD, UNPOOL>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        });
        if (e != hipSuccess) return e;
    }
    k_conv_split<LGW, MT, BWD, UNPOOL><<<grid, 256, lds, s>>>(dp, u, B, d, w, wstride, src, dst, mask_src, amax);
    return hipGetLastError();
}

}  // namespace

// Where this form is the faster one, time here / with kernels_conv_mfma.hip, forward | backward-data,
// by the workgroups' worth of tiles of 256 pixels x 32 destination channels:
//                     96            128           192           512           768 and more
//   32 x 32 px  1.00 | 1.07                  0.70 | 0.85   0.71 | 0.71   0.75 | 0.83
//   16 x 16     1.02 | 1.07   1.01 | 1.06   0.72 | 0.73   0.62 | 0.74   0.74 | 0.84
//   8 x 8       0.71 | 0.73   0.72 | 0.73   0.50 | 0.54   0.44 | 0.47
// (8 x 8 images fill half a workgroup there; 32 x 32 and 32 channels, 1,536 | 3,072 | 8,192 workgroups'
// worth: forward 0.66, 0.63, 0.62, backward-data 0.69, 0.77, 0.77, and 0.57, 0.53, 0.62 where it takes the
// pooled gradient, with the pooling kernel's time on the other side.)  Below that a launch is a chain of trips through
// memory, one for each chunk of channels, on either.  16 destination channels fill half a
// tile: 0.9 to 1.4 everywhere.
static bool conv_split_pays(const LayerGeom &L, bool bwd, int B, int nact) {
    SplitDir d;
    if (!split_dir(L, bwd, 2, &d) || d.DC < 32) return false;
    const int64_t wgs = (int64_t)d.rblocks * ((B + d.NS - 1) / d.NS) * ((d.DC + 31) / 32) * nact;
    return wgs >= (L.iw == 8 ? 96 : 192);
}

// (the rule is taken by the more clients, the more often)
size_t conv_split_weight_bytes(const LayerGeom &L, bool bwd, int B, int n_clients) {
    SplitDir d;
    return conv_split_pays(L, bwd, B, n_clients) && split_dir(L, bwd, 2, &d) ? (size_t)(d.SC / 16) * ((d.DC + 31) / 32) * kSplitPiece : 0;
}

bool conv_split_used(const LayerGeom *lay, int l, bool bwd, int B, int nact, const SplitWeights &sw) {
    return sw.base && sw.off[l][bwd] >= 0 && conv_split_pays(lay[l], bwd, B, nact);
}

hipError_t launch_split_weights(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, const LayerGeom *lay, int L, int B,
                                const SplitWeights &sw) {
    SplitJobs jobs;
    jobs.n = 0;
    int pieces = 0;
    for (int l = 0; l < L; ++l)
        for (int bwd = 0; bwd < 2; ++bwd) {
            if (!conv_split_used(lay, l, bwd, B, nact, sw)) continue;
            SplitJob &j = jobs.j[jobs.n++];
            j.bwd = bwd;
            j.ic = lay[l].ic; j.oc = lay[l].oc;
            j.w_off = lay[l].w_off;
            j.dst = sw.base + sw.off[l][bwd];
            j.piece0 = pieces;
            j.nblk = ((bwd ? lay[l].ic : lay[l].oc) + 31) / 32;
            pieces += (bwd ? lay[l].oc : lay[l].ic) / 16 * j.nblk;
        }
    if (pieces == 0) return hipSuccess;
    const bool timed = prof && prof->on[F_CONV_FWD];   // for both directions
    if (timed) prof->before(F_CONV_FWD, s);
    k_split_weights<<<dim3((unsigned)pieces, 1, (unsigned)nact), 192, 0, s>>>(dp, u, jobs, sw.stride);
    if (timed) prof->after(F_CONV_FWD, s);
    return hipGetLastError();
}

hipError_t launch_conv_split(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int u, int B,
                             const LayerGeom &L, bool bwd, const SplitWeights &sw, int64_t off, const float *src, float *dst,
                             const float *mask_src, uint8_t *amax) {
    SplitDir d;
    const u4 *w = reinterpret_cast<const u4 *>(sw.base + off);
    const int MT = 2;
    if (!split_dir(L, bwd, MT, &d)) return hipErrorInvalidValue;
    d.pool = !bwd && amax;
    const dim3 grid((unsigned)((d.DC + 31) / 32), (unsigned)(d.rblocks * ((B + d.NS - 1) / d.NS)), (unsigned)nact);
    const int fam = bwd ? F_CONV_BWD_DATA : F_CONV_FWD;
    const bool timed = prof && prof->on[fam];
    if (timed) prof->before(fam, s);
    hipError_t e = hipErrorInvalidValue;
#define AET_SPLIT(lgw, mt)                                                                                                     \
    if (L.iw == 1 << lgw && MT == mt)                                                                                          \
        e = !bwd   ? split_launch<lgw, mt, false, false>(s, grid, dp, u, B, d, w, sw.stride, src, dst, mask_src, amax)         \
            : amax ? split_launch<lgw, mt, true, true>(s, grid, dp, u, B, d, w, sw.stride, src, dst, mask_src, amax)           \
                   : split_launch<lgw, mt, true, false>(s, grid, dp, u, B, d, w, sw.stride, src, dst, mask_src, amax);
    AET_SPLIT(3, 2) AET_SPLIT(4, 2) AET_SPLIT(5, 2)
#undef AET_SPLIT
    if (timed) prof->after(fam, s);
    return e;
}

// ---- backward-weight -----------------------------------------------------------------------------
template <int LGW, bool UNPOOL>
static hipError_t wgrad_split_launch(hipStream_t s, dim3 grid, const RoundParams *dp, int u, int B, const SplitWgrad &g,
                                     const float *in, const float *dout, const uint8_t *amax, float *partial) {
    constexpr int lds = SplitWgradTile<LGW>::BYTES;
    if (lds > 64 * 1024) {
        int dev = 0, done = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        static PerDevice allowed;
        e = allowed.get(dev, &done, [](int *v) {
            *v = 1;
            return hipFuncSetAttribute(reinterpret_cast<const void *>(k_conv_wgrad_split<LGW, UNPOOL>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        });
        if (e != hipSuccess) return e;
    }
    k_conv_wgrad_split<LGW, UNPOOL><<<grid, kWgThreads, lds, s>>>(dp, u, B, g, in, dout, amax, partial);
    return hipGetLastError();
}

// Where it is the faster form, time here / with kernels_conv_mfma.hip, finish included:
//   more than one block of 32 x 32 channels: 0.54 .. 0.91 at every size
//   one block, by its pixels / 256   up to 32       48 .. 128      192           512 and more
//     32 -> 32 channels              0.64 .. 1.08   0.96 .. 1.14   0.83 .. 0.98   0.67 .. 0.88
//     16 -> 32                       0.71 .. 1.12   0.96 .. 1.25   0.94 .. 0.97   0.81 .. 0.82
//     16 -> 16                       0.97 .. 1.13   1.02 .. 1.34   1.07 .. 1.15   1.01 .. 1.16
// (CNN on 32 x 32, 32 clients, 4 rounds: 42.6 -> 37.0 ms.)
int conv_wgrad_split_slices(const LayerGeom &L, int B, int nact, int cap) {
    if (L.type != 0 || L.k != 3 || L.pad != 1 || L.ic % 16 != 0 || L.oc % 16 != 0) return 0;
    const int W = L.iw, R = W == 32 ? 4 : 8;
    if ((W != 8 && W != 16 && W != 32) || L.ih % R != 0) return 0;
    if (L.in_size >= (int64_t)1 << 28 || L.out_size >= (int64_t)1 << 28) return 0;   // 32-bit byte offsets
    const int pairs = ((L.oc + 31) / 32) * ((L.ic + 31) / 32), units = B * L.ih * W / 32;
    if (pairs == 1 && (L.ic * L.oc < 512 || (int64_t)units * nact < 8 * 192)) return 0;
    int S = kSplitResident / (nact * pairs);
    if (S * nact > cap) S = cap / nact;
    if (S < 1) S = 1;
    const int U = (units + S - 1) / S;
    return (units + U - 1) / U;   // the fewest slices with the same longest share
}

hipError_t launch_conv_wgrad_split(hipStream_t s, const RoundParams *dp, int nact, int u, int B, const LayerGeom &L, int S, int KP,
                                   int OCP, const float *in, const float *dout, const uint8_t *amax, float *partial) {
    SplitWgrad g;
    g.IC = L.ic; g.OC = L.oc; g.H = L.ih;
    const int W = L.iw, R = W == 32 ? 4 : 8;
    g.items = L.ih / R;
    g.units = B * L.ih * W / 32;
    g.U = (g.units + S - 1) / S;
    g.S = S;
    g.KP = KP; g.OCP = OCP;
    g.cblocks = (L.ic + 31) / 32;
    const dim3 grid((unsigned)S, (unsigned)((L.oc + 31) / 32 * g.cblocks), (unsigned)nact);
#define AET_WGRAD_SPLIT(lgw)                                                                   \
    if (W == 1 << lgw)                                                                         \
        return amax ? wgrad_split_launch<lgw, true>(s, grid, dp, u, B, g, in, dout, amax, partial) \
                    : wgrad_split_launch<lgw, false>(s, grid, dp, u, B, g, in, dout, amax, partial);
    AET_WGRAD_SPLIT(3) AET_WGRAD_SPLIT(4) AET_WGRAD_SPLIT(5)
#undef AET_WGRAD_SPLIT
    return hipErrorInvalidValue;
}

}  // namespace aet
