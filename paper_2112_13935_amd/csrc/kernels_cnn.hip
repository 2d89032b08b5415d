// Fused local round for small convolutional networks: 3 x 3 convolutions with padding 1, each with
// an optional 2 x 2 pooling layer behind it, then a hidden dense layer and the classes.
//
// One launch = one round of every active client.  A client is a cluster of G workgroups on one XCD, A of
// which take whole samples of the mini-batch (workgroup g takes g, g + A, ...): every activation and every
// gradient of a sample stays in its workgroup's LDS from the gathered row to the gradient of the
// first filter, the convolutions run on the matrix cores straight from there, and the only things that
// cross workgroups are, once per recursion,
//   up:    each workgroup's sum of the filters' gradients, and of each sample the inputs and
//          gradients of the two dense layers;
//   down:  the updated weights.  The gradients are added, w <- w - eta g and U <- U + g applied, by all
//          workgroups of the cluster in equal shares, in a fixed order (workgroups, samples ascending).
// Two barriers of the cluster separate the two (tagged words, as in the other fused rounds).
//
// What bounds it: the chain of one sample, a step for each layer each way (eight for four convolutions) with a barrier of
// the workgroup between them.  A step of a small layer is some 4,000 clocks of scalar and address work, LDS
// latency and its epilogue, in a large one the fp32 matrix instructions (32 clocks each) take
// as much again; the two barriers of the cluster and three trips through L2 (weights, dense layers,
// gradients) are a quarter of a recursion.  Of its 130 K clocks (16 x 16 half-width CNN, mini-batch 16): forward 33 K,
// backward-data 37 K, filter gradients 26 K, dense layers and softmax 19 K, update and barriers 13 K.  The layer
// engine spends 13 - 15 launches on a recursion, each a launch boundary and two to four dependent trips through memory.
// 6 clients of that CNN with compute factors, 6 rounds: 5.93 -> 3.63 ms; 12 x 12, 6 and 12 channels, 3 clients, mini-batch
// 5, 6 rounds: 1.94 -> 0.84 ms.  Sixteen waves of 128 registers: eight of 256 took 10 - 30 % longer in the
// products, which wait for LDS.  One body for both directions of the convolutions, and steps worked out by the
// host: with each form written out the kernel had 84 KB of code, more than the instruction cache
// holds, and took 1.7 times as long.  The update by whole waves, filters and dense layers side by side
// and not one after the other: 14.5 -> 9.2 K clocks.  Workgroups without samples of their own help with the update (one
// sample per recursion: 105 -> 59 us); how many there are is the launch's to say, and no sum depends on it.
//
// Layout of a map in LDS: a plane per channel, rows of W + 1 floats of which the first is zero (left
// edge of its row and right edge of the one before), a row of zeros above and below.  So every tap of a
// filter is the pixel's address plus a number, and the gradient of a filter is a dot product over
// consecutive floats.  Planes are 20 floats apart modulo 32: four channels by sixteen pixels (forward,
// backward-data) and sixteen channels by four pixels (gradient) both spread over the banks.
//
// The filters' weights are kept twice more, as images: rows in the order in which the contraction walks
// them, forward and turned round for the way down, so that a workgroup stages them as they lie.  Where all images
// fit in LDS together they are staged once per recursion (12 x 12 above: 0.96 -> 0.89 ms).
#include <type_traits>

#include "aet_device.h"
#include "aet_internal.h"
#include "cluster_plan.h"
#include "cluster_post.h"

namespace aet {

namespace {

typedef unsigned long long u64;
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kCnWaves = 16;
constexpr int kCnThreads = 64 * kCnWaves;
constexpr int kCnConvs = 7;        // convolutions, at most
constexpr int kCnSteps = 16;       // chunks of weights of all layers and directions, at most
constexpr int kCnPrefetch = 4096 / kCnThreads;   // 16-byte pieces of the next weights that a thread has on the way
constexpr int kCnChunk = 4 * kCnThreads * kCnPrefetch;   // floats of weights staged at a time, at most
constexpr int kCnRow = 4096 / kCnThreads;        // floats of the next sample that a thread has on the way
constexpr int kCnBatch = 16;       // values of a sum over workgroups or samples on the way at a time
constexpr int kCnRed = kCnWaves * 256;   // floats of the partial sums of split tiles; two such places take turns
constexpr int kNowhere = -2147483647 - 1;   // a byte offset beyond every buffer: reads zero, writes nothing

typedef int i16v __attribute__((ext_vector_type(16)));

// One step of a sample's way up or down the convolutions: a chunk of one layer's weights in one direction.
// The numbers come in three records of sixteen, so that each is one scalar load.
//   P: the product (taps over planes)
enum { P_KIND, P_TILES, P_MTILES, P_DIVM, P_HW, P_AT, P_SRC, P_PL, P_SWP, P_KROW, P_ROWS, P_NCQ, P_LG, P_WBUF, P_NEXT, P_FLOATS };
enum { K_NONE, K_UP, K_WINDOWS, K_DOWN, K_UNPOOL };   // kinds: forward, forward pooled; gradient of the input, of a pooled one
//   E: where its results go, and the edges that are cleared on the way
enum { E_DST, E_DPL, E_DSWP, E_AT, E_RELU, E_MASK, E_MPL, E_MAT, E_WIN, E_WPL, E_CLEAR, E_CPL, E_CPLANES, E_CH, E_CSWP };
//   G: the gradient of the filters (G_TILES 0: not in this step)
enum { G_TILES, G_LG, G_COLS, G_DIVC, G_PER, G_OC, G_NI, G_DEL, G_DPL, G_SRC, G_AT, G_WOFF, G_BOFF, G_CELLS };
struct CnnStep { i16v p, e, g; };

// Tables in LDS that save the steps their divisions, in 16-bit places.
struct CnnTable {
    int at, n;             // first place, places
    int w, swp, windows;   // pixel m of a map w wide in rows of swp floats, row by row or window by window ...
    int pl;                // ... or, where not 0, column m of the filters: channel m / 9, planes pl apart, tap m % 9
};

struct CnnPlan {
    CnnStep step[kCnSteps];
    int nsteps, turn;                  // steps; the first on the way down
    int first, first_floats;           // the first chunk of weights
    int B, G, A;                       // mini-batch; workgroups of a cluster, at most, and those of them that take samples
    int F0, H, C, relu_h;              // dense: F0 -> H -> C
    int w1, b1, w2, b2;                // offsets into the parameters
    int conv_params;                   // they come first
    int in_size, in_w, in_hw, in_src, in_pl;
    int feat, hid, dhid, logit;        // LDS: inputs and gradients of the dense layers
    int wbuf, red;                     // LDS: staged weights, partial sums of split tiles
    int lds_floats;
    // the gradient of the features: its planes, the uppermost convolution
    int t_del, t_pl, t_planes, t_h, t_swp, t_clear, t_relu, t_pool, t_win, t_per, t_w;
    unsigned t_divper, t_divw;
    int nconv, ntables;
    CnnTable table_of[3 * kCnConvs + 1];
    int rec, rec_h, rec_d1, rec_d2, rec_loss, records;   // a sample's record: features, hidden, gradients, loss
    int part, partials;                // a workgroup's gradients of the filters
    int table;                         // where each filter weight lies in the two images
    int client_floats;                 // scratch floats per client
    struct Conv { int ic, oc, kf, kb, image_f, image_b, w_off, b_off; } conv[kCnConvs];
};

typedef const CnnPlan __attribute__((address_space(4))) ConstantPlan;

// n / d for n * d < 2^32: div = ceil(2^32 / d), or 0 for d = 1
__device__ __forceinline__ unsigned quotient(unsigned n, unsigned div) { return div ? __umulhi(n, div) : n; }

// ---- words that other workgroups of the cluster write or read --------------------------------------
// They carry no tag: what makes them visible is the cluster's barrier, which waits until the L2 (or, where the cluster
// is on several XCDs, memory) has acknowledged the workgroup's stores before it posts its tagged word.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const float *p, int floats) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, 4 * floats, kBufferFlags);
}
// at: in bytes; base: in floats, the same for the whole wave
__device__ __forceinline__ float get1(__amdgpu_buffer_rsrc_t r, int at, int base) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, at, 4 * base, kAgent));
}
__device__ __forceinline__ f4 get4(__amdgpu_buffer_rsrc_t r, int at, int base) {
    return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, at, 4 * base, kAgent));
}
__device__ __forceinline__ void put1(__amdgpu_buffer_rsrc_t r, int at, int base, float v, bool one_xcd) {
    if (one_xcd) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, at, 4 * base, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, at, 4 * base, kAgent);
}

__device__ __forceinline__ f4 mfma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// ---- sums over the lanes of a wave: lane swaps of gfx950 between rows, DPP inside a row of 16 -----------
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
struct Two { float a, b; };
__device__ __forceinline__ Two swap32(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, x), __builtin_bit_cast(int, y), false, false);
    return {__builtin_bit_cast(float, (int)r[0]), __builtin_bit_cast(float, (int)r[1])};
}
__device__ __forceinline__ Two swap16(float x, float y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, x), __builtin_bit_cast(int, y), false, false);
    return {__builtin_bit_cast(float, (int)r[0]), __builtin_bit_cast(float, (int)r[1])};
}
__device__ __forceinline__ float row_sum(float v) {
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    v += dpp<0x140>(v);
    return v;
}
__device__ __forceinline__ float all_sum(float v) {
    Two t = swap32(v, v);
    v = t.a + t.b;
    t = swap16(v, v);
    return row_sum(t.a + t.b);
}
__device__ __forceinline__ float all_max(float v) {
    Two t = swap32(v, v);
    v = fmaxf(t.a, t.b);
    t = swap16(v, v);
    v = fmaxf(t.a, t.b);
    v = fmaxf(v, dpp<0xB1>(v));
    v = fmaxf(v, dpp<0x4E>(v));
    v = fmaxf(v, dpp<0x141>(v));
    return fmaxf(v, dpp<0x140>(v));
}
// four sums at once: row r of 16 lanes gets the sum of v[r]
__device__ __forceinline__ float rows_sum(const float (&v)[4]) {
    const Two p = swap32(v[0], v[2]), q = swap32(v[1], v[3]);   // lanes 0 .. 31: v[0], v[1]; the others v[2], v[3]
    const Two t = swap16(p.a + p.b, q.a + q.b);
    return row_sum(t.a + t.b);
}

// ---- products over channels and taps (forward, backward-data) --------------------------------------
// acc += sum over channel groups cq0 .. cq1 - 1 and nine taps.  a: the lane's pixel (top left tap) in the
// plane of channel lg; b: the lane's row of the weights' image, element lg.
__device__ __forceinline__ void taps(f4 &acc, const float *lds, int a, int pl4, int swp, int b, int cq0, int cq1) {
    struct Ops { float a[9], b[9]; };
    const float *ap = lds + a + cq0 * pl4, *bp = lds + b + 36 * cq0;
    auto load = [&](Ops &o) {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                o.a[3 * ky + kx] = ap[ky * swp + kx];
                o.b[3 * ky + kx] = bp[4 * (3 * ky + kx)];
            }
        ap += pl4;
        bp += 36;
    };
    auto products = [&](const Ops &o) {
#pragma unroll
        for (int t = 0; t < 9; ++t) acc = mfma(o.a[t], o.b[t], acc);
    };
    Ops x, y;
    const int n = cq1 - cq0;
    if (n <= 0) return;
    load(x);
#pragma unroll 1
    for (int i = 2; i <= n; i += 2) {
        load(y);
        products(x);
        if (i < n) load(x);
        products(y);
    }
    if (n & 1) products(x);
}

// acc += sum over n groups of 16 floats of a plane: gradient a (the lane's channel, its four floats of a
// group) times input b (the lane's channel and tap)
__device__ __forceinline__ void pixels(f4 &acc, const float *lds, int a, int b, int n) {
    struct Ops { f4 a; float b[4]; };
    const float *ap = lds + a, *bp = lds + b;
    auto load = [&](Ops &o) {
        o.a = *reinterpret_cast<const f4 *>(ap);
#pragma unroll
        for (int j = 0; j < 4; ++j) o.b[j] = bp[j];
        ap += 16;
        bp += 16;
    };
    auto products = [&](const Ops &o) {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = mfma(o.a[j], o.b[j], acc);
    };
    Ops x[2], y[2];
    if (n <= 0) return;
    // (what is loaded beyond the last group is not multiplied)
    load(x[0]);
    load(x[1]);
#pragma unroll 1
    for (;;) {
        load(y[0]);
        load(y[1]);
        products(x[0]);
        if (n > 1) products(x[1]);
        n -= 2;
        if (n <= 0) break;
        load(x[0]);
        load(x[1]);
        products(y[0]);
        if (n > 1) products(y[1]);
        n -= 2;
        if (n <= 0) break;
    }
}

// The tiles of a product dealt over the waves: whole rounds, then the remainder, each of whose contractions is
// split over 1 << lg_rest waves.  body(acc, tile, part, log2 parts) adds up, store(acc, tile) is for the
// wave of part 0.  Holds a barrier for everybody where the remainder is split.
template <class Body, class Store>
__device__ __forceinline__ void deal_tiles(int tiles, int lg_rest, float *red, Body body, Store store) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int whole = lg_rest ? tiles & ~(kCnWaves - 1) : tiles;
#pragma unroll 1
    for (int t0 = 0; t0 < tiles; t0 += kCnWaves) {
        const bool split = t0 >= whole;
        const int lg = split ? lg_rest : 0, t = t0 + (wave >> lg), part = wave & ((1 << lg) - 1);
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
        if (t < tiles) body(acc, t, part, lg);
        if (split) {
            if (part > 0) *reinterpret_cast<f4 *>(red + 4 * (64 * wave + lane)) = acc;
            __syncthreads();
            if (part == 0)
                for (int q = 1; q < 1 << lg; ++q) acc += *reinterpret_cast<const f4 *>(red + 4 * (64 * (wave + q) + lane));
        }
        if (t < tiles && part == 0) store(acc, t);
    }
}

// Zero edges of the planes of a gradient buffer that another geometry may have used.
__device__ __forceinline__ void clear_edges(float *lds, int base, int pl, int planes, int h, int swp) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int top = swp + 1, mid = h - 1, tail = (h + 1) * swp;
    for (int t = lane; t < top + mid + pl - tail; t += 64) {
        const int at = t < top ? t : t < top + mid ? (t - top + 2) * swp : tail + t - top - mid;
        for (int c = wave; c < planes; c += kCnWaves) lds[base + c * pl + at] = 0.f;
    }
}

__global__ void __launch_bounds__(kCnThreads, 1)
k_cnn_round(const RoundParams *__restrict__ rp, int nact, int G, int first, const float *Wg, const CnnPlan *plan, float *scratch, u64 *words,
            u64 *places, u64 *claims, int skew, uint32_t tag0, int *errflag) {
    const ConstantPlan &g = *(const ConstantPlan *)plan;   // read with scalar loads
    extern __shared__ __attribute__((aligned(16))) float lds[];
    uint8_t *const lds8 = reinterpret_cast<uint8_t *>(lds);
    // Workgroups with ids equal modulo 8 share an XCD; which one begins differs from queue to queue.  Where the launch has
    // to know (others are beside it), client 0 is on XCD `first` and the workgroup asks where it is.
    const int xcd = (first < 0 ? (int)blockIdx.x : xcc_id() - first) & 7, slot = blockIdx.x >> 3;
    const int who = (slot / G) * 8 + xcd, me = slot % G;   // client of the launch, workgroup of its cluster
    if (who >= nact) return;
    const RoundParams p = rp[who];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    bool dead = false;
    u64 *const place = places ? places + (size_t)p.client * kPlaces : nullptr;
    if (first < 0) cluster_announce(place, me, tag0, skew);
    else if (!cluster_claim(claims + (size_t)p.client * kPlaces, me, tag0, skew, lds)) return;

    float *const mine = scratch + (size_t)p.client * g.client_floats;   // the client's scratch memory
    const gf_ptr U = as_global(p.U);
    const gcf_ptr W0 = as_global(Wg ? Wg : p.W);
    const int Pc = g.conv_params;
    const __amdgpu_buffer_rsrc_t rw = buffer_of(p.W, g.b2 + g.C), rs = buffer_of(mine, g.client_floats);
    u64 *const word = words + (size_t)p.client * whole_lines(kClusterMax);
    uint32_t tag = tag0;

    for (int e = tid; e < g.lds_floats; e += kCnThreads) lds[e] = 0.f;
    __syncthreads();
    int16_t *const lds16 = reinterpret_cast<int16_t *>(lds);
    for (int k = 0; k < g.ntables; ++k) {
        const auto &c = g.table_of[k];
        for (int m = tid; m < c.n; m += kCnThreads) {
            int v;
            if (c.pl) {
                const int ic = m / 9, t = m - 9 * ic;
                v = ic * c.pl + (t / 3 - 1) * c.swp + t % 3 - 1;
            } else if (c.windows) {
                const int win = m >> 2, wy = win / (c.w >> 1), wx = win - wy * (c.w >> 1);
                v = (2 * wy + (m >> 1 & 1)) * c.swp + 2 * wx + (m & 1);
            } else {
                const int y = m / c.w;
                v = y * c.swp + m - y * c.w;
            }
            lds16[c.at + m] = (int16_t)v;
        }
    }

    // the rows: workgroup `me` takes samples me, me + A, ... of a recursion
    const int B = g.B;
    float xrow[kCnRow];
    int label = 0;
    auto fetch_row = [&](int u, int b) {
        if (u >= p.m) return;
        const uint32_t row = sample_row(p.key, (uint64_t)(p.q0 + (int64_t)u * B + b), p.n_samples);
        const gcf_ptr X = as_global(p.X) + (int64_t)row * g.in_size;
        label = as_global(p.y)[row];
#pragma unroll
        for (int j = 0; j < kCnRow; ++j) xrow[j] = X[min(tid + kCnThreads * j, g.in_size - 1)];
    };
    int xat[kCnRow];   // where those floats go
#pragma unroll
    for (int j = 0; j < kCnRow; ++j) {
        const int e = tid + kCnThreads * j;
        const int ch = e / g.in_hw, r = e - ch * g.in_hw, y = r / g.in_w;
        xat[j] = e < g.in_size ? g.in_src + ch * g.in_pl + (y + 1) * (g.in_w + 1) + r - y * g.in_w + 1 : -1;
    }
    if (me < g.A) fetch_row(0, me);

    const bool one_xcd = cluster_on_one_xcd(place, me, G, tag0, errflag, &dead);
    // all of the cluster's stores before it are there after it
    auto cluster_barrier = [&]() {
        ++tag;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (wave == 0) {
            if (lane == 0) cluster_post(word + me, tag, 0.f, one_xcd);
            BoundedWait wait;
            while (!dead) {
                const u64 v = __hip_atomic_load(word + min(lane, G - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__all((uint32_t)(v >> 32) >= tag)) break;
                if (wait.gave_up(errflag)) dead = true;
            }
        }
        __syncthreads();
        asm volatile("" ::: "memory");
    };

    // ---- the start: images of the filters, the replica, U ----------------------------------------------
    // where a filter's weight lies in the two images; kept in a table that only the thread that wrote it reads
    typedef int i2 __attribute__((ext_vector_type(2)));
    typedef i2 __attribute__((address_space(1))) *i2_ptr;
    const i2_ptr table = (i2_ptr)(mine + g.table);
    auto image_places = [&](int i) {
        i2 at = {kNowhere, kNowhere};
        for (int l = 0; l < g.nconv; ++l) {
            const auto &c = g.conv[l];
            const int per = 9 * c.ic;
            if (i >= c.w_off && i < c.w_off + c.oc * per) {
                const int k = i - c.w_off, oc = k / per, r = k - oc * per, ic = r / 9, t = r - 9 * ic;
                at[0] = 4 * (c.image_f + oc * c.kf + ((ic >> 2) * 9 + t) * 4 + (ic & 3));
                if (l > 0) at[1] = 4 * (c.image_b + ic * c.kb + ((oc >> 2) * 9 + 8 - t) * 4 + (oc & 3));
            } else if (i >= c.b_off && i < c.b_off + c.oc) {   // the bias: behind the row's weights
                at[0] = 4 * (c.image_f + (i - c.b_off) * c.kf + 36 * ((c.ic + 3) >> 2));
            }
        }
        return at;
    };
    // The parameters' owners, by the wave: 64 filter weights, or 64 columns of four units of a dense layer (the
    // last column of a layer is its biases).  Wave w of workgroup g takes pieces 16 g + w, ...
    const int conv_pieces = (Pc + 63) >> 6, cols1 = (g.F0 + 64) >> 6, cols2 = (g.H + 64) >> 6;
    const int pieces1 = conv_pieces + ((g.H + 3) >> 2) * cols1, pieces = pieces1 + ((g.C + 3) >> 2) * cols2;
    struct Item { bool second; int u0, f, F, un, first, step; };   // first: of the units' weights, step from one to the next
    auto dense_item = [&](int piece) {
        Item o;
        o.second = piece >= pieces1;
        const int r = piece - (o.second ? pieces1 : conv_pieces), n = o.second ? cols2 : cols1, q = r / n;
        o.u0 = 4 * q;
        o.f = 64 * (r - q * n) + lane;
        o.F = o.second ? g.H : g.F0;
        o.un = o.f <= o.F ? min(4, (o.second ? g.C : g.H) - o.u0) : 0;   // 0: no such column
        const bool bias = o.f >= o.F;
        o.first = bias ? (o.second ? g.b2 : g.b1) + o.u0 : (o.second ? g.w2 : g.w1) + o.u0 * o.F + o.f;
        o.step = bias ? 1 : o.F;
        return o;
    };
    // (the images' padding, channels and taps that do not exist, is zero)
    for (int e = me * kCnThreads + tid; e < g.rec; e += G * kCnThreads) put1(rs, 4 * e, 0, 0.f, one_xcd);
    cluster_barrier();
    for (int piece = me * kCnWaves + wave; piece < pieces; piece += G * kCnWaves) {
        if (piece < conv_pieces) {
            const int i = 64 * piece + lane;
            if (i < Pc) {
                const float w = W0[i];
                const i2 at = image_places(i);
                put1(rs, at[0], 0, w, one_xcd);
                put1(rs, at[1], 0, w, one_xcd);
                if (Wg) put1(rw, 4 * i, 0, w, one_xcd);
                U[i] = 0.f;
                table[i] = at;
            }
            continue;
        }
        const Item o = dense_item(piece);
        for (int j = 0; j < o.un; ++j) {
            const int i = o.first + j * o.step;
            if (Wg) put1(rw, 4 * i, 0, W0[i], one_xcd);
            U[i] = 0.f;
        }
    }
    cluster_barrier();

    // ---- weights on their way from the images to LDS (a load beyond the chunk asks for nothing) ---------
    f4 wv[kCnPrefetch];
    auto fetch_weights = [&](int at, int floats) {
#pragma unroll
        for (int j = 0; j < kCnPrefetch; ++j) {
            const int e = 4 * (tid + kCnThreads * j);
            wv[j] = get4(rs, e < floats ? 4 * e : kNowhere, at);
        }
    };
    auto stash_weights = [&](int floats) {
#pragma unroll
        for (int j = 0; j < kCnPrefetch; ++j) {
            const int e = 4 * (tid + kCnThreads * j);
            if (e < floats) *reinterpret_cast<f4 *>(lds + g.wbuf + e) = wv[j];
        }
    };
    const float invB = 1.0f / (float)B;
    float loss_acc = 0.f;

    for (int u = 0; u < p.m; ++u) {
        for (int b = me; b < B && me < g.A; b += g.A) {
            fetch_weights(g.first, g.first_floats);
            const int rec = g.rec + b * g.records, part = g.part + me * g.partials;
            const bool again = b > me;   // not the workgroup's first sample of the recursion
            const int lab = label;
#pragma unroll
            for (int j = 0; j < kCnRow; ++j)
                if (xat[j] >= 0) lds[xat[j]] = xrow[j];
            if (again) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the sums of the samples before have arrived
            stash_weights(g.first_floats);
            __syncthreads();

#pragma unroll 1
            for (int t = 0; t < g.nsteps; ++t) {
                if (t == g.turn) {
                    // ---- dense layers, softmax -------------------------------------------------------------------
                    // a wave per four units; Q * 64 inputs on the way at a time
                    auto dense = [&](auto q_const, int F, int N, int w_off, int b_off, int in, int out, bool relu) {
                        constexpr int Q = decltype(q_const)::value;
#pragma unroll 1
                        for (int u0 = 4 * wave; u0 < N; u0 += 4 * kCnWaves) {
                            float acc[4] = {0.f, 0.f, 0.f, 0.f};
                            const float bias = get1(rw, 4 * min(u0 + lg, N - 1), b_off);
#pragma unroll 1
                            for (int f0 = 0; f0 < F; f0 += 64 * Q) {
                                float w[Q][4];
#pragma unroll
                                for (int q = 0; q < Q; ++q)
#pragma unroll
                                    for (int j = 0; j < 4; ++j)
                                        w[q][j] = get1(rw, 4 * min(f0 + 64 * q + lane, F - 1), w_off + min(u0 + j, N - 1) * F);
#pragma unroll
                                for (int q = 0; q < Q; ++q) {
                                    const int f = f0 + 64 * q + lane;
                                    const float x = f < F ? lds[in + f] : 0.f;
#pragma unroll
                                    for (int j = 0; j < 4; ++j) acc[j] += w[q][j] * x;
                                }
                            }
                            float z = rows_sum(acc) + bias;
                            if (relu) z = fmaxf(z, 0.f);
                            if (li == 0 && u0 + lg < N) lds[out + u0 + lg] = z;
                        }
                    };
                    if (g.F0 > 128) dense(std::integral_constant<int, 8>{}, g.F0, g.H, g.w1, g.b1, g.feat, g.hid, g.relu_h != 0);
                    else dense(std::integral_constant<int, 2>{}, g.F0, g.H, g.w1, g.b1, g.feat, g.hid, g.relu_h != 0);
                    __syncthreads();
                    dense(std::integral_constant<int, 2>{}, g.H, g.C, g.w2, g.b2, g.hid, g.logit, false);
                    __syncthreads();
                    if (wave == 0) {
                        const bool real = lane < g.C;
                        const float z = real ? lds[g.logit + lane] : -INFINITY;   // (a finite value could be above the logits)
                        const float zmax = all_max(z);
                        const float lse = zmax + logf(all_sum(real ? expf(z - zmax) : 0.f));
                        const float dz = real ? expf(z - lse) - (lane == lab ? 1.f : 0.f) : 0.f;
                        lds[g.logit + lane] = dz;
                        if (real) put1(rs, 4 * lane, rec + g.rec_d2, dz, one_xcd);
                        if (lane == lab) put1(rs, 0, rec + g.rec_loss, lse - z, one_xcd);
                    }
                    __syncthreads();
                    // d(hidden), masked (the gradients of classes and units that do not exist are zero)
                    for (int f = tid; f < g.H; f += kCnThreads) {
                        float d = 0.f;
                        for (int o0 = 0; o0 < g.C; o0 += 16) {
                            float w[16];
#pragma unroll
                            for (int j = 0; j < 16; ++j) w[j] = get1(rw, 4 * f, g.w2 + min(o0 + j, g.C - 1) * g.H);
#pragma unroll
                            for (int j = 0; j < 16; ++j) d += w[j] * lds[g.logit + o0 + j];
                        }
                        const float h = lds[g.hid + f];
                        if (g.relu_h && !(h > 0.f)) d = 0.f;
                        lds[g.dhid + f] = d;
                        put1(rs, 4 * f, rec + g.rec_h, h, one_xcd);
                        put1(rs, 4 * f, rec + g.rec_d1, d, one_xcd);
                    }
                    __syncthreads();
                    // sum over units o0 .. o1 - 1 of gradient times weight
                    auto features = [&](int f, int o0, int o1) {
                        float d = 0.f;
#pragma unroll 1
                        for (; o0 < o1; o0 += 32) {
                            float w[32];
#pragma unroll
                            for (int j = 0; j < 32; ++j) w[j] = get1(rw, 4 * f, g.w1 + min(o0 + j, g.H - 1) * g.F0);
#pragma unroll
                            for (int j = 0; j < 32; j += 4) {
                                const f4 dh = *reinterpret_cast<const f4 *>(lds + g.dhid + o0 + j);
                                d += w[j] * dh[0] + w[j + 1] * dh[1] + (w[j + 2] * dh[2] + w[j + 3] * dh[3]);
                            }
                        }
                        return d;
                    };
                    if (g.t_clear) clear_edges(lds, g.t_del, g.t_pl, g.t_planes, g.t_h, g.t_swp);
                    // d(features), masked and put where the maxima came from.  Up to half as many features as
                    // threads: two threads a feature, the first half of the units and the second
                    const bool halves = 2 * g.F0 <= kCnThreads && g.H > 32;
                    const int mid = halves ? (g.H / 2 + 31) & ~31 : g.H;
                    if (halves) {
                        const int f = tid - kCnThreads / 2;
                        if (f >= 0 && f < g.F0) lds[g.red + f] = features(f, mid, g.H);
                        else if (tid < g.F0) lds[g.red + g.F0 + tid] = features(tid, 0, mid);
                        __syncthreads();
                    }
#pragma unroll 1
                    for (int f = tid; f < g.F0; f += kCnThreads) {
                        float d = halves ? lds[g.red + g.F0 + f] + lds[g.red + f] : features(f, 0, g.H);
                        const float a = lds[g.feat + f];
                        put1(rs, 4 * f, rec, a, one_xcd);
                        if (g.t_relu && !(a > 0.f)) d = 0.f;
                        const int ch = (int)quotient((unsigned)f, g.t_divper), r = f - ch * g.t_per;
                        const int y = (int)quotient((unsigned)r, g.t_divw), x = r - y * g.t_w;
                        float *const plane = lds + g.t_del + ch * g.t_pl;
                        if (g.t_pool) {
                            const int at = lds8[g.t_win + f];
                            float *const to = plane + (2 * y + 1) * g.t_swp + 2 * x + 1;
                            to[0] = at == 0 ? d : 0.f;
                            to[1] = at == 1 ? d : 0.f;
                            to[g.t_swp] = at == 2 ? d : 0.f;
                            to[g.t_swp + 1] = at == 3 ? d : 0.f;
                        } else {
                            plane[(y + 1) * g.t_swp + x + 1] = d;
                        }
                    }
                    __syncthreads();
                }

                // ---- a step: taps over planes -----------------------------------------------------------------
                const i16v P = g.step[t].p, E = g.step[t].e;
                // The weights of the next step are on their way meanwhile.  Nothing else is when they are asked
                // for: where older loads may be pending on some way here, the compiler waits for all
                // of them, these too, as soon as it takes one of the older ones' registers.
                __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
                if (P[P_FLOATS]) fetch_weights(P[P_NEXT], P[P_FLOATS]);
                if (t == 0) {   // so is the next row
                    if (b + g.A < B) fetch_row(u, b + g.A);
                    else fetch_row(u + 1, me);
                }
                if (E[E_CPLANES]) clear_edges(lds, E[E_CLEAR], E[E_CPL], E[E_CPLANES], E[E_CH], E[E_CSWP]);
                const int kind = P[P_KIND], ncq = P[P_NCQ];
                if (kind != K_NONE)
                    deal_tiles(P[P_TILES], P[P_LG], lds + g.red,
                        [&](f4 &acc, int tile, int part_, int lgp) {
                            const int n = (int)quotient((unsigned)tile, (unsigned)P[P_DIVM]), mt = tile - n * P[P_MTILES];
                            const int at = lds16[P[P_AT] + min(16 * mt + li, P[P_HW] - 1)];
                            taps(acc, lds, P[P_SRC] + __mul24(lg, P[P_PL]) + at, 4 * P[P_PL], P[P_SWP],
                                 P[P_WBUF] + __mul24(min(16 * n + li, P[P_ROWS] - 1), P[P_KROW]) + lg, ncq * part_ >> lgp, ncq * (part_ + 1) >> lgp);
                        },
                        [&](const f4 &acc, int tile) {
                            // the lane has channel 16 n + li, four consecutive pixels
                            const int n = (int)quotient((unsigned)tile, (unsigned)P[P_DIVM]), mt = tile - n * P[P_MTILES];
                            const int row = 16 * n + li, m0 = 16 * mt + 4 * lg;
                            if (row >= P[P_ROWS] || m0 >= P[P_HW]) return;
                            float *const dst = lds + E[E_DST] + __mul24(row, E[E_DPL]);
                            if (kind <= K_WINDOWS) {
                                const float bias = lds[P[P_WBUF] + __mul24(row, P[P_KROW]) + 36 * ncq];
                                float v[4];
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    v[r] = acc[r] + bias;
                                    if (E[E_RELU]) v[r] = fmaxf(v[r], 0.f);
                                }
                                if (kind == K_WINDOWS) {
                                    int at = 0;
                                    float best = v[0];
#pragma unroll
                                    for (int r = 1; r < 4; ++r)
                                        if (v[r] > best) best = v[r], at = r;
                                    dst[lds16[E[E_AT] + (m0 >> 2)]] = best;
                                    lds8[E[E_WIN] + __mul24(row, E[E_WPL]) + (m0 >> 2)] = (uint8_t)at;
                                } else {
#pragma unroll
                                    for (int r = 0; r < 4; ++r)
                                        if (m0 + r < P[P_HW]) dst[lds16[E[E_AT] + m0 + r]] = v[r];
                                }
                                return;
                            }
                            // the gradient of what went through a ReLU, of the maxima's places
                            const float *const below = lds + E[E_MASK] + __mul24(row, E[E_MPL]);
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int m = min(m0 + r, P[P_HW] - 1);
                                const float d = E[E_RELU] && !(below[lds16[E[E_MAT] + m]] > 0.f) ? 0.f : acc[r];
                                if (kind == K_DOWN) {
                                    if (m0 + r < P[P_HW]) dst[lds16[E[E_AT] + m]] = d;
                                } else if (m0 + r < P[P_HW]) {
                                    const int at = lds8[E[E_WIN] + __mul24(row, E[E_WPL]) + m];
                                    float *const to = dst + lds16[E[E_AT] + 4 * m];
                                    to[0] = at == 0 ? d : 0.f;
                                    to[1] = at == 1 ? d : 0.f;
                                    to[E[E_DSWP]] = at == 2 ? d : 0.f;
                                    to[E[E_DSWP] + 1] = at == 3 ? d : 0.f;
                                }
                            }
                        });
                // ---- gradient of the filters ---------------------------------------------------------------------
                // (hidden, so that a step's third record is loaded here: all three at once fill half of the scalar registers, and what they
                // push out comes back through vector ones.  Us a job: 3 clients, 12 x 12 images, 6 channels 853 -> 841; 8, 8 x 8, 6
                // channels 592 -> 582; 6, 16 x 16, 16 channels 3,662 -> 3,630; 20, 12 x 12, 24 channels 1,403 -> 1,389.)
                const i16v Q = g.step[opaque_scalar(t)].g;
                if (Q[G_TILES]) {
                    const int ni = Q[G_NI], per = Q[G_PER];
                    deal_tiles(Q[G_TILES], Q[G_LG], lds + g.red + kCnRed,
                        [&](f4 &acc, int tile, int part_, int lgp) {
                            const int mg = (int)quotient((unsigned)tile, (unsigned)Q[G_DIVC]), n = tile - mg * Q[G_COLS];
                            const int i0 = ni * part_ >> lgp, i1 = ni * (part_ + 1) >> lgp, from = 4 * lg + 16 * i0;
                            pixels(acc, lds, Q[G_DEL] + __mul24(min(16 * mg + li, Q[G_OC] - 1), Q[G_DPL]) + from,
                                   Q[G_SRC] + lds16[Q[G_AT] + min(16 * n + li, per - 1)] + from, i1 - i0);
                        },
                        [&](const f4 &acc, int tile) {
                            const int mg = (int)quotient((unsigned)tile, (unsigned)Q[G_DIVC]), n = tile - mg * Q[G_COLS], col = 16 * n + li;
                            const int oc = 16 * mg + 4 * lg, base = part + Q[G_WOFF];
                            f4 sum = acc;
                            const int at0 = 4 * (__mul24(oc, per) + col), left = col < per ? Q[G_OC] - oc : 0;
                            int at[4];
#pragma unroll
                            for (int r = 0; r < 4; ++r) at[r] = r < left ? at0 : kNowhere;
                            if (again) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) sum[r] += get1(rs, at[r], base + r * per);
                            }
                            if (one_xcd) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) put1(rs, at[r], base + r * per, sum[r], true);
                            } else {
#pragma unroll
                                for (int r = 0; r < 4; ++r) put1(rs, at[r], base + r * per, sum[r], false);
                            }
                        });
                    // the biases: sums over the planes (the edges are zero)
                    for (int oc = wave; oc < Q[G_OC]; oc += kCnWaves) {
                        float sum = 0.f;
                        for (int e = lane; e < Q[G_CELLS]; e += 64) sum += lds[Q[G_DEL] + oc * Q[G_DPL] + e];
                        sum = all_sum(sum);
                        if (lane == 0) {
                            if (again) sum += get1(rs, 4 * oc, part + Q[G_BOFF]);
                            put1(rs, 4 * oc, part + Q[G_BOFF], sum, one_xcd);
                        }
                    }
                }
                __syncthreads();
                if (P[P_FLOATS]) {
                    stash_weights(P[P_FLOATS]);
                    __syncthreads();
                }
            }
        }
        cluster_barrier();

        // ---- this workgroup's share of the sums and of the update -----------------------------------------
#pragma unroll 1
        for (int piece = me * kCnWaves + wave; piece < pieces; piece += G * kCnWaves) {
            if (piece < conv_pieces) {
                const int i = min(64 * piece + lane, Pc - 1);
                const float w = get1(rw, 4 * i, 0), uo = U[i];
                const i2 at = table[i];
                float sum = 0.f;
#pragma unroll 1
                for (int k0 = 0; k0 < g.A; k0 += kCnBatch) {
                    float v[kCnBatch];
#pragma unroll
                    for (int k = 0; k < kCnBatch; ++k) v[k] = get1(rs, 4 * i, g.part + min(k0 + k, g.A - 1) * g.partials);
#pragma unroll
                    for (int k = 0; k < kCnBatch; ++k)
                        if (k0 + k < g.A) sum += v[k];
                }
                if (64 * piece + lane < Pc) {
                    const float gr = sum * invB, wn = w - p.eta * gr;
                    put1(rw, 4 * i, 0, wn, one_xcd);
                    put1(rs, at[0], 0, wn, one_xcd);
                    put1(rs, at[1], 0, wn, one_xcd);
                    U[i] = uo + gr;
                }
                continue;
            }
            const Item o = dense_item(piece);
            const bool bias = o.f >= o.F;
            const int in = 4 * ((o.second ? g.rec_h : 0) + min(o.f, o.F - 1)), out = (o.second ? g.rec_d2 : g.rec_d1) + o.u0;
            float w[4], uo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = o.first + max(min(j, o.un - 1), 0) * o.step;
                w[j] = get1(rw, o.un > 0 ? 4 * i : kNowhere, 0);
                uo[j] = U[o.un > 0 ? i : 0];
            }
            f4 sum = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int b0 = 0; b0 < B; b0 += kCnBatch) {
                // the units' gradients are the same for all lanes: lane k brings sample b0 + k's
                const f4 d = get4(rs, 4 * min(b0 + (lane & (kCnBatch - 1)), B - 1) * g.records, g.rec + out);
                float a[kCnBatch];
#pragma unroll
                for (int k = 0; k < kCnBatch; ++k) a[k] = get1(rs, in, g.rec + min(b0 + k, B - 1) * g.records);
#pragma unroll
                for (int k = 0; k < kCnBatch; ++k) {
                    const float x = b0 + k >= B ? 0.f : bias ? 1.f : a[k];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float dj = d[j];   // (a bit cast of the element itself takes the first one's bits)
                        sum[j] += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dj), k)) * x;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < o.un) {
                    const int i = o.first + j * o.step;
                    const float gr = sum[j] * invB;
                    put1(rw, 4 * i, 0, w[j] - p.eta * gr, one_xcd);
                    U[i] = uo[j] + gr;
                }
        }
        if (me == G - 1 && wave == kCnWaves - 1) {   // the mini-batch's loss
            float t = 0.f;
            for (int b = lane; b < B; b += 64) t += get1(rs, 4 * b * g.records, g.rec + g.rec_loss);
            loss_acc += all_sum(t) * invB;
        }
        cluster_barrier();
    }
    if (me == G - 1 && tid == kCnThreads - 64) *as_global(p.loss) = loss_acc;
}

// The plan, from the kernel's arguments to where every launch reads it.  (Arguments are in host memory, and
// a workgroup goes through three kilobytes of them once per recursion.)
__global__ void k_put_plan(const CnnPlan g, CnnPlan *dst, int *errflag) {
    const int n = (int)(sizeof(CnnPlan) / 4);
    for (int i = threadIdx.x; i < n; i += blockDim.x) reinterpret_cast<int *>(dst)[i] = reinterpret_cast<const int *>(&g)[i];
    if (threadIdx.x == 0) *errflag = 0;
}

__global__ void k_zero_words_cnn(u64 *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

int up(int x, int to) { return (x + to - 1) / to * to; }

// floats from one plane to the next: the map with its edges, whole groups of 16 for the gradients
// of the filters, 20 modulo 32
int plane_floats(int h, int w) {
    const int swp = w + 1, q0 = swp & ~3;
    int need = (h + 2) * swp + 1;
    if (need < q0 + up(h * swp + swp - q0, 16)) need = q0 + up(h * swp + swp - q0, 16);
    return need + ((20 - need) & 31);
}

unsigned reciprocal(int d) { return d > 1 ? (unsigned)((0xFFFFFFFFull + d) / d) : 0u; }   // for quotient()

// log2 of the waves that share a tile of the last, partial round: as many as there are, at most max_parts
int split_of(int tiles, int max_parts) {
    const int rem = tiles % kCnWaves;
    int lg = 0;
    while (rem > 0 && (rem << (lg + 1)) <= kCnWaves && (2 << lg) <= max_parts) ++lg;
    return lg;
}

// The plan of a network, or false if it is not of this kind or does not fit.
bool cnn_plan(const LayerGeom *lay, int L, int B, int n_clients, CnnPlan *g) {
    *g = CnnPlan{};
    if (L < 3 || lay[L - 1].type != 2 || lay[L - 2].type != 2 || lay[0].type != 0) return false;
    if (lay[L - 1].relu || lay[L - 1].oc > 64 || B < 1) return false;
    struct Map {
        int ic, oc, h, w, relu, pool, swp, pl;     // pl: of the planes of its input and of its output's gradient
        int lin, pairs, out, cols;                 // tables: pixels, pixels by windows, of the output, columns of the filters
        int src, act, act_pl, act_swp, win, del;   // LDS: input planes, output (0, 0), winners (bytes), gradient
        int kf, kb, chunk_f, chunk_b;              // floats of a row of the images, rows staged at a time
    } map[kCnConvs];
    g->B = B;
    const int turns = (B + kClusterMax - 1) / kClusterMax;   // samples per workgroup
    g->A = (B + turns - 1) / turns;
    int n = 0, params = 0;
    for (int l = 0; l < L - 2; ++l) {
        const LayerGeom &q = lay[l];
        if (q.type != 0 || q.k != 3 || q.pad != 1 || n == kCnConvs) return false;
        if (q.ih > 32 || q.iw > 32 || q.oc > 1024 || q.ic > 1024) return false;
        Map &c = map[n];
        CnnPlan::Conv &o = g->conv[n++];
        c.ic = o.ic = q.ic; c.oc = o.oc = q.oc; c.h = q.ih; c.w = q.iw; c.relu = q.relu;
        c.swp = c.w + 1;
        c.pl = plane_floats(c.h, c.w);
        o.w_off = (int)q.w_off; o.b_off = (int)q.b_off;
        if (o.w_off != params || o.b_off != o.w_off + c.oc * 9 * c.ic) return false;
        params = o.b_off + c.oc;
        c.pool = l + 1 < L - 2 && lay[l + 1].type == 1;
        if (c.pool) ++l;
        // rows of the images: 2 modulo 32 floats apart, room for the bias behind the weights
        auto row = [](int channels) { const int k = 36 * ((channels + 3) / 4) + 1; return k + ((2 - k) & 31); };
        c.kf = o.kf = row(c.ic);
        c.kb = o.kb = row(c.oc);
    }
    if (!n) return false;
    const LayerGeom &d1 = lay[L - 2], &d2 = lay[L - 1];
    if (d1.in_size > 4096 || d1.oc > 1024) return false;
    g->nconv = n;
    g->conv_params = params;
    g->F0 = (int)d1.in_size; g->H = d1.oc; g->C = d2.oc; g->relu_h = d1.relu;
    g->w1 = (int)d1.w_off; g->b1 = (int)d1.b_off; g->w2 = (int)d2.w_off; g->b2 = (int)d2.b_off;
    // Where compute units are left over, workgroups that take no samples help with the update: as many as an
    // XCD has room for beside the other clients', up to one per two thousand parameters.
    const int per_xcd = (n_clients + 7) / 8, room_for = kClusterMax / (per_xcd < kClusterMax ? per_xcd : kClusterMax);
    const int wanted = ((int)(d2.b_off + d2.oc) + 2047) / 2048, helped = wanted < room_for ? wanted : room_for;
    g->G = helped > g->A ? helped : g->A;
    g->in_size = (int)lay[0].in_size;
    if (g->in_size > kCnRow * kCnThreads) return false;
    // LDS: the input planes of every convolution, what goes to the dense layers, winners
    int at = 16;
    for (int l = 0; l < n; ++l) {
        map[l].src = at;
        at += up(map[l].ic, 4) * map[l].pl;
        if (at > 40960) return false;
    }
    g->in_w = map[0].w; g->in_hw = map[0].h * map[0].w; g->in_src = map[0].src; g->in_pl = map[0].pl;
    g->feat = at; at += up(g->F0, 4);
    g->hid = at; at += up(g->H, 4);
    g->dhid = at; at += up(g->H, 32);   // read in whole groups
    g->logit = at; at += 64;
    for (int l = 0; l < n; ++l) {
        Map &c = map[l];
        const int oh = c.pool ? c.h / 2 : c.h, ow = c.pool ? c.w / 2 : c.w;
        c.win = 0;
        if (c.pool) { c.win = 4 * at; at += up(c.oc * oh * ow, 16) / 4; }
        if (l + 1 == n) { c.act = g->feat; c.act_swp = ow; c.act_pl = oh * ow; }
        else { c.act = map[l + 1].src + map[l + 1].swp + 1; c.act_swp = map[l + 1].swp; c.act_pl = map[l + 1].pl; }
    }
    // tables, each once
    at = up(at, 4);
    int place16 = 2 * at;
    auto table = [&](int m, int w, int swp, int windows, int pl) {
        for (int k = 0; k < g->ntables; ++k) {
            const CnnTable &o = g->table_of[k];
            if (o.n == m && o.w == w && o.swp == swp && o.windows == windows && o.pl == pl) return o.at;
        }
        g->table_of[g->ntables++] = {place16, m, w, swp, windows, pl};
        place16 += up(m, 4);
        return place16 - up(m, 4);
    };
    for (int l = 0; l < n; ++l) {
        Map &c = map[l];
        if (c.ic * c.pl + c.swp > 32767) return false;
        c.lin = table(c.h * c.w, c.w, c.swp, 0, 0);
        c.pairs = c.pool ? table(c.h * c.w, c.w, c.swp, 1, 0) : c.lin;
        c.cols = table(9 * c.ic, 0, c.swp, 0, c.pl);
    }
    for (int l = 0; l < n; ++l) {
        Map &c = map[l];
        const int ow = c.pool ? c.w / 2 : c.w;
        c.out = l + 1 < n ? map[l + 1].lin : table(c.act_pl, ow, ow, 0, 0);
    }
    at = up((place16 + 1) / 2, 4);
    // the gradients: two buffers that take turns, or two for each geometry where there is room (their
    // edges are then cleared once)
    int most = 0;
    auto place_gradients = [&](int from, bool apart) {
        int end = from, base[2] = {0, 0}, size[2] = {0, 0};
        for (int l = n - 1; l >= 0; --l) {
            Map &c = map[l];
            const int turn = l & 1, need = up(c.oc, 4) * c.pl;
            if (apart) {
                bool found = false;
                for (int k = n - 1; k > l && !found; --k)
                    if ((k & 1) == turn && map[k].pl == c.pl && map[k].w == c.w && map[k].h == c.h && up(map[k].oc, 4) >= up(c.oc, 4)) {
                        c.del = map[k].del;
                        found = true;
                    }
                if (!found) { c.del = end; end += need; }
            } else if (need > size[turn]) {
                size[turn] = need;
            }
        }
        if (!apart) {
            base[0] = end; base[1] = end + size[0];
            end += size[0] + size[1];
            for (int l = 0; l < n; ++l) map[l].del = base[l & 1];
        }
        return up(end + 40, 4);   // the last group of a dot product may read past the planes
    };
    auto place_weights = [&](int from) {   // the staged weights, or 0
        const int room = 160 * 256 - from, lim = room < kCnChunk ? room / 4 * 4 : kCnChunk;
        most = 0;
        for (int l = 0; l < n; ++l) {
            Map &c = map[l];
            auto chunk = [&](int rows, int k) { return up(rows * k, 4) <= lim ? rows : lim / k / 16 * 16; };
            c.chunk_f = lim > 0 ? chunk(c.oc, c.kf) : 0;
            c.chunk_b = lim <= 0 ? 0 : l > 0 ? chunk(c.ic, c.kb) : c.ic;
            if (c.chunk_f < 1 || c.chunk_b < 1) return false;
            const int f = up(c.chunk_f * c.kf, 4), b = l > 0 ? up(c.chunk_b * c.kb, 4) : 0;
            most = f > most ? f : most;
            most = b > most ? b : most;
        }
        return true;
    };
    // the images; all of them stay in LDS for a whole sample where they fit beside the rest
    int64_t image = 0;
    for (int l = 0; l < n; ++l) {
        g->conv[l].image_f = (int)image; image += up(map[l].oc * map[l].kf, 32);
        g->conv[l].image_b = (int)image; image += l > 0 ? up(map[l].ic * map[l].kb, 32) : 0;
    }
    bool apart = true, resident = false;
    int end = place_gradients(at, true);
    auto whole = [&] {   // no layer's weights come in more than one chunk
        for (int l = 0; l < n; ++l)
            if (map[l].chunk_f < map[l].oc || map[l].chunk_b < map[l].ic) return false;
        return true;
    };
    if (!place_weights(end + 2 * kCnRed) || !whole()) {
        apart = false;
        end = place_gradients(at, false);
        if (!place_weights(end + 2 * kCnRed)) return false;
    }
    g->red = end;
    g->wbuf = end + 2 * kCnRed;
    if (image <= kCnChunk && g->wbuf + image <= 160 * 256) {
        resident = true;
        most = (int)image;
        for (int l = 0; l < n; ++l) { map[l].chunk_f = map[l].oc; map[l].chunk_b = map[l].ic; }
    }
    g->lds_floats = g->wbuf + most;
    if (4 * g->lds_floats > 160 * 1024) return false;
    // the client's scratch memory: images, records, gradients of the filters, table
    g->rec = (int)image;
    g->rec_h = up(g->F0, 4);
    g->rec_d1 = g->rec_h + up(g->H, 4);
    g->rec_d2 = g->rec_d1 + up(g->H, 4);
    g->rec_loss = g->rec_d2 + up(g->C, 4);
    g->records = up(g->rec_loss + 1, 32);
    g->partials = up(params, 32);
    const int64_t part = image + (int64_t)B * g->records, tab = part + (int64_t)g->A * g->partials, total = tab + up(2 * params, 32);
    if (total > (1 << 26)) return false;
    g->part = (int)part; g->table = (int)tab; g->client_floats = (int)total;
    // the steps: each names the weights of the one after it
    auto dirty = [&](int l) {   // the buffer of this gradient was last used with other planes
        if (apart) return false;
        const Map &c = map[l];
        for (int k = 0; k < n; ++k)
            if ((k & 1) == (l & 1) && (map[k].w != c.w || map[k].h != c.h || map[k].pl != c.pl)) return true;
        return false;
    };
    int previous = -1;
    auto append = [&](int l, bool bwd, int r0) {
        if (g->nsteps == kCnSteps) return false;
        const Map &c = map[l];
        CnnStep &st = g->step[g->nsteps];
        const int outs = bwd ? c.ic : c.oc, chunk = bwd ? c.chunk_b : c.chunk_f, rows = outs - r0 < chunk ? outs - r0 : chunk;
        const int hw = c.h * c.w, mtiles = (hw + 15) / 16, nt = (rows + 15) / 16;
        const bool product = !bwd || l > 0;
        if (product) {
            const int floats = up(rows * (bwd ? c.kb : c.kf), 4), from = (bwd ? g->conv[l].image_b + r0 * c.kb : g->conv[l].image_f + r0 * c.kf);
            st.p[P_WBUF] = g->wbuf + (resident ? from : 0);
            if (previous < 0) { g->first = from; g->first_floats = resident ? (int)image : floats; }
            else if (!resident) { g->step[previous].p[P_NEXT] = from; g->step[previous].p[P_FLOATS] = floats; }
            previous = g->nsteps;
            st.p[P_TILES] = mtiles * nt; st.p[P_MTILES] = mtiles; st.p[P_DIVM] = (int)reciprocal(mtiles);
            st.p[P_LG] = split_of(mtiles * nt, ((bwd ? c.oc : c.ic) + 3) / 4);
            st.p[P_HW] = hw; st.p[P_AT] = bwd ? c.lin : c.pairs;
            st.p[P_SRC] = bwd ? c.del : c.src; st.p[P_PL] = c.pl; st.p[P_SWP] = c.swp;
            st.p[P_KROW] = bwd ? c.kb : c.kf; st.p[P_ROWS] = rows; st.p[P_NCQ] = ((bwd ? c.oc : c.ic) + 3) / 4;
            if (!bwd) {
                st.p[P_KIND] = c.pool ? K_WINDOWS : K_UP;
                st.e[E_DST] = c.act + r0 * c.act_pl; st.e[E_DPL] = c.act_pl; st.e[E_AT] = c.out; st.e[E_RELU] = c.relu;
                st.e[E_WIN] = c.win + r0 * (hw / 4); st.e[E_WPL] = hw / 4;
            } else {
                const Map &o = map[l - 1];
                st.p[P_KIND] = o.pool ? K_UNPOOL : K_DOWN;
                st.e[E_DST] = o.del + r0 * o.pl + o.swp + 1; st.e[E_DPL] = o.pl; st.e[E_DSWP] = o.swp; st.e[E_AT] = o.pool ? o.pairs : c.lin;
                st.e[E_RELU] = o.relu; st.e[E_MASK] = c.src + r0 * c.pl + c.swp + 1; st.e[E_MPL] = c.pl; st.e[E_MAT] = c.lin;
                st.e[E_WIN] = o.win + r0 * hw; st.e[E_WPL] = hw;
                if (r0 == 0 && dirty(l - 1)) {
                    st.e[E_CLEAR] = o.del; st.e[E_CPL] = o.pl; st.e[E_CPLANES] = up(o.oc, 4); st.e[E_CH] = o.h; st.e[E_CSWP] = o.swp;
                }
            }
        }
        if (bwd && r0 + rows == outs) {
            const int per = 9 * c.ic, cols = (per + 15) / 16, q0 = c.swp & ~3;
            st.g[G_TILES] = cols * ((c.oc + 15) / 16); st.g[G_LG] = split_of(st.g[G_TILES], (c.h * c.swp + c.swp - q0 + 15) / 16); st.g[G_COLS] = cols; st.g[G_DIVC] = (int)reciprocal(cols);
            st.g[G_PER] = per; st.g[G_OC] = c.oc; st.g[G_NI] = (c.h * c.swp + c.swp - q0 + 15) / 16;
            st.g[G_DEL] = c.del + q0; st.g[G_DPL] = c.pl; st.g[G_SRC] = c.src + q0; st.g[G_AT] = c.cols;
            st.g[G_WOFF] = g->conv[l].w_off; st.g[G_BOFF] = g->conv[l].b_off; st.g[G_CELLS] = (c.h + 1) * c.swp - q0;
        }
        ++g->nsteps;
        return true;
    };
    for (int l = 0; l < n; ++l)
        for (int r0 = 0; r0 < map[l].oc; r0 += map[l].chunk_f)
            if (!append(l, false, r0)) return false;
    g->turn = g->nsteps;
    for (int l = n - 1; l >= 0; --l)
        for (int r0 = 0; r0 < map[l].ic; r0 += map[l].chunk_b)
            if (!append(l, true, r0)) return false;
    const Map &top = map[n - 1];
    g->t_del = top.del; g->t_pl = top.pl; g->t_planes = up(top.oc, 4); g->t_h = top.h; g->t_swp = top.swp;
    g->t_clear = dirty(n - 1); g->t_relu = top.relu; g->t_pool = top.pool; g->t_win = top.win;
    g->t_per = top.act_pl; g->t_w = top.act_swp;
    g->t_divper = reciprocal(g->t_per); g->t_divw = reciprocal(g->t_w);
    return true;
}

// [client][words of the cluster's barrier], [client][places], error flag; plan; [client][scratch]
size_t cnn_words(int n_clients) { return (size_t)n_clients * (whole_lines(kClusterMax) + kPlaces); }
size_t cnn_plan_at(int n_clients) { return (cnn_words(n_clients) * 8 + 8 + 255) / 256 * 256; }
size_t cnn_head_bytes(int n_clients) { return cnn_plan_at(n_clients) + (sizeof(CnnPlan) + 255) / 256 * 256; }

}  // namespace

// A turn is what one launch does with one sample per workgroup.  Time here / in the layer engine, per
// recursion, for clients x mini-batch (8 x 8 maps and 16 channels | 8 x 8, 32 | 12 x 12, 24 | 16 x 16, 16 | seven
// layers of 16 on 8 x 8 | 32 x 32, 4; hidden layers of 64 and 30 units):
//   one turn    1 x 1   0.47 0.70 0.65 0.70 0.64 0.82    4 x 5   0.45 0.61 0.56 0.64 0.58 0.71    16 x 16  0.38 0.51 0.43 0.46 0.49 0.41
//   two turns   1 x 33  0.80 1.25 1.06 1.13 1.03 1.04    4 x 64  0.70 0.97 0.82 0.83 0.89 0.68     5 x 64  0.50 0.76 0.68 0.66 0.64 0.62
//               6 x 64  0.49 0.75 0.65 0.63 0.64 0.58   12 x 32  0.52 0.77 0.67 0.66 0.67 0.66   24 x 16  0.55 0.76 0.65 0.68 0.70 0.63
// So one turn pays, two pay for small convolutions or with many samples, beyond that the layer engine keeps what it had.
//
// That is without the dense layers' part: every workgroup reads the first one's weights twice per sample, 0.155 us
// per thousand, where the layer engine reads them once for many samples.  Features x units that it has time for
// come with the convolutions (launches of the layer engine) and, a little, with all clients' parameters.  One
// convolution on 8 x 8 maps, 1 x 1 and 8 x 32: 65 K weights 0.63 - 0.92 and 0.54 - 0.87, 131 K 0.83 - 0.92 and 0.72 - 0.75,
// 262 K 1.13 - 1.31 and 0.95 - 1.03, 4 M 7.4 and 2.6.  And a client's only workgroup makes the whole update, 0.85 us per thousand
// parameters: two launches of 300 clients, mini-batch 1: 8 x 8, 16 channels (25 K) 0.75, 12 x 12, 24 (65 K) 1.15, 8 x 8, 32 (72 K) 1.31.
// Of 3,243 random networks (1 - 7 convolutions of 3 - 64 channels, maps of 4 x 4 to 32 x 32, 8 - 1,024 units, 1 - 500
// clients, mini-batch 1 - 64) of up to two turns the dense limits turn 128 away, of which half had lost (up to 4.1);
// of those that are taken, ten take longer than the layer engine by more than 2 %, 1.17 at most (median 0.41, with two turns 0.56).
bool cnn_round_pays(const LayerGeom *lay, int L, int B, int n_clients) {
    CnnPlan g;
    if (!cnn_plan(lay, L, B, n_clients, &g)) return false;
    const int per_launch = 8 * (kClusterMax / g.G), launches = (n_clients + per_launch - 1) / per_launch;
    const int turns = launches * ((B + g.A - 1) / g.A);
    int64_t macs = 0;
    for (int l = 0; l < L; ++l)
        if (lay[l].type == 0) macs += lay[l].out_size * lay[l].ic * 9;
    const int64_t params = g.b2 + g.C, dense = (int64_t)turns * g.F0 * g.H, clients = n_clients;
    if (turns == 1) return dense <= 200000 * g.nconv + clients * params / 200;
    if (g.G == 1 && params > 16000 * g.nconv) return false;
    return turns == 2 && dense <= 130000 * g.nconv + clients * params / 200 && (macs <= 1000000 || clients * B >= 384);
}

size_t cnn_round_scratch_bytes(const LayerGeom *lay, int L, int n_clients, int B) {
    CnnPlan g;
    return cnn_plan(lay, L, B, n_clients, &g) ? cnn_head_bytes(n_clients) + (size_t)n_clients * g.client_floats * 4 : 0;
}

hipError_t cnn_prepare(hipStream_t s, const LayerGeom *lay, int L, int B, void *scratch, int n_clients) {
    CnnPlan g;
    if (!cnn_plan(lay, L, B, n_clients, &g)) return hipErrorInvalidValue;
    char *base = static_cast<char *>(scratch);
    k_put_plan<<<1, 256, 0, s>>>(g, reinterpret_cast<CnnPlan *>(base + cnn_plan_at(n_clients)),
                                 reinterpret_cast<int *>(base + cnn_words(n_clients) * 8));
    return hipGetLastError();
}

const int *cnn_error_flag_ptr(void *scratch, int n_clients) {
    return reinterpret_cast<const int *>(static_cast<u64 *>(scratch) + cnn_words(n_clients));
}

hipError_t cnn_cluster_need(const LayerGeom *lay, int L, int B, int n_clients, int *cus, int *least, int *most) {
    CnnPlan g;
    if (!cnn_plan(lay, L, B, n_clients, &g)) return hipErrorInvalidValue;
    int dev = 0, all = 0, xcds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&all, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = device_xcds(&xcds);
    if (e != hipSuccess) return e;
    *cus = xcds == 8 ? all / xcds : 0;
    *least = g.A;
    *most = g.G;
    return hipSuccess;
}

hipError_t launch_cnn_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact, int max_m, const float *Wg,
                            const LayerGeom *lay, int L, int B, void *scratch, int n_clients, int size, int first, uint32_t *epoch) {
    if (nact <= 0) return hipSuccess;
    CnnPlan g;
    if (!cnn_plan(lay, L, B, n_clients, &g) || size < g.A || size > g.G || first > 7) return hipErrorInvalidValue;
    const size_t lds = (size_t)g.lds_floats * 4;
    int dev = 0, cus = 0, per_cu = 0, sized = 0, xcds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    static PerDevice lds_allowed;
    e = lds_allowed.get(dev, &sized, [](int *done) {
        *done = 1;
        return hipFuncSetAttribute(reinterpret_cast<const void *>(k_cnn_round), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_cnn_round, kCnThreads, lds);
    if (e == hipSuccess) e = device_xcds(&xcds);
    if (e != hipSuccess) return e;
    const int per_launch = resident_clusters(cus * per_cu, xcds, size);
    if (per_launch < 1) return hipErrorLaunchOutOfResources;
    u64 *words = static_cast<u64 *>(scratch), *all_places = words + (size_t)n_clients * whole_lines(kClusterMax);
    u64 *places = g_posts_to_memory ? nullptr : all_places;
    int *errflag = reinterpret_cast<int *>(words + cnn_words(n_clients));
    const CnnPlan *plan = reinterpret_cast<const CnnPlan *>(static_cast<char *>(scratch) + cnn_plan_at(n_clients));
    float *data = reinterpret_cast<float *>(static_cast<char *>(scratch) + cnn_head_bytes(n_clients));
    // Two tags per recursion and two ahead: never 0 (the cleared state), never one of an earlier launch.  A
    // captured launch carries its tags into every replay: there the words are cleared ahead of it.
    const uint32_t need = 2u * (uint32_t)max_m + 4u;
    const bool spent = *epoch == 0 || *epoch > 0xFFFFFFFFu - need;
    if (spent || stream_is_capturing(s)) {
        const size_t n = cnn_words(n_clients);
        k_zero_words_cnn<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(words, n);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (spent) *epoch = 1;
    const uint32_t tag0 = *epoch;
    *epoch += need;
    for (int a0 = 0; a0 < nact; a0 += per_launch) {
        const int here = nact - a0 < per_launch ? nact - a0 : per_launch;
        const unsigned grid = (unsigned)(8 * ((here + 7) / 8) * size);
        if (prof && prof->on[F_CNN_ROUND]) prof->before(F_CNN_ROUND, s);
        k_cnn_round<<<grid, kCnThreads, lds, s>>>(dp + a0, here, size, first, Wg, plan, data, words, places, all_places, g_xcd_skew, tag0, errflag);
        if (prof && prof->on[F_CNN_ROUND]) prof->after(F_CNN_ROUND, s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace aet
