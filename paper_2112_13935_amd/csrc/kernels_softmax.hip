// Fused local round for softmax regression (one dense layer D -> C, per-sample SGD, B = 1).
//
// One workgroup (8 waves; fewer where a row has no columns for them) per client runs the client's whole round (Algorithm 2,
// MainComputeNode: s_i recursions).  The replica w_c (C x D weights + C biases) and the
// gradient sum U stay in registers for the round: thread t owns columns t, t+512, ... of
// every class row.  Per recursion the only memory traffic is the sampled row (fetched three
// recursions ahead: the index hash is a counter, so the rows are known).
//
//   z_o = b_o + sum_k W[o][k] x[k]   per-thread partial sums, lane swaps and DPP inside a wave,
//                                    one LDS hop across the 8 waves (fixed order)
//   p = softmax(z), dz = p - onehot  lane o of every 16-lane row handles class o (DPP row
//                                    reductions); the matrix cores take dz from there
//   W[o][k] -= eta dz_o x[k];  U[o][k] += dz_o x[k]      in registers, as 4 x 4 outer products
//                                    on the matrix cores (g never stored)
//
// At the end of the round w_c and U are written to HBM once.
#include <type_traits>

#include "aet_device.h"
#include "aet_internal.h"

namespace aet {

constexpr int kSmWaves = 8;    // at most
constexpr int kSmThreads = 64 * kSmWaves;
constexpr int kSmDepth = 4;    // rows in registers: at work, just done with, and two on the way
constexpr int kSmBlock = 48;   // recursions per block of row numbers; a multiple of kSmDepth

// Sums of N values over the 64 lanes of a wave, several values per instruction.  The lane
// swaps of gfx950 exchange half-waves (rows of 16 lanes) between two registers, so that one
// addition folds two (then four) different values at once:
//   swap32(a, b) -> [a.lo, b.lo], [a.hi, b.hi]; their sum holds a folded to 32 lanes in the
//                   lower half and b in the upper half;
//   swap16(p, q) -> rows [p0, q0, p2, q2], [p1, q1, p3, q3]; their sum holds four values, one
//                   per row of 16 lanes;
// four shuffle-and-add stages inside the rows finish.  Register k of the result holds, in all
// 16 lanes of row r, the total of value 4k + rowmap(r), rowmap = {0, 2, 1, 3}.
template <int N>
__device__ __forceinline__ void wave_sum_rows(const float (&v)[N], float (&out)[(N + 3) / 4]) {
    static_assert(N % 2 == 0, "values come in pairs");
    constexpr int NP = N / 2, NQ = (N + 3) / 4;
    float p[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, v[2 * k]),
                                                        __builtin_bit_cast(int, v[2 * k + 1]), false, false);
        p[k] = __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const float a = p[2 * k], b = 2 * k + 1 < NP ? p[2 * k + 1] : 0.f;
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
        out[k] = __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) out[k] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, out[k]), 0xB1, 0xF, 0xF, true));
#pragma unroll
    for (int k = 0; k < NQ; ++k) out[k] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, out[k]), 0x4E, 0xF, 0xF, true));
#pragma unroll
    for (int k = 0; k < NQ; ++k) out[k] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, out[k]), 0x141, 0xF, 0xF, true));
#pragma unroll
    for (int k = 0; k < NQ; ++k) out[k] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, out[k]), 0x140, 0xF, 0xF, true));
}

// sum / max over each row of 16 lanes (every lane of the row gets the result)
__device__ __forceinline__ float row_sum_dpp(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));
    return v;
}
// (One instruction a step.  From fmaxf of a lane move the compiler makes three, the move, a maximum of the moved value with itself
// for the sake of signalling NaNs, and the maximum.  Two wait states between a write and a lane move that reads it.)
__device__ __forceinline__ float row_max_dpp(float v) {
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "+v"(v));
    return v;
}

// __logf of a sum of exponentials, bit for bit as the AMD compiler expands it: the unit's base-2 logarithm times ln 2 in two parts,
// the products' rounding caught by fused multiply-adds.  Its scaling for arguments below 2^-126 is left out, five instructions of the chain:
// the largest exponential is 1, so the sum is 1 .. 10, or NaN where the largest logit is not finite.  Us a job: 4 clients x 784 columns 1,435 -> 1,424; 5 x 60 943 -> 909;
// 346 x 114 1,487 -> 1,428; 1,024 x 3,072, 10 rounds 1,852 -> 1,833.
__device__ __forceinline__ float log_of_sum(float v) {
    const float y = __builtin_amdgcn_logf(v), ln2 = __uint_as_float(0x3f317217u), rest = __uint_as_float(0x3377d1cfu);
    const float r = fmaf(y, ln2, fmaf(y, rest, fmaf(y, ln2, -(y * ln2))));
    return fabsf(y) < INFINITY ? r : y;
}

// ---- the round kernel: rank-1 updates on the matrix cores ----------------------------------
// Two thirds of a recursion's multiply-adds are the rank-1 updates  W -= eta dz x^T  and
// U += dz x^T.  v_mfma_f32_4x4x1_16b_f32 computes 16 independent 4 x 4 outer products
// D[b] += A[b] B[b]^T: lane l supplies A[b = l/4][i = l%4] and B[b][n = l%4] and receives, in
// its four result registers, the products of the four A entries of its block with ITS OWN B
// entry.  With B = the lane's own column of the sampled row and A = four entries of
// (-eta) dz (the same four in every block: the instruction's block broadcast takes them from
// four neighbouring lanes, so dz needs no lane exchange), one instruction updates four class rows of the
// lane's own column: the replica keeps the ownership it has in the vector-ALU form (thread t
// owns columns t, t+512, ... of every class row), so the logits still need no other lane's
// data, and three instructions per 64 columns cover classes 0..11 (rows 10 and 11 stay
// zero).  The vector ALU is left with the dot products, the reductions and the softmax.
//
// What bounds it: with many clients instruction issue (two waves per SIMD, some 140 vector and 36
// matrix instructions each per recursion at D = 3072), with few clients the chain dots - wave
// reduction - LDS hop - softmax - update, the same for every width.  So what need not be on that
// chain is off it: U of a recursion is added while the next one's partial logits travel through
// LDS; row numbers are hashed 48 recursions at a time; rows are asked for three recursions
// ahead, and no load stands behind a branch or goes through the scalar cache, so that nothing
// waits for more than the row it needs.  Measured, 1,024 clients x 3,072 columns, 40 rounds:
// 23.8 -> 19.0 ms, with fewer instructions in the softmax 17.7 (2.6, 3.3 and 3.5 TB/s of rows); 4 clients x 784 columns,
// 20 rounds: 1.73 -> 1.43 -> 1.30 ms.  Four waves with twice the columns each, two rows ahead: slower; five ahead: no faster.
//
// The arithmetic of dz = exp(z - lse) - onehot, its sums' order included, is fixed (the GPU tests
// hold digests of it).  Its entries add up to an error that is not centred; with features of one
// sign every recursion moves all ten rows by a little of x, and the models of many clients
// keep that: 600 clients x 40 columns, 20 rounds, 4e-5 of the norm against 64 bits.  ex * (1 / sum)
// is as good a softmax and came to 2.4e-6 there, -(sum - ex) / sum for the label's entry to
// 2.4e-7, but each moves every model by those 4e-5.
// dword 3 of a raw buffer descriptor for 32-bit untyped accesses on this part
constexpr int kBufferFlags = 0x00020000;

typedef float f4v __attribute__((ext_vector_type(4)));

// NW waves of NC columns per thread; EXACT: D == 64 * NW * NC, no column guards.
template <int NC, bool EXACT, int NW>
__global__ void __launch_bounds__(64 * NW, NC == 3 ? 4 : 1)
k_softmax_round(const RoundParams *__restrict__ rp, const float *Wg, int D) {
    constexpr int C = 10, Q = 3;   // classes, groups of four class rows
    constexpr int T = 64 * NW, QW = (NW + 3) / 4, DEPTH = kSmDepth;
    const RoundParams p = rp[blockIdx.x];
    const gci_ptr yg = as_global(p.y);
    const gf_ptr Wc = as_global(p.W), Uc = as_global(p.U);
    const int tid = threadIdx.x, lane = tid & 63, cls = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // partial logits [parity][four waves][class]: a lane reads the eight waves' sums of its class
    // as two 16-byte pieces, the lanes of a row from neighbouring places
    __shared__ __attribute__((aligned(16))) float zpart[2][QW][16][4];

    const gcf_ptr W0 = as_global(Wg ? Wg : p.W);
    f4v W[NC][Q], U[NC][Q];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int k = tid + T * j;
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = 4 * q + r;
                W[j][q][r] = (o < C && (EXACT || k < D)) ? W0[(int64_t)o * D + k] : 0.f;
                U[j][q][r] = 0.f;
            }
    }
    // lane o of every row of 16 looks after class o; the lanes beyond have a bias and so a logit of minus infinity: their
    // exponential and their dz are zero by themselves
    const bool real = cls < C;
    float bias = real ? W0[(int64_t)C * D + cls] : -INFINITY, Ub = 0.f, dz = 0.f;
    float loss_acc = 0.f;

    // Row numbers and labels come a block of kSmBlock recursions at a time: lane l hashes
    // recursion l of the block (the lanes beyond it the rows that are fetched ahead), and each
    // recursion picks its own with a lane read: the hash of one recursion alone is a chain of
    // some forty scalar instructions.  Beyond the round's end the last row stands.
    uint32_t rowv = 0, rown = 0;
    int labv = 0, labn = 0;
    auto next_block = [&](int u) {
        rown = sample_row(p.key, (uint64_t)(p.q0 + min(u + lane, p.m - 1)), p.n_samples);
        labn = yg[rown];
    };
    // The loads of a row have no branches, so that the compiler can count them and wait for the
    // one row it needs: a range-checked buffer per row (columns beyond D read zero).
    auto load_row = [&](int i, float (&x)[NC]) {
        const uint32_t row = __builtin_amdgcn_readlane(rowv, i);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(p.X) + (int64_t)row * D, 0, 4 * D, kBufferFlags);
#pragma unroll
        for (int j = 0; j < NC; ++j)
            x[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, 4 * (tid + T * j), 0, 0));
    };
    // M <- M + a x^T: cbsz = 4, abid = q broadcasts block q of A, that is lanes 4q .. 4q + 3 of the
    // first row with classes 4q .. 4q + 3 (10 .. 15: zeros), to all sixteen blocks
    auto rank1 = [&](f4v (&M)[NC][Q], float a, const float (&x)[NC]) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            M[j][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, x[j], M[j][0], 4, 0, 0);
            M[j][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, x[j], M[j][1], 4, 1, 0);
            M[j][2] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, x[j], M[j][2], 4, 2, 0);
        }
    };

    // x: this recursion's row; xp: the row of the recursion before, whose dz is still in dz;
    // that row's registers then take the row of recursion u + DEPTH - 1.  The loads stand
    // outside of the branches on `live` (false for the up to DEPTH - 1 steps that fill the last
    // group): between two of them the same number of loads is issued on every way.
    auto recursion = [&](int u, int i, const float (&x)[NC], float (&xp)[NC], const auto all_live) __attribute__((always_inline)) {
        const bool live = all_live || u < p.m;
        const int lab = __builtin_amdgcn_readlane(labv, i);
        f4v za[QW];
        if (live) {
            float(*zp)[16][4] = zpart[u & 1];
            float s[C];
#pragma unroll
            for (int o = 0; o < C; ++o) {
                s[o] = 0.f;
#pragma unroll
                for (int j = 0; j < NC; ++j) s[o] += W[j][o >> 2][o & 3] * x[j];
            }
            float t[(C + 3) / 4];
            wave_sum_rows<C>(s, t);
#pragma unroll
            for (int k = 0; k < (C + 3) / 4; ++k) asm("" : "+v"(t[k]));   // the last step of the sums ahead of the branch, one instruction each
            if ((lane & 15) == 0) {
                const int row = lane >> 4, o0 = ((row & 1) << 1) | (row >> 1);
#pragma unroll
                for (int k = 0; k < (C + 3) / 4; ++k) zp[wave >> 2][4 * k + o0][wave & 3] = t[k];   // (places 10 and 11: never read)
            }
            __syncthreads();
#pragma unroll
            for (int h = 0; h < QW; ++h) za[h] = *reinterpret_cast<const f4v *>(zp[h][real ? cls : 0]);
        }
        // while those travel: the sum U of the recursion before (not on the way to the next
        // logits), and the row that is needed DEPTH - 1 recursions from now
        __builtin_amdgcn_sched_barrier(0);
        rank1(U, dz, xp);
        __builtin_amdgcn_sched_barrier(0);
        load_row(i + DEPTH - 1, xp);
        if (live) {
            float z = bias;   // the waves' sums in wave order
#pragma unroll
            for (int w = 0; w < NW; ++w) z += za[w >> 2][w & 3];
            const float zmax = row_max_dpp(z);
            const float lse = zmax + log_of_sum(row_sum_dpp(__expf(z - zmax)));
            dz = __expf(z - lse) - (cls == lab ? 1.f : 0.f);
            __builtin_amdgcn_sched_barrier(0);
            rank1(W, -p.eta * dz, x);   // w <- w - eta g with g = dz x^T
            __builtin_amdgcn_sched_barrier(0);   // (what the next logits do not need comes after it)
            bias -= p.eta * dz;
            Ub += dz;
            if (cls == lab) loss_acc += lse - z;
        } else {
            dz = 0.f;
        }
    };

    // DEPTH rows live in registers: the one at work, the one before it and DEPTH - 2 on the way
    float x[DEPTH][NC];
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {
#pragma unroll
        for (int j = 0; j < NC; ++j) x[i][j] = 0.f;
    }
    if (p.m > 0) {
        next_block(0);
        rowv = rown;
#pragma unroll
        for (int i = 0; i < DEPTH - 1; ++i) load_row(i, x[i]);
        // everything has arrived when the loop starts: what is in flight at its head is then
        // the same on the way in and on the way round, and the compiler waits for a count
        __builtin_amdgcn_s_waitcnt(0x0F70);
        for (int u0 = 0; u0 < p.m; u0 += kSmBlock) {
            rowv = rown;
            labv = labn;
            next_block(u0 + kSmBlock);
            const int n = min(kSmBlock, p.m - u0);
            int i0 = 0;
            // Groups without filling steps once more without their tests, where both fit the registers (the forms of
            // three and six columns spilled).  Us a job: 4 clients x 784 columns 1,334 -> 1,303; 5 x 60 895 -> 843.
            if constexpr (NC != 3 && NC != 6) {
                for (; i0 + DEPTH <= n; i0 += DEPTH)
#pragma unroll
                    for (int i = 0; i < DEPTH; ++i) recursion(u0 + i0 + i, i0 + i, x[i], x[(i + DEPTH - 1) % DEPTH], std::true_type());
            }
            for (; i0 < n; i0 += DEPTH) {
#pragma unroll
                for (int i = 0; i < DEPTH; ++i) recursion(u0 + i0 + i, i0 + i, x[i], x[(i + DEPTH - 1) % DEPTH], std::false_type());
            }
        }
        rank1(U, dz, x[DEPTH - 1]);   // the last recursion's, unless a filling step has done it
    }

#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int k = tid + T * j;
        if (EXACT || k < D) {
#pragma unroll
            for (int o = 0; o < C; ++o) {
                Wc[(int64_t)o * D + k] = W[j][o >> 2][o & 3];
                Uc[(int64_t)o * D + k] = U[j][o >> 2][o & 3];
            }
        }
    }
    if (tid < C) {
        Wc[(int64_t)C * D + tid] = bias;
        Uc[(int64_t)C * D + tid] = Ub;
    }
    if (wave == 0) {
        const float l = row_sum_dpp(loss_acc);
        if (lane == 0) *as_global(p.loss) = l;
    }
}

bool softmax_round_supported(int D, int C, int B) {
    return B == 1 && C == 10 && D >= 1 && D <= kSmThreads * 6;
}

hipError_t launch_softmax_round(hipStream_t s, Profiler *prof, const RoundParams *dp, int nact,
                                const float *Wg, int D, int C) {
    if (nact <= 0) return hipSuccess;
    (void)C;
    const bool timed = prof && prof->on[F_SOFTMAX_ROUND];
    if (timed) prof->before(F_SOFTMAX_ROUND, s);
    // As many waves as have columns, and as many columns a thread: a wave or a column without data adds zeros to the logits,
    // in its place (so every form gives the widest one's bits), but takes part in every barrier, softmax and update.
    // us a job of 20 rounds, eight waves / as many as have columns: 903 clients x 19 (12 rounds) 1,980 / 959; 5 x 60 1,281 / 945;
    // 20 x 84 (11 rounds) 439 / 360; 346 x 114 2,219 / 1,492; 300 x 200 2,197 / 1,518.  Six columns a thread / as many as there
    // are, 18 rounds: 5 x 1,500 956 / 740; 300 x 1,500 2,003 / 1,320; 1,000 x 1,500 4,063 / 2,635; 300 x 2,000 2,042 / 1,785;
    // 300 x 2,400 2,075 / 1,960.  (Three columns fit 128 registers, so that a compute unit holds two clients.)
    if (D <= 64)
        k_softmax_round<1, false, 1><<<nact, 64, 0, s>>>(dp, Wg, D);
    else if (D <= 128)
        k_softmax_round<1, false, 2><<<nact, 128, 0, s>>>(dp, Wg, D);
    else if (D <= 256)
        k_softmax_round<1, false, 4><<<nact, 256, 0, s>>>(dp, Wg, D);
    else if (D <= kSmThreads)
        k_softmax_round<1, false, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    else if (D <= 2 * kSmThreads)
        k_softmax_round<2, false, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    else if (D <= 3 * kSmThreads)
        k_softmax_round<3, false, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    else if (D <= 4 * kSmThreads)
        k_softmax_round<4, false, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    else if (D <= 5 * kSmThreads)
        k_softmax_round<5, false, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    else if (D == 6 * kSmThreads)
        k_softmax_round<6, true, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    else
        k_softmax_round<6, false, kSmWaves><<<nact, kSmThreads, 0, s>>>(dp, Wg, D);
    if (timed) prof->after(F_SOFTMAX_ROUND, s);
    return hipGetLastError();
}

}  // namespace aet
