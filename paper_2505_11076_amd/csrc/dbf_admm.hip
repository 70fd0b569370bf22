// One ADMM update of the factorisation (paper, section 3.2, the three-line update after the SVID
// definition), with the two matrices that stay constant while B and W are fixed formed by the caller:
//
//     Minv = (B^T B + rho I)^-1  (q x q),   C = B^T W  (q x r)
//
//     R  = C + rho (a . S . m^T - U)           dbf_admm_operands_kernel (A = a . S . m^T never exists densely: S is read
//                                                                       from the packed tile layout; R only as fp16 planes)
//     Z  = Minv^T R + U   (= W_hat + U)        dbf_split_gemm_kernel   fp16 matrix cores, operands split in two
//                                                                       (dbf_split_gemm.h), U added in the epilogue
//     (S', a', m') = SVID(Z)                   dbf_svid (dbf_svid.hip)
//     U' = Z - a' . S' . m'^T  (= U + W_hat - A')   dbf_svid_dual (dbf_svid.hip)
//
// The contraction is q x q x r in fp32 accuracy (34 GFLOP at q = 2048, r = 4096) and dominates; the elementwise
// kernels and the projection are bandwidth bound.  Measured at that size: the contraction 331 us on the fp32 matrix cores, 219 on the bf16
// ones with operands in three parts, 106-110 on the fp16 ones with operands in two, whose planes, with the making of R, take 22 us in one launch; the update
// with two rounds of SVID 388, 287, now 178-180 us; error against 64 bits 8.1e-6, 5.1e-6, 1.6e-6 (fewer roundings: 16 products enter the accumulator at
// once, and half as many of them).
// The paper gives no kernel design for this step.
#include "dbf_kernels.h"
#include "dbf_split_gemm.h"

#include <algorithm>
#include <cmath>
#include <utility>

namespace {

// The operands of the contraction in one launch: the planes of Minv (blockIdx.y below q_blocks), and R = C + rho (a_k m_j s_kj - U) (q x r; k = its
// row is the summation index of the contraction), written straight into fp16 planes: R exists nowhere in fp32.  A lane's eight rows of R are
// one bit of eight bytes 16 apart of one sign tile.
__global__ __launch_bounds__(256) void dbf_admm_operands_kernel(const float* __restrict__ Minv, uint8_t* __restrict__ Minv_planes, int q_blocks,
                                                               const float* __restrict__ C, const float* __restrict__ U, float rho,
                                                               const float* __restrict__ a, const float* __restrict__ m,
                                                               const uint8_t* __restrict__ bits, int q, int r, int n_ct,
                                                               uint8_t* __restrict__ planes) {
    if ((int)blockIdx.y < q_blocks) {
        __shared__ float part[4][32];
        sg_split_dense<true>(Minv, q, q, q, nullptr, Minv_planes, blockIdx.y, blockIdx.x, threadIdx.x, part);
        return;
    }
    const SgSite s = sg_site(q, 2, blockIdx.y - q_blocks);
    const int j = min(s.i, r - 1);
    const float mj = m[j];
    float x[2][8], u[2][8], ak[2][8];
    unsigned sign[2][8];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const uint8_t* sb = bits + ((size_t)blockIdx.x * n_ct + (j >> 6)) * DBF_TILE_BYTES + 256 * ((j >> 4) & 3) + 16 * (s.k0[n] & 15) + (j & 15);   // (a chunk is a row tile)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(s.k0[n] + e, q - 1);
            const size_t at = (size_t)k * r + j;
            x[n][e] = C[at];
            u[n][e] = U[at];
            ak[n][e] = a[k];
            sign[n][e] = sb[16 * e];
        }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int bit = (s.k0[n] & 127) >> 4;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            asm("" : "+v"(x[n][e]), "+v"(u[n][e]), "+v"(ak[n][e]), "+v"(sign[n][e]));   // (as in sg_split_dense: the loads of all sixteen rows in flight)
            const float am = ak[n][e] * mj;
            const float v = x[n][e] + rho * (((sign[n][e] >> bit) & 1 ? am : -am) - u[n][e]);
            x[n][e] = (s.k0[n] + e < q && s.i < r) ? v : 0.f;
        }
    }
    sg_split_chunk(planes, q, r, s, x);
}

// ---------------------------------------------------------------------------------------------
// Inverse of the symmetric positive definite G = B^T B + rho I by a blocked Cholesky factorisation G = R^T R (R upper
// triangular), blocks of 128: forward elimination of the augmented matrix [G | I] gives [R | Y] with Y = R^-T, and
// G^-1 = Y^T Y is one more contraction.  Block row j is one launch (dbf_chol_row_kernel), with T = R_jj^-T from the launch before:
//   [R | Y][j, :] = T [G | Y][j, :]     [G | Y][i, :] -= R[j, i]^T [R | Y][j, :] for the block rows i > j
// A workgroup has block (i, c) of the second and makes the two blocks of row j that it needs, R[j, i] and [R | Y][j, c], by itself: three
// products for one, but no launch before it.  The workgroup of diagonal block j + 1 goes on to factor it and to invert its factor: that
// chain of 128 pivots, the longest of the whole, runs beside the other blocks' products.
// G and Y share one q x q matrix: block (i, c) is G's for c >= i and Y's for c < i (it starts at zero at j = c); row j is read
// only.  A finished row of Y is written as the fp16 planes that the last contraction reads; R is kept nowhere.
// What bounds it: the chain.  Per block row a launch of 22 us at q = 2048: 2 to the loads' arrival, 6 to the diagonal block, four times 2.5 for 32 pivots and
// 0.4 for the next row's share of them, 0.7 for T.  (As two launches, a panel of 6 us and an update of 24 whose chain held an inverse's product behind each 32
// pivots, the constants took 744 us with p = r = 4096; so 627.)  Blocks that fill the chip more than once make row j too often: for more than 256 blocks
// dbf_chol_panel_kernel makes it first (q = 3328 870 us without, 819 so; 4096 with p = r = 4096 1681, 1484).
// ---------------------------------------------------------------------------------------------
constexpr int NB = 128;        // block size: the contraction's tile
constexpr int CH_LD = NB + 4;  // LDS row length of a diagonal block: rows start on 16 bytes
constexpr int CH_THREADS = 512;
constexpr int CH_UNITS = 256;   // compute units
constexpr int CH_MADE = 256;    // more blocks than this: row j first, in a launch of its own
static_assert(CH_MADE >= CH_UNITS, "a launch with parts of C beside it (chol_free) makes row j itself");
constexpr int CH_PLANES = 64 * SG_FRAG;   // the two pieces of a 128 x 128 operand: [k / 16][piece][line / 32]
// T's planes leave fragments of k beyond a line empty: the first of these has its lines' scales, and behind them what the rows that T's columns meet are multiplied by.
constexpr int CH_T_UP = (7 * 2 * 4) * SG_FRAG;

struct CholPivot {
    float v0, v1, t;   // lanes 0-15 of a pivot row in every 16 lanes, lanes 16-31 in every 16; the row over its pivot
};
// x -= (entry R of the pivot row) * t
template <int R>
__device__ __forceinline__ void chol_sub(float (&x)[32], const CholPivot& p) {
    asm("v_fmac_f32_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(x[R]) : "v"(R < 16 ? p.v0 : p.v1), "v"(p.t), "n"(R & 15));
}
template <int FROM, int... R>
__device__ __forceinline__ void chol_subs(float (&x)[32], const CholPivot& p, std::integer_sequence<int, R...>) {
    (chol_sub<FROM + R>(x, p), ...);
}
// Pivot C, its value to lane C of piv: t = row C / pivot (reciprocal, product and one correction: met to its last bit or nearly so) and the row's entries for
// the rows below.  Row C is up to date; `before`, the pivot before it, is still owed to the rows below, and the first six of them get it here, where the chain
// from row C to row C + 1 would leave the wavefront waiting (eight cycles from a result to its use, four to issue an instruction).  (One block, so that what the
// instructions want between a write and a use -- one other before a lane read of a fresh register, two between the lane read and a use of its scalar
// register, two before a lane swap of a fresh register and before a lane broadcast of one, one behind the reciprocal -- is the work itself as
// far as it goes.  The build checks the assembly for them: _wait_states_report in build.py.)
#define CHOL_OWED(n) "v_fmac_f32_dpp %" #n ", -%" CHOL_FROM_##n ", %[bt] row_newbcast:%[n" #n "] row_mask:0xf bank_mask:0xf\n\t"
#define CHOL_FROM_0 "[b0]"
#define CHOL_FROM_1 "[b1]"
#define CHOL_FROM_2 "[b2]"
#define CHOL_FROM_3 "[b3]"
#define CHOL_FROM_4 "[b4]"
#define CHOL_FROM_5 "[b5]"
#define CHOL_PIVOT(o0, o1, o2, o3, o4, o5)                                                                                                        \
    asm(o0 o1 "v_mov_b32 %[v0], %[xc]\n\t"                                                                                                        \
        "v_readlane_b32 %[p], %[xc], %[c]\n\t"                                                                                                    \
        "v_mov_b32 %[v1], %[xc]\n\t" o2 "v_rcp_f32 %[r], %[p]\n\t"                                                                                \
        "v_permlane32_swap_b32 %[v0], %[v1]\n\t" o3 "v_mul_f32 %[t0], %[xc], %[r]\n\t"                                                            \
        "v_mov_b32 %[v1], %[v0]\n\t" o4 "v_fma_f32 %[t], -%[t0], %[p], %[xc]\n\t" o5 "v_permlane16_swap_b32 %[v0], %[v1]\n\t"                     \
        "v_fma_f32 %[t], %[t], %[r], %[t0]\n\t"                                                                                                   \
        "v_writelane_b32 %[piv], %[p], %[c]"                                                                                                      \
        : "+v"(x[X(0)]), "+v"(x[X(1)]), "+v"(x[X(2)]), "+v"(x[X(3)]), "+v"(x[X(4)]), "+v"(x[X(5)]), [v0] "=&v"(now.v0), [v1] "=&v"(now.v1),       \
          [t] "=&v"(now.t), [t0] "=&v"(t0), [r] "=&v"(r), [p] "=&s"(p), [piv] "+v"(piv)                                                           \
        : [xc] "v"(x[C]), [bt] "v"(before.t), [b0] "v"(from(0)), [b1] "v"(from(1)), [b2] "v"(from(2)), [b3] "v"(from(3)), [b4] "v"(from(4)),      \
          [b5] "v"(from(5)), [c] "n"(C), [n0] "n"(X(0) & 15), [n1] "n"(X(1) & 15), [n2] "n"(X(2) & 15), [n3] "n"(X(3) & 15), [n4] "n"(X(4) & 15), \
          [n5] "n"(X(5) & 15))
template <int C>
__device__ __forceinline__ void chol_pivot(float (&x)[32], float& piv, CholPivot& before) {
    CholPivot now;
    float r, t0;
    int p;
    constexpr int LEFT = C > 0 ? 31 - C : 0;   // the rows that `before` is owed to
    // (rows that do not exist: operands of a block that does not use them)
    constexpr auto X = [](int n) { return n < LEFT ? C + 1 + n : (C + 26 + n) % 32; };
    auto from = [&](int n) { return X(n) < 16 ? before.v0 : before.v1; };
    if constexpr (C == 0) before.v0 = before.v1 = before.t = 0.f;
    if constexpr (LEFT >= 6) CHOL_PIVOT(CHOL_OWED(0), CHOL_OWED(1), CHOL_OWED(2), CHOL_OWED(3), CHOL_OWED(4), CHOL_OWED(5));
    else if constexpr (LEFT == 5) CHOL_PIVOT(CHOL_OWED(0), "", CHOL_OWED(1), CHOL_OWED(2), CHOL_OWED(3), CHOL_OWED(4));
    else if constexpr (LEFT == 4) CHOL_PIVOT(CHOL_OWED(0), "", CHOL_OWED(1), CHOL_OWED(2), "", CHOL_OWED(3));
    else if constexpr (LEFT == 3) CHOL_PIVOT("", "", CHOL_OWED(0), CHOL_OWED(1), "", CHOL_OWED(2));
    else if constexpr (LEFT == 2) CHOL_PIVOT("", "", CHOL_OWED(0), "", "", CHOL_OWED(1));
    else if constexpr (LEFT == 1) CHOL_PIVOT("", "", CHOL_OWED(0), "", "", "s_nop 0\n\t");
    else CHOL_PIVOT("", "", "s_nop 0\n\t", "", "", "s_nop 0\n\t");
    chol_subs<C + 7>(x, before, std::make_integer_sequence<int, (LEFT > 6 ? LEFT - 6 : 0)>());
    if constexpr (C < 31) chol_sub<C + 1>(x, now);
    before = now;
}
template <int... C>
__device__ __forceinline__ void chol_pivots(float (&x)[32], float& piv, std::integer_sequence<int, C...>) {
    CholPivot before;
    (chol_pivot<C>(x, piv, before), ...);
}
// x *= lane N of each 16 of v.  (The waits of a DPP operand are the caller's for the first.)
template <int N>
__device__ __forceinline__ void chol_mul(float& x, float v) {
    asm volatile("v_mul_f32_dpp %0, %1, %0 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(x) : "v"(v), "n"(N));
}
template <int... R>
__device__ __forceinline__ void chol_scale_rows(float (&x)[16], float v, std::integer_sequence<int, R...>) {
    asm volatile("s_nop 1" : "+v"(v));
    (chol_mul<R>(x[R], v), ...);
}

// The same for any pivots, in LDS (64 columns at X) and at leisure, with roots alone: pivots down to subnormal numbers (the instructions take none: a
// scaled copy) and up to the largest, rows of pivots that are not positive set to zero.  Returns whether there was one of the latter.  (The diagonal becomes the pivots' roots.)
__device__ __forceinline__ int chol_rows32_any(volatile float* X, int lane) {
    int bad = 0;
#pragma unroll 1
    for (int c = 0; c < 32; ++c) {
        const float piv = X[c * 64 + c];
        const bool tiny = piv < 0x1p-64f, pos = piv > 0.f;
        const float ps = tiny ? piv * 0x1p64f : piv;
        float y = __builtin_amdgcn_rsqf(ps);
        y = fmaf(0.5f * y, fmaf(-ps * y, y, 1.f), y);
        y = tiny ? y * 0x1p32f : y;
        bad |= !pos;
        __builtin_amdgcn_wave_barrier();
        const float xc = X[c * 64 + lane] * (pos ? y : 0.f);
        X[c * 64 + lane] = xc;
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int r = c + 1; r < 32; ++r) X[r * 64 + lane] = fmaf(-X[c * 64 + r], xc, X[r * 64 + lane]);
        __builtin_amdgcn_wave_barrier();
    }
    return bad;
}

// The planes of a row of 32 x 32 blocks in LDS: of each block the two pieces of eight k for a line at [pair of eight][piece][half][line] in 16 bytes; a lane's
// half h and pair f have rows 16 h + 8 f .. + 7 (any order of k does, if both operands have it).
constexpr int CH_ROW = 4 * SG_FRAG;
struct CholBlock {
    // Y: block s of its diagonal in columns 32 s .. + 31; spare: a wavefront's each
    float H[NB * CH_LD], Y[32 * CH_LD], spare[4][32 * 64], up[2][NB], even[NB];
    uint8_t rows[2][4 * CH_ROW];
    unsigned largest[NB];
};

// One wavefront: the 32 rows of a diagonal block `diag` (upper triangle read) and of the 32 more columns at `right` are eliminated, the latter to planes (`row`, `up`)
// and, with `keep`, in place.  Lane l < 32 holds column l of the block, lane 32 + l column l of the others.
// A pivot row's entries reach the other rows through lane broadcasts that are part
// of the multiplication; the rows are scaled by 1 / sqrt(pivot) at the end, all roots at once.  What bounds it: a wavefront on its own issues one
// instruction in four to five cycles, here 13 and one per row below for a pivot, eight where an instruction waits for the one before it.  (32 pivots
// 4250 cycles, and 1700 for loads, roots and planes.)
// `even`, unless NULL: the roots of the pivots, rounded down (or up) to powers of two, zero where there is none.
// Returns whether a pivot was not positive.
__device__ __forceinline__ int chol_rows32(const float* diag, float* right, bool keep, uint8_t* row, float* up, float* even, float* spare, int lane) {
    const bool upper = lane >= 32;
    const int l32 = lane & 31, h = lane >> 5;
    const float* src = (upper ? right : diag) + l32;
    float x[32], piv = 1.f, o[16];
    int bad = 0;
#pragma unroll
    for (int r = 0; r < 32; ++r) x[r] = src[r * CH_LD];
    chol_pivots(x, piv, std::make_integer_sequence<int, 32>());
    // (below 2^-126, whose reciprocal and root the instructions do not take, 2^126 and more, whose reciprocal they do not return, or not positive)
    if (__any(__builtin_bit_cast(unsigned, piv) - 0x00800000u >= 0x7e000000u)) {
#pragma unroll 1
        for (int r = 0; r < 32; ++r) spare[r * 64 + lane] = src[r * CH_LD];
        __builtin_amdgcn_wave_barrier();
        bad = chol_rows32_any(spare, lane);
        if (even && lane < 32) {   // (zero for a pivot that was not positive: T's column is)
            const unsigned root = __builtin_bit_cast(unsigned, spare[65 * lane]) & 0x7f800000u;
            even[lane] = __builtin_bit_cast(float, root < 0x7f800000u ? root : 0u);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) o[r] = spare[(16 * h + r) * 64 + 32 + l32];
    } else {
        // the columns on the right to all lanes: rows 0-15 of column l to lane l, 16-31 to lane 32 + l
#pragma unroll
        for (int r = 0; r < 16; ++r)
            o[r] = __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x[r]), __builtin_bit_cast(unsigned, x[16 + r]), false, false)[1]);
        float y = __builtin_amdgcn_rsqf(piv);
        y = fmaf(0.5f * y, fmaf(-piv * y, y, 1.f), y);
        if (even && lane < 32) even[lane] = __builtin_bit_cast(float, (254u << 23) - (__builtin_bit_cast(unsigned, y) & 0x7f800000u));
        // lanes 0-15 of y in lanes 0-15 and 16-31, lanes 16-31 in lanes 32-47 and 48-63
        const unsigned yb = __builtin_bit_cast(unsigned, y);
        const unsigned both = __builtin_amdgcn_permlane32_swap(yb, yb, false, false)[0];
        const auto halves = __builtin_amdgcn_permlane16_swap(both, both, false, false);
        chol_scale_rows(o, __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_permlane32_swap((unsigned)halves[0], (unsigned)halves[1], false, false)[0]),
                        std::make_integer_sequence<int, 16>());
    }
    if (keep) {
#pragma unroll
        for (int r = 0; r < 16; ++r) right[(16 * h + r) * CH_LD + l32] = o[r];
    }
    float mx = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, fabsf(o[r]));
    const unsigned mb = __builtin_bit_cast(unsigned, mx);
    const auto two = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
    const SgScale scale = sg_scale(fmaxf(__builtin_bit_cast(float, (unsigned)two[0]), __builtin_bit_cast(float, (unsigned)two[1])));
    if (lane < 32) up[l32] = scale.up;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        float part[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) part[e] = o[8 * f + e];
        sg_store2<false, SG_FRAG>(row + 2 * f * SG_FRAG + lane * 16, part, scale);
    }
    return bad;
}

// d -= P^T Q (or d = -P^T Q) for 16 x 32 values at d, row length CH_LD, from the planes of two blocks, lines 16 r16 .. + 15 of P's.  All four products of the pieces.
__device__ __forceinline__ void chol_update16(float* d, const uint8_t* P, const float* p_up, int r16, const uint8_t* Q, const float* q_up, bool fresh, int lane) {
    const int l16 = lane & 15, g = lane >> 4;
    auto at = [&](const uint8_t* base, int piece, int line) { return *reinterpret_cast<const v8h*>(base + (4 * (g >> 1) + 2 * piece + (g & 1)) * (SG_FRAG / 2) + line * 16); };
    v8h a[2], b[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        a[p] = at(P, p, 16 * r16 + l16);
#pragma unroll
        for (int n = 0; n < 2; ++n) b[n][p] = at(Q, p, 16 * n + l16);
    }
    const v4f pu = *reinterpret_cast<const v4f*>(p_up + 16 * r16 + 4 * g);
    float qu[2];
    v4f old[2];
    d += 4 * g * CH_LD + l16;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        qu[n] = q_up[16 * n + l16];
#pragma unroll
        for (int v = 0; v < 4; ++v) old[n][v] = d[v * CH_LD + 16 * n];
    }
    v4f hh[2], hl[2], ll[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        hh[n] = hl[n] = ll[n] = (v4f){0.f, 0.f, 0.f, 0.f};
        ll[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[1], b[n][1], ll[n], 0, 0, 0);
        hl[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[1], b[n][0], hl[n], 0, 0, 0);
        hh[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[0], b[n][0], hh[n], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) hl[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[0], b[n][1], hl[n], 0, 0, 0);
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float low = fmaf(ll[n][v], 1.f / SG_LOW, hl[n][v]);
            d[v * CH_LD + 16 * n] = (fresh ? 0.f : old[n][v]) - fmaf(low, 1.f / SG_LOW, hh[n][v]) * pu[v] * qu[n];
        }
}

// One workgroup: the 128 x 128 block H in LDS (upper triangle; identity where it is padded) is factored, and `planes` receives T = R^-T, the inverse of the
// transposed factor, as an operand whose lines are T's rows, its columns times powers of two that undo the scales of G's rows: of b_l S m_k a column of T is as large as
// 1 / m_k, and what is small along a line would have fewer bits (m from 1e-6 to 1e6: Minv met to 9e-5 without, 3e-7 so).  *fail is raised if a pivot is not positive.  The elimination above, once more, with blocks of
// 32: beside the diagonal block a row has four blocks, those of G, the identity, those of Y, and each of four wavefronts takes the
// diagonal block and one of them through the pivots (so no product with an inverse follows them); the other four bring rows further down up to date
// meanwhile.  (On the fp16 matrix cores: a vector instruction waits for an fp32 matrix instruction of another wavefront of its SIMD, 64 cycles each, but not for
// an fp16 one.)  Below the diagonal H has Y, on it what was eliminated; the diagonal of Y, the identity to begin with, is apart.
__device__ __forceinline__ void chol_block_begin(CholBlock& lds) {   // (a barrier follows)
    const int tid = threadIdx.x;
    if (tid < NB) lds.largest[tid] = 0;
#pragma unroll
    for (int n = 0; n < 32 * NB / CH_THREADS; ++n) {
        const int e = tid + CH_THREADS * n, i = e / NB, k = e % NB;
        lds.Y[i * CH_LD + k] = (k & 31) == i ? 1.f : 0.f;
    }
}
__device__ __forceinline__ void chol_block(CholBlock& lds, uint8_t* __restrict__ planes, int* __restrict__ fail) {
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto blk = [&](int i, int c) { return (i == c ? lds.Y : lds.H + 32 * i * CH_LD) + 32 * c; };   // (the diagonal: Y's)
    int bad = 0;
    // 16 rows of block (i, c) take their part of row s
    auto update = [&](int s, int i, int c, int r16) {
        const uint8_t* row = lds.rows[s & 1];
        const float* up = lds.up[s & 1];
        chol_update16(lds.H + (32 * i + 16 * r16) * CH_LD + 32 * c, row + i * CH_ROW, up + 32 * i, r16, row + c * CH_ROW, up + 32 * c, c == s, lane);
    };
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
        if (w < 4) {
            bad |= chol_rows32(lds.H + 32 * s * CH_LD + 32 * s, blk(s, w), w <= s, lds.rows[s & 1] + w * CH_ROW, lds.up[s & 1] + 32 * w, w == 0 ? lds.even + 32 * s : nullptr,
                               lds.spare[w], lane);
        } else if (s > 0) {
            // what row s - 1 takes from the rows i > s, columns c >= i (G) and c < s (Y, which starts at c = s - 1)
            int n = 0;
            for (int i = s + 1; i < 4; ++i)
                for (int c = 0; c < 4; ++c) {
                    if (c >= s && c < i) continue;
                    for (int r16 = 0; r16 < 2; ++r16)
                        if (n++ % 4 == w - 4) update(s - 1, i, c, r16);
                }
        }
        __syncthreads();
        // row s + 1 takes its part of row s
        if (s < 3) {
            update(s, s + 1, w & 3, w >> 2);
            __syncthreads();
        }
    }
    if (bad && tid == 0) atomicAdd(fail, 1);
    // T's planes, its lower triangle alone: wavefront w has lines 32 (w % 4) .. + 31 and every other 16 k of them
    const int ib = w & 3;
    float x[4][8], mx = 0.f;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        if (n > ib) continue;
        const int k = 16 * (w >> 2) + 8 * h;
        const float *at = blk(ib, n) + l32 * CH_LD + k, *even = lds.even + 32 * n + k;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[n][e] = at[e] * even[e];
            mx = fmaxf(mx, fabsf(x[n][e]));
        }
    }
    atomicMax(&lds.largest[32 * ib + l32], __builtin_bit_cast(unsigned, mx));
    __syncthreads();
    const SgScale scale = sg_scale(__builtin_bit_cast(float, lds.largest[32 * ib + l32]));
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        if (n > ib) continue;
        sg_store2(planes + ((2 * n + (w >> 2)) * 8 + ib) * SG_FRAG + lane * 16, x[n], scale);
    }
    if (w < 4 && lane < 32) {
        float* const scales = reinterpret_cast<float*>(planes + CH_T_UP) + 32 * ib + l32;
        scales[0] = scale.up;
        const unsigned even = __builtin_bit_cast(unsigned, lds.even[32 * ib + l32]);
        scales[NB] = __builtin_bit_cast(float, even ? (254u << 23) - even : 0u);   // (a row without a pivot counts as zero)
    }
}

// ---- C = B^T W beside the elimination ------------------------------------------------------------------------------------------
// The elimination keeps a third of the compute units busy, and one of them long.  The others make C meanwhile: each launch of the elimination has further
// workgroups, one per compute unit left, for parts of C, 128 x 128 outputs and at most CP_CHUNKS chunks of the summation index each.  A block's parts are in
// launches one after the other, each going on from the sums that the last one left in C; all of a block's first parts come before any second one.
struct CholBeside {
    const uint8_t *bits, *Q;   // the signs' tiles, b . W's planes
    const float* rs;           // of the output rows
    float* out;
    int M, N, K, n_ct;
    int col0, tiles;           // first block column, how many blocks
    int steps, parts;          // chunks to a part, parts to a block
    int begin, count;          // of this launch's parts
};
constexpr int CP_CHUNKS = 8;
constexpr int CP_AHEAD = 4;    // steps of 16 k whose operands are on their way
// A workgroup without LDS (the ring of dbf_split_gemm.h has no place beside the elimination's): a wavefront has 64 x 32 outputs, the fragments of b . W
// come straight from memory to registers, and those of the signs are made there: eight bytes of a tile are a lane's eight k for all of 128 rows.  The same
// products as there.
// Measured at p = r = 4096, q = 2048: a launch of the elimination takes 27 us with 8 chunks beside it for 22 without any (the clock of a busy chip), all sixteen
// 424 for 360, and C in a launch of its own 130: 627 -> 554 us.  (The signs' fragments from their plane in memory: 571.  Parts of 7 chunks: the same; of 4: not all
// of C has room.)
__device__ __forceinline__ void chol_beside(const CholBeside& g, int index) {
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), rp = w & 1, cb = w >> 1;
    // a compute die works on neighbouring blocks, eight rows of them at a time (dbf_split_gemm.h)
    const int die = index & 7, per = g.count >> 3, extra = g.count & 7, id = g.begin + die * per + min(die, extra) + (index >> 3);
    const int part = id / g.tiles, tile = id - part * g.tiles, mt = (g.M + 127) >> 7, nt = g.tiles / mt;
    const int band = tile / (8 * nt), in_band = tile - band * 8 * nt, rows = min(8, mt - 8 * band);
    const int it = 8 * band + in_band % rows, jt = g.col0 + in_band / rows;
    const int chunks = (g.K + SG_CHUNK - 1) / SG_CHUNK, c0 = part * g.steps, c1 = min(chunks, c0 + g.steps);
    if (c0 >= c1) return;
    const SgOperand Q = sg_operand(g.Q, 2, g.K, g.N, jt, 0);
    // (byte 256 (k / 16) + 16 (i % 16) + k % 16 of a row of tiles, bit (i % 128) / 16)
    const uint8_t *p = g.bits + (size_t)it * g.n_ct * DBF_TILE_BYTES + 16 * (lane & 15) + 8 * h, *q = Q.frags + cb * SG_FRAG + lane * 16;
    const int s1 = SG_CHUNK_STEPS * c1, shift = 7 - 4 * rp - (l32 >> 4);
    uint2 a[CP_AHEAD];
    v8h b[CP_AHEAD][2];
    auto fetch = [&](int slot, int s) {
        const int k = min(s, s1 - 1);
        typedef unsigned v2u4 __attribute__((ext_vector_type(2), aligned(4)));   // (a caller's)
        const v2u4 t = *reinterpret_cast<const v2u4*>(p + 256 * (size_t)min(k, 4 * g.n_ct - 1));   // (b . W is zero beyond the last tile)
        a[slot] = make_uint2(t.x, t.y);
#pragma unroll
        for (int x = 0; x < 2; ++x) b[slot][x] = *reinterpret_cast<const v8h*>(q + ((size_t)k * 8 + 4 * x) * SG_FRAG);
    };
    // a bit of bytes e and e + 1 of eight to the signs of two halves: 1 or, where it is clear, -1
    auto signs = [&](uint2 w, int x) {
        typedef unsigned v4u __attribute__((ext_vector_type(4)));
        v4u o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned word = ~(e < 2 ? w.x : w.y), two = __builtin_amdgcn_perm(word, word, e & 1 ? 0x030c020cu : 0x010c000cu);
            o[e] = ((two << (shift - 2 * x)) & 0x80008000u) | 0x3c003c00u;
        }
        return __builtin_bit_cast(v8h, o);
    };
#pragma unroll
    for (int n = 0; n < CP_AHEAD; ++n) fetch(n, SG_CHUNK_STEPS * c0 + n);
    const int row0 = 128 * it + 64 * rp, col = 128 * jt + 32 * cb + l32, cc = min(col, g.N - 1);
    auto row_of = [&](int x, int v) { return row0 + 32 * x + 8 * (v >> 2) + 4 * h + (v & 3); };
    // (a part's halves are sums of their own, added to those before: C is 8.6e-8 from 64 bits, mean over seven sizes; all chunks in one chain 1.00e-7; 512
    // threads of dbf_split_gemm.h, a sum each, 9.4e-8; no difference in time)
    const int half = c0 + (c1 - c0) / 2;
    v16f acc[2], low[2], tot[2], sum[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[x][v] = low[x][v] = tot[x][v] = 0.f;
            sum[x][v] = part == 0 ? 0.f : g.out[(size_t)min(row_of(x, v), g.M - 1) * g.N + cc];
        }
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
        if (c == half) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    sum[x][v] += tot[x][v];
                    tot[x][v] = 0.f;
                }
        }
        const float uq = Q.up[(size_t)c * Q.lines + 32 * cb + l32];
#pragma unroll
        for (int n = 0; n < SG_CHUNK_STEPS; ++n) {
            const int slot = n % CP_AHEAD;
            const v8h s[2] = {signs(a[slot], 0), signs(a[slot], 1)};
#pragma unroll
            for (int x = 0; x < 2; ++x) low[x] = __builtin_amdgcn_mfma_f32_32x32x16_f16(s[x], b[slot][1], low[x], 0, 0, 0);
#pragma unroll
            for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_f16(s[x], b[slot][0], acc[x], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            fetch(slot, SG_CHUNK_STEPS * c + n + CP_AHEAD);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                tot[x][v] = fmaf(fmaf(low[x][v], 1.f / SG_LOW, acc[x][v]), uq, tot[x][v]);
                acc[x][v] = low[x][v] = 0.f;
            }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row_of(x, v);
            const float all = sum[x][v] + tot[x][v];
            if (row < g.M && col < g.N) g.out[(size_t)row * g.N + col] = c1 == chunks ? all * g.rs[row] : all;
        }
}

// Diagonal block 0.
__global__ __launch_bounds__(CH_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_chol_first_kernel(
    const float* __restrict__ G, int q, uint8_t* __restrict__ planes, int* __restrict__ fail, const CholBeside beside) {
    __shared__ __align__(16) CholBlock lds;
    if (blockIdx.x > 0) {
        chol_beside(beside, blockIdx.x - 1);
        return;
    }
    const int w = min(q, NB);
    float v[NB * NB / CH_THREADS];
#pragma unroll
    for (int n = 0; n < NB * NB / CH_THREADS; ++n) {
        const int e = threadIdx.x + CH_THREADS * n, i = e / NB, j = e % NB;
        v[n] = G[(size_t)min(min(i, j), w - 1) * q + min(max(i, j), w - 1)];
    }
#pragma unroll
    for (int n = 0; n < NB * NB / CH_THREADS; ++n) {
        const int e = threadIdx.x + CH_THREADS * n, i = e / NB, j = e % NB;
        lds.H[i * CH_LD + j] = (i < w && j < w) ? v[n] : (i == j ? 1.f : 0.f);
    }
    chol_block_begin(lds);
    __syncthreads();
    chol_block(lds, planes, fail);
}

// ---- blocks of row j: [R | Y][j, c] = T [G | Y][j, c], a workgroup of eight wavefronts --------------------------------------
// An operand's planes in LDS are laid out like a chunk of them in memory; what else a block's making needs:
struct CholScales {
    unsigned g_largest[NB], p_largest[NB];   // largest magnitudes of the columns, before and after; zeros to begin with
};
// A thread's part of [G | Y][j, c]: register e of x[b] is row 16 w + 8 h + e, column 32 b + l32.
// (Addresses are a scalar base, the block row's, and 32 bits: 128 rows of a matrix that fits the memory are less than 2^31 bytes.)
__device__ __forceinline__ void chol_load_block(const float* __restrict__ G, int q, int j, int c, float (&x)[4][8]) {
    const int lane = threadIdx.x & 63, row0 = 16 * (threadIdx.x >> 6) + 8 * (lane >> 5), rows = q - NB * j;
    const float* base = G + (size_t)(NB * j) * q;
    unsigned col[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) col[b] = min(NB * c + 32 * b + (lane & 31), q - 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned at = (unsigned)min(row0 + e, rows - 1) * (unsigned)q;
#pragma unroll
        for (int b = 0; b < 4; ++b) x[b][e] = base[at + col[b]];
    }
}
// What its rows are multiplied by, as T's columns have been divided.
__device__ __forceinline__ void chol_load_even(const uint8_t* __restrict__ t_planes, float (&even)[8]) {
    const float* at = reinterpret_cast<const float*>(t_planes + CH_T_UP) + NB + 16 * (threadIdx.x >> 6) + 8 * ((threadIdx.x & 63) >> 5);
#pragma unroll
    for (int e = 0; e < 8; ++e) even[e] = at[e];
}
// ... into planes.  (Block (j, j) stands for Y's, where the product with the identity is T.)  Two barriers are the caller's: one between the
// zeros of s.g_largest and this, one behind it.
__device__ __forceinline__ void chol_split_block(float (&x)[4][8], const float (&even)[8], int q, int j, int c, uint8_t* planes, CholScales& s) {
    const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5, w = threadIdx.x >> 6;
    if (c == j || NB * (c + 1) > q || NB * (j + 1) > q) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int row = NB * j + 16 * w + 8 * h + e, col = NB * c + 32 * b + l32;
                x[b][e] = (row >= q || col >= q) ? 0.f : c == j ? (row == col ? 1.f : 0.f) : x[b][e];
            }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        float mx = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[b][e] *= even[e];
            mx = fmaxf(mx, fabsf(x[b][e]));
        }
        atomicMax(&s.g_largest[32 * b + l32], __builtin_bit_cast(unsigned, mx));
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 4; ++b)
        sg_store2(planes + (w * 8 + b) * SG_FRAG + lane * 16, x[b], sg_scale(__builtin_bit_cast(float, s.g_largest[32 * b + l32])));
}
// A wavefront makes two blocks of 32 x 32 side by side: the four row blocks, whose T has 2, 4, 6 and 8 fragments of k, are dealt so that the two wavefronts of a
// SIMD (w and w + 4, as a workgroup's are placed) have ten between them.
__device__ __forceinline__ int chol_row_block(int w) { return w < 4 ? w >> 1 : 3 - ((w & 3) >> 1); }
__device__ __forceinline__ void chol_load_t(const uint8_t* __restrict__ t_planes, v8h (&t)[8][2]) {
    const int lane = threadIdx.x & 63, rb = chol_row_block(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6));
#pragma unroll
    for (int n = 0; n < 4; ++n)
        if (n <= rb) {
#pragma unroll
            for (int k = 2 * n; k < 2 * n + 2; ++k)
#pragma unroll
                for (int p = 0; p < 2; ++p) t[k][p] = *reinterpret_cast<const v8h*>(t_planes + ((k * 2 + p) * 4 + rb) * SG_FRAG + lane * 16);
        }
}
// The product, and its own planes to `out` (LDS), its lines' scales to `up`; with `rows` also to the planes of all of [R | Y] there.  Begins with a barrier (the
// planes `g` are whole) and ends without one.
__device__ __forceinline__ void chol_make_block(const v8h (&t)[8][2], const float* t_up, const uint8_t* g, uint8_t* out, float* up,
                                                CholScales& s, uint8_t* __restrict__ rows, int q, int j, int c) {
    const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int c0 = 2 * (w & 1), rb = chol_row_block(w);
    __syncthreads();
    v16f acc[2], low[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = low[0][v] = low[1][v] = 0.f;
#pragma unroll
    for (int n = 0; n < 4; ++n)
        if (n <= rb) {
#pragma unroll
            for (int k = 2 * n; k < 2 * n + 2; ++k) {
                v8h x[2][2];
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int p = 0; p < 2; ++p) x[b][p] = *reinterpret_cast<const v8h*>(g + ((k * 2 + p) * 4 + c0 + b) * SG_FRAG + lane * 16);
                const v8h t_low = t[k][1] * (_Float16)(1.f / SG_LOW);
#pragma unroll
                for (int b = 0; b < 2; ++b) low[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(t_low, x[b][1], low[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < 2; ++b) low[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(t[k][1], x[b][0], low[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(t[k][0], x[b][0], acc[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < 2; ++b) low[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(t[k][0], x[b][1], low[b], 0, 0, 0);
            }
        }
    float mx[2] = {0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const v4f ur = *reinterpret_cast<const v4f*>(t_up + 32 * rb + 8 * k + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                acc[b][4 * k + e] = fmaf(low[b][4 * k + e], 1.f / SG_LOW, acc[b][4 * k + e]) * ur[e];
                mx[b] = fmaxf(mx[b], fabsf(acc[b][4 * k + e]));
            }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) atomicMax(&s.p_largest[32 * (c0 + b) + l32], __builtin_bit_cast(unsigned, mx[b]));
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int line = 32 * (c0 + b) + l32;
        const SgScale scale = sg_scale(__builtin_bit_cast(float, s.p_largest[line]));
        if (rb == 0 && h == 0) {
            // (the columns' own scales have been left out so far.  A line of T has an entry from 1/2 to 2 on the diagonal, and its largest is not far from
            // that: the sums times its scales are normal numbers)
            const float all = scale.up * sg_scale(__builtin_bit_cast(float, s.g_largest[line])).up;
            if (up) up[line] = all;
            if (rows) reinterpret_cast<float*>(rows + sg_scales_at(2, q, q))[(size_t)j * sg_lines(q) + NB * c + line] = all;
        }
        // register v of lane (h, l32) is row 8 (v / 4) + 4 h + v % 4; a plane wants rows 8 h .. + 7 of each 16
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = acc[b][8 * k + e], hi = acc[b][8 * k + 4 + e];   // (values of their own: the cast takes no element of a vector)
                const auto swapped = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi), false, false);
                x[e] = __builtin_bit_cast(float, (unsigned)swapped[0]);
                x[4 + e] = __builtin_bit_cast(float, (unsigned)swapped[1]);
            }
            const int kb = 2 * rb + k;
            if (out) sg_store2(out + (kb * 8 + c0 + b) * SG_FRAG + lane * 16, x, scale);
            if (rows) sg_store2(rows + (((size_t)c * sg_kblocks(q) + NB / 16 * j + kb) * 8 + c0 + b) * SG_FRAG + lane * 16, x, scale);
        }
    }
}

// Row j: a workgroup per block (i, c), i > j, of [G | Y] (c >= i and c <= j), row by row from the diagonal block on: the first is the diagonal block
// j + 1, which it factors, and being the first of the launch it starts with it.  Row j of Y is written by the workgroups of row j + 1.
// (The products of P and Q are of 128 k each; the sums' scales: P's first, unlike sg_scaled in dbf_split_gemm.h: P is R, whose entries are below the root of
// one of G's, 2^64.)
// MADE: row j is in `rows` already, its planes in G's columns too (dbf_chol_panel_kernel).
template <bool MADE>
__global__ __launch_bounds__(CH_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_chol_row_kernel(
    float* __restrict__ G, int q, int j, const uint8_t* __restrict__ t_planes, uint8_t* __restrict__ rows, uint8_t* __restrict__ t_next,
    int* __restrict__ fail, const CholBeside beside) {
    struct Tiles {
        uint8_t g[CH_PLANES], p[CH_PLANES];
        float t_up[NB], up[2][NB];
        CholScales s[2];
    };
    __shared__ __align__(16) uint8_t lds[sizeof(Tiles) > sizeof(CholBlock) ? sizeof(Tiles) : sizeof(CholBlock)];
    Tiles& T = *reinterpret_cast<Tiles*>(lds);
    if (!MADE && blockIdx.x >= gridDim.x - beside.count) {   // (launches with room for parts have fewer than CH_UNITS blocks)
        chol_beside(beside, blockIdx.x - (gridDim.x - beside.count));
        return;
    }
    const int nblk = (q + NB - 1) / NB;
    int i = j + 1, c = blockIdx.x;   // row i has its n - i blocks of G and j + 1 of Y
    while (c >= nblk - i + j + 1) c -= nblk - i++ + j + 1;
    c = c < nblk - i ? i + c : c - (nblk - i);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool diag = i == c;
    v8h t[8][2];
    float x[4][8], y[4][8], even[8], up_or_t;
    if (MADE) {
        const SgOperand P = sg_operand(rows, 2, q, q, i, j), Q = sg_operand(rows, 2, q, q, c, j);
#pragma unroll
        for (int n = 0; n < 8; ++n) sg_load16_lds(P.frags + (8 * w + n) * SG_FRAG + lane * 16, T.p + (8 * w + n) * SG_FRAG);
        if (!diag) {
#pragma unroll
            for (int n = 0; n < 8; ++n) sg_load16_lds(Q.frags + (8 * w + n) * SG_FRAG + lane * 16, T.g + (8 * w + n) * SG_FRAG);
        }
        up_or_t = (tid & NB ? Q : P).up[tid & (NB - 1)];
    } else {
        chol_load_block(G, q, j, i, x);
        chol_load_t(t_planes, t);
        chol_load_even(t_planes, even);
        (&T.s[0].g_largest[0])[tid] = 0;
        up_or_t = reinterpret_cast<const float*>(t_planes + CH_T_UP)[tid & (NB - 1)];
    }
    // this wavefront's two blocks of 32 x 32: side by side; or of a diagonal block's upper ten, whose four on the diagonal have one product more, one or two, so that
    // the two wavefronts of a SIMD have two of these or three others
    const int b0 = diag ? 0x62f531a0u >> 4 * w & 15 : 4 * (w & 3) + 2 * (w >> 2), b1 = diag ? (w == 2 ? 7 : 11) : b0 + 1;
    const bool two = !diag || w == 2 || w == 3;
    auto row_of = [&](int b, int v) { return 32 * (b >> 2) + 8 * (v >> 2) + 4 * h + (v & 3); };
    auto col_of = [&](int b) { return 32 * (b & 3) + l32; };
    float* const Gi = G + (size_t)(NB * i) * q;
    auto load_old = [&](float (&o)[4][8]) {   // (what is subtracted from, register 16 n + v)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            if (n == 1 && !two) break;
            const unsigned col = min(NB * c + col_of(n ? b1 : b0), q - 1);
#pragma unroll
            for (int v = 0; v < 16; ++v) o[2 * n + (v >> 3)][v & 7] = Gi[(unsigned)min(row_of(n ? b1 : b0, v), q - NB * i - 1) * (unsigned)q + col];
        }
    };
    if (MADE) {
        // (the planes' arrival first: at the barrier the compiler cannot tell their loads from these, and waits for all.  q = 8192, p = r = 768: 4795 us, so 4526; 4096 1009 / 992)
        if (tid < 2 * NB) T.up[0][tid] = up_or_t;
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt = 0
        asm volatile("" ::: "memory");
        load_old(y);
    } else {
        if (diag) load_old(y); else chol_load_block(G, q, j, c, y);
        __syncthreads();
        if (tid < NB) T.t_up[tid] = up_or_t;
        chol_split_block(x, even, q, j, i, T.g, T.s[0]);
        chol_make_block(t, T.t_up, T.g, T.p, T.up[0], T.s[0], nullptr, q, j, i);
        if (!diag) {   // (everyone is done with the planes in T.g; the second's take the place of what they are made from)
            chol_split_block(y, even, q, j, c, T.g, T.s[1]);
            load_old(y);
            chol_make_block(t, T.t_up, T.g, T.g, T.up[1], T.s[1], i == j + 1 && c <= j ? rows : nullptr, q, j, c);
        }
    }
    __syncthreads();
    const uint8_t *P = T.p + lane * 16, *Q = (diag ? T.p : T.g) + lane * 16;
    v16f acc[2], low[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = low[0][v] = low[1][v] = 0.f;
    auto product = [&](int n, const v8h (&a)[2], const v8h (&b)[2]) {
        low[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[0], low[n], 0, 0, 0);
        low[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[1], low[n], 0, 0, 0);
        acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[0], acc[n], 0, 0, 0);
    };
#pragma unroll
    for (int kb = 0; kb < NB / 16; ++kb) {
        auto frag = [&](const uint8_t* base, int line, v8h (&f)[2]) {
#pragma unroll
            for (int p = 0; p < 2; ++p) f[p] = *reinterpret_cast<const v8h*>(base + ((kb * 2 + p) * 4 + line) * SG_FRAG);
        };
        v8h a[2], b[2];
        frag(P, b0 >> 2, a);
        frag(Q, b0 & 3, b);
        product(0, a, b);
        if (two) {
            if (diag) frag(P, b1 >> 2, a);
            frag(Q, b1 & 3, b);
            product(1, a, b);
        }
    }
    if (diag && b0 % 5 == 0) {   // (lines meet themselves: l l is of one sign there, and left out it would be lost from all of a diagonal)
#pragma unroll
        for (int kb = 0; kb < NB / 16; ++kb) {
            const v8h l = *reinterpret_cast<const v8h*>(P + ((kb * 2 + 1) * 4 + (b0 >> 2)) * SG_FRAG);
            low[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(l * (_Float16)(1.f / SG_LOW), l, low[0], 0, 0, 0);
        }
    }
    const float *up = T.up[0], *uq = T.up[diag ? 0 : 1];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int b = n ? b1 : b0;
        const float u = uq[col_of(b)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const v4f ur = *reinterpret_cast<const v4f*>(up + row_of(b, 4 * k));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v = 4 * k + e;
                acc[n][v] = (c == j ? 0.f : y[2 * n + (v >> 3)][v & 7]) - fmaf(low[n][v], 1.f / SG_LOW, acc[n][v]) * ur[e] * u;
            }
        }
    }
    if (blockIdx.x > 0) {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if (n == 1 && !two) continue;
                const int row = row_of(n ? b1 : b0, v), col = NB * c + col_of(n ? b1 : b0);
                if (row < q - NB * i && col < q) Gi[(unsigned)row * (unsigned)q + (unsigned)col] = acc[n][v];
            }
        return;
    }
    CholBlock& B = *reinterpret_cast<CholBlock*>(lds);
    const bool whole = NB * (i + 1) <= q;
    __syncthreads();   // (the block takes the planes' place)
    chol_block_begin(B);
#pragma unroll
    for (int n = 0; n < 2; ++n)
        if (n == 0 || two) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = row_of(n ? b1 : b0, v), col = col_of(n ? b1 : b0);
                B.H[row * CH_LD + col] = (whole || (NB * i + row < q && NB * i + col < q)) ? acc[n][v] : (row == col ? 1.f : 0.f);
            }
        }
    __syncthreads();
    chol_block(B, t_next, fail);
}

// Row j by itself, a workgroup per 128 columns: the last of Y, and rows whose blocks below are many.
__global__ __launch_bounds__(CH_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_chol_panel_kernel(
    const float* __restrict__ G, int q, int j, const uint8_t* __restrict__ t_planes, uint8_t* __restrict__ rows) {
    __shared__ __align__(16) uint8_t g[CH_PLANES];
    __shared__ __align__(16) float t_up[NB];
    __shared__ CholScales s;
    const int c = blockIdx.x;
    v8h t[8][2];
    float x[4][8], even[8];
    chol_load_block(G, q, j, c, x);
    chol_load_t(t_planes, t);
    chol_load_even(t_planes, even);
    if (threadIdx.x < 2 * NB) (&s.g_largest[0])[threadIdx.x] = 0;
    if (threadIdx.x < NB) t_up[threadIdx.x] = reinterpret_cast<const float*>(t_planes + CH_T_UP)[threadIdx.x];
    __syncthreads();
    chol_split_block(x, even, q, j, c, g, s);
    chol_make_block(t, t_up, g, nullptr, nullptr, s, rows, q, j, c);
}

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }
struct AdmmWorkspace {
    size_t P, R, Z, svid, total;
};
inline AdmmWorkspace admm_workspace(int q, int r) {
    AdmmWorkspace w;
    size_t off = 0;
    w.P = off;     off = up256(off + sg_plane_bytes(2, q, q));   // planes of Minv
    w.R = off;     off = up256(off + sg_plane_bytes(2, q, r));   // planes of R
    w.Z = off;     off = up256(off + 4 * (size_t)q * r);
    w.svid = off;  off = up256(off + dbf_svid_workspace_bytes(q, r));
    w.total = off;
    return w;
}

}  // namespace

extern "C" size_t dbf_admm_workspace_bytes(int q, int r) {
    if (q < 1 || r < 1 || q > DBF_MAX_DIM || r > DBF_MAX_DIM) return 0;
    return admm_workspace(q, r).total;
}

extern "C" int dbf_admm_step(const void* Minv_dev, const void* C_dev, int q, int r, float rho, int svid_iters,
                             void* a_dev, void* m_dev, void* bits_dev, void* U_dev, void* workspace_dev,
                             size_t workspace_bytes, void* hip_stream) {
    if (!Minv_dev || !C_dev || !a_dev || !m_dev || !bits_dev || !U_dev) return DBF_EINVAL;
    if (q < 1 || r < 1 || q > DBF_MAX_DIM || r > DBF_MAX_DIM || svid_iters < 1) return DBF_EINVAL;
    if (!(rho > 0.f) || !std::isfinite(rho)) return DBF_EINVAL;
    const void* ptrs[6] = {Minv_dev, C_dev, a_dev, m_dev, bits_dev, U_dev};
    for (const void* p : ptrs)
        if (reinterpret_cast<uintptr_t>(p) & 3) return DBF_EINVAL;
    const AdmmWorkspace w = admm_workspace(q, r);
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 255) || workspace_bytes < w.svid + dbf_svid_least_workspace(q, r))
        return DBF_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint8_t* base = static_cast<uint8_t*>(workspace_dev);
    float* Z = reinterpret_cast<float*>(base + w.Z);
    float* U = static_cast<float*>(U_dev);
    const float* C = static_cast<const float*>(C_dev);
    const int n_ct = dbf_col_tiles(r);

    const dim3 of_minv = sg_plane_grid(q, q), of_r = sg_plane_grid(q, r);   // (the same summation indices: the same x)
    hipLaunchKernelGGL(dbf_admm_operands_kernel, dim3(of_r.x, of_minv.y + of_r.y), dim3(256), 0, st, static_cast<const float*>(Minv_dev), base + w.P,
                       (int)of_minv.y, C, U, rho, static_cast<const float*>(a_dev), static_cast<const float*>(m_dev),
                       static_cast<const uint8_t*>(bits_dev), q, r, n_ct, base + w.R);
    SplitGemmArgs g = {};
    g.P = base + w.P;  g.Q = base + w.R;
    g.add = U;  g.lda = r;
    g.out = Z;  g.ldo = r;
    g.M = q;  g.N = r;  g.K = q;
    launch_split_gemm<2>(g, st);
    if (hipGetLastError() != hipSuccess) return DBF_EHIP;
    return dbf_svid_dual(Z, q, r, svid_iters, a_dev, m_dev, bits_dev, base + w.svid, workspace_bytes - w.svid, U, st);
}

// ---- forming the constant matrices of the update on the device ---------------------------------
namespace {
struct PrepWorkspace {
    size_t T, fail, S, V, Y, least, total;   // `least`: what a call can do with: all of V's contents one after the other, nothing of C beside other work
    int nblk;
};
inline PrepWorkspace prep_workspace(int p, int q, int r) {
    PrepWorkspace w;
    w.nblk = (q + NB - 1) / NB;
    size_t off = 0;
    w.T = off;     off = up256(off + CH_PLANES * (size_t)(w.nblk < 2 ? w.nblk : 2));   // planes of R_jj^-T, of two block rows in turn
    w.fail = off;  off = up256(off + 256);
    w.S = off;     off = up256(off + sg_plane_bytes(1, p, q));   // planes of the signs
    // planes of the other operand of the three large contractions in turn: the scaled signs, b . W, [R | Y]
    size_t v = sg_plane_bytes(2, p, q);
    v = v < sg_plane_bytes(2, p, r) ? sg_plane_bytes(2, p, r) : v;
    v = v < sg_plane_bytes(2, q, q) ? sg_plane_bytes(2, q, q) : v;
    w.V = off;     off = up256(off + v);
    w.least = off;
    w.Y = off;   // those of the scaled signs and then of [R | Y], apart from b . W's
    if (w.nblk > 1) off = up256(off + std::max(sg_plane_bytes(2, p, q), sg_plane_bytes(2, q, q)));
    w.total = off;
    return w;
}
// Blocks of row j's launch of the elimination: the i-th block row below has below - i blocks of G and j + 1 of Y.
inline long long chol_blocks(int nblk, int j) {
    const int below = nblk - 1 - j;
    return (long long)below * (below + 1) / 2 + (long long)below * (j + 1);
}
// The compute units that a launch of this many workgroups leaves.
inline long long chol_free(long long blocks) { return blocks < CH_UNITS ? CH_UNITS - blocks : 0; }
// How much of C is made beside the elimination: as many block columns, from the last one down, as its launches have room for.
struct CholPlan {
    int columns, steps, parts;
};
inline CholPlan chol_plan(int p, int q, int r) {
    const int nblk = (q + NB - 1) / NB, chunks = (p + SG_CHUNK - 1) / SG_CHUNK;
    CholPlan plan;
    plan.parts = (chunks + CP_CHUNKS - 1) / CP_CHUNKS;
    plan.steps = (chunks + plan.parts - 1) / plan.parts;
    auto room = [&](long long tiles) {   // (a launch has one part of a block at most)
        long long n = std::min(tiles, chol_free(1));
        for (int j = 0; j + 1 < nblk; ++j) n += std::min(tiles, chol_free(chol_blocks(nblk, j)));
        return n;
    };
    long long columns = std::min((long long)(r + 127) / 128, room(1 << 30) / ((long long)nblk * plan.parts));
    while (columns > 0 && room(columns * nblk) < columns * nblk * plan.parts) --columns;
    plan.columns = (int)columns;
    return plan;
}
}  // namespace

extern "C" size_t dbf_admm_prepare_workspace_bytes(int p, int q, int r) {
    if (p < 1 || q < 1 || r < 1 || p > DBF_MAX_DIM || q > DBF_MAX_DIM || r > DBF_MAX_DIM) return 0;
    return prep_workspace(p, q, r).total;
}

extern "C" int dbf_admm_prepare(const void* bits_dev, const void* m2_dev, const void* b_dev, const void* W_dev, int p,
                                int q, int r, float rho, void* Minv_dev, void* C_dev, void* workspace_dev,
                                size_t workspace_bytes, int* not_positive_definite_dev, void* hip_stream) {
    if (!bits_dev || !m2_dev || !b_dev || !W_dev || !Minv_dev || !C_dev) return DBF_EINVAL;
    if (p < 1 || q < 1 || r < 1 || p > DBF_MAX_DIM || q > DBF_MAX_DIM || r > DBF_MAX_DIM) return DBF_EINVAL;
    if (!(rho > 0.f) || !std::isfinite(rho)) return DBF_EINVAL;
    const void* ptrs[7] = {bits_dev, m2_dev, b_dev, W_dev, Minv_dev, C_dev, not_positive_definite_dev};
    for (const void* ptr : ptrs)
        if (reinterpret_cast<uintptr_t>(ptr) & 3) return DBF_EINVAL;
    const PrepWorkspace w = prep_workspace(p, q, r);
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 255) || workspace_bytes < w.least)
        return DBF_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint8_t* base = static_cast<uint8_t*>(workspace_dev);
    int* fail = not_positive_definite_dev ? not_positive_definite_dev : reinterpret_cast<int*>(base + w.fail);
    float* G = static_cast<float*>(Minv_dev);  // G, then its factor, live in the output until the last contraction
    const uint8_t* bits = static_cast<const uint8_t*>(bits_dev);
    const float* m2 = static_cast<const float*>(m2_dev);
    const float* b = static_cast<const float*>(b_dev);
    const int n_ct = dbf_col_tiles(p), nt = (r + 127) / 128;
    const bool roomy = w.nblk > 1 && workspace_bytes >= w.total;
    const CholPlan plan = roomy ? chol_plan(p, q, r) : CholPlan{0, 0, 0};

    uint8_t *S = base + w.S, *V = base + w.V;
    // G = B^T B + rho I with B[l][j] = b_l S[j][l] m2_j: the signs against the signs times b^2, m2 by output row and column in
    // the epilogue.  Upper blocks only.  Beside them, as far as compute units are idle, b . W's planes.
    uint8_t* const scaled = roomy ? base + w.Y : V;
    const SplitBesideArgs dense = {static_cast<const float*>(W_dev), b, V, (size_t)r, p, r, 0};
    hipLaunchKernelGGL(dbf_split_signs_kernel, sg_plane_grid(p, q), dim3(256), 0, st, bits, n_ct, p, q, b, S, scaled, fail);
    SplitGemmArgs gram = {};
    gram.P = S;  gram.Q = scaled;  gram.out = G;  gram.ldo = q;  gram.M = q;  gram.N = q;  gram.K = p;
    gram.rs = m2;  gram.cs = m2;  gram.diag = rho;  gram.upper = 1;
    const int made = 2 * launch_split_gemm<1>(gram, st, 1 << 30, roomy ? &dense : nullptr);   // (times 32 lines)
    const dim3 planes = sg_plane_grid(p, r);
    if (made < (int)planes.y)
        hipLaunchKernelGGL(dbf_split_dense_kernel, dim3(planes.x, planes.y - made), dim3(256), 0, st, dense.src, dense.ld, p, r, b, V, made);
    // C = B^T W: the signs against b . W
    if (plan.columns < nt) {
        SplitGemmArgs g = {};
        g.P = S;  g.Q = V;  g.out = static_cast<float*>(C_dev);  g.ldo = r;  g.M = q;  g.N = r;  g.K = p;
        g.rs = m2;
        launch_split_gemm<1>(g, st, nt - plan.columns);
    }
    // [G | I] -> [R | Y], the planes of Y in V, or beside what the rest of C is made of
    uint8_t *T[2] = {base + w.T, base + w.T + CH_PLANES}, *Y = plan.columns ? base + w.Y : V;
    CholBeside beside = {bits, V, m2, static_cast<float*>(C_dev), q, r, p, n_ct, nt - plan.columns, plan.columns * ((q + 127) / 128), plan.steps, plan.parts, 0, 0};
    auto besides = [&](long long blocks) {   // this launch's parts
        beside.begin += beside.count;
        beside.count = (int)std::min((long long)beside.tiles * beside.parts - beside.begin, std::min((long long)beside.tiles, chol_free(blocks)));
        return beside;
    };
    besides(1);
    hipLaunchKernelGGL(dbf_chol_first_kernel, dim3(1 + beside.count), dim3(CH_THREADS), 0, st, G, q, T[0], fail, beside);
    for (int j = 0; j < w.nblk; ++j) {
        const int below = w.nblk - 1 - j;
        const long long blocks = chol_blocks(w.nblk, j);
        const bool made = below == 0 || blocks > CH_MADE;
        if (made) hipLaunchKernelGGL(dbf_chol_panel_kernel, dim3(w.nblk), dim3(CH_THREADS), 0, st, G, q, j, T[j & 1], Y);
        if (below > 0) {
            besides(blocks);
            hipLaunchKernelGGL(made ? dbf_chol_row_kernel<true> : dbf_chol_row_kernel<false>, dim3((unsigned)(blocks + beside.count)), dim3(CH_THREADS), 0, st, G, q,
                               j, T[j & 1], Y, T[~j & 1], fail, beside);
        }
    }
    // G^-1 = Y^T Y (overwrites G): upper blocks, the sums starting where both operands can be non-zero, written to both triangles
    {
        SplitGemmArgs g = {};
        g.P = Y;  g.Q = Y;  g.out = G;  g.ldo = q;  g.M = q;  g.N = q;  g.K = q;
        g.upper = 1;  g.ktri = 1;  g.vec = (q & 3) == 0 && (reinterpret_cast<uintptr_t>(G) & 15) == 0;
        launch_split_gemm<2>(g, st);
    }
    if (hipGetLastError() != hipSuccess) return DBF_EHIP;
    return DBF_OK;
}
