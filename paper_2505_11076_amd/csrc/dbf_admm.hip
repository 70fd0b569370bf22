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
//     U' = Z - a' . S' . m'^T  (= U + W_hat - A')   dbf_admm_dual_kernel
//
// The contraction is q x q x r in fp32 accuracy (34 GFLOP at q = 2048, r = 4096) and dominates; the elementwise
// kernels and the projection are bandwidth bound.  Measured at that size: the contraction 331 us on the fp32 matrix cores, 219 on the bf16
// ones with operands in three parts, 108 on the fp16 ones with operands in two, whose planes, with the making of R, take 22 us in one launch; the update
// with two rounds of SVID 388, 287, now 184 us; error against 64 bits 8.1e-6, 5.1e-6, 1.6e-6 (fewer roundings: 16 products enter the accumulator at
// once, and half as many of them).
// The paper gives no kernel design for this step.
#include "dbf_kernels.h"
#include "dbf_split_gemm.h"

#include <cmath>
#include <utility>

namespace {

// ---------------------------------------------------------------------------------------------
// Elementwise kernels.  One workgroup per 128 x 64 tile of the sign matrix; thread t takes the four
// columns 4 (t % 16) .. + 3 of rows 16 s + t / 16, s = 0 .. 7.  Their eight sign quadruples are the
// eight bits of the four bytes of ONE 32-bit word of the tile (byte 256 g + 16 r + j, bit s = sign of
// row 16 s + r, column 16 g + j), and a wavefront touches four rows of 256 contiguous bytes per pass.
// ---------------------------------------------------------------------------------------------
struct TileThread {
    int row0, col, word;  // first row (s = 0), first column, word index in the tile
};
__device__ inline TileThread tile_thread(int t) {
    const int rr = t >> 4, cq = t & 15;
    TileThread x;
    x.row0 = blockIdx.y * DBF_TILE_ROWS + rr;
    x.col = blockIdx.x * DBF_TILE_COLS + 4 * cq;
    x.word = 64 * (cq >> 2) + 4 * rr + (cq & 3);
    return x;
}

// U' = Z - a_i m_j s_ij
__global__ __launch_bounds__(256) void dbf_admm_dual_kernel(const float* __restrict__ Z, const float* __restrict__ a,
                                                           const float* __restrict__ m, const uint8_t* __restrict__ bits,
                                                           int rows, int cols, int n_ct, int vec_ok, float* __restrict__ out) {
    const TileThread x = tile_thread(threadIdx.x);
    if (x.col >= cols) return;
    const unsigned w =
        reinterpret_cast<const unsigned*>(bits + ((size_t)blockIdx.y * n_ct + blockIdx.x) * DBF_TILE_BYTES)[x.word];
    const bool vec = vec_ok && x.col + 4 <= cols;
    float mj[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) mj[e] = x.col + e < cols ? m[x.col + e] : 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int row = x.row0 + 16 * s;
        if (row >= rows) break;
        const float ai = a[row];
        const size_t at = (size_t)row * cols + x.col;
        float v[4], res[4];
        if (vec) {
            const v4f p = *reinterpret_cast<const v4f*>(Z + at);
            v[0] = p.x;  v[1] = p.y;  v[2] = p.z;  v[3] = p.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = x.col + e < cols ? Z[at + e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float am = ai * mj[e];
            res[e] = v[e] - (((w >> (8 * e + s)) & 1u) ? am : -am);
        }
        if (vec) {
            *reinterpret_cast<v4f*>(out + at) = (v4f){res[0], res[1], res[2], res[3]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (x.col + e < cols) out[at + e] = res[e];
        }
    }
}

// The operands of the contraction in one launch: the planes of Minv (blockIdx.y below q_blocks), and R = C + rho (a_k m_j s_kj - U) (q x r; k = its
// row is the summation index of the contraction), written straight into fp16 planes: R exists nowhere in fp32.  A lane's eight rows of R are
// one bit of eight bytes 16 apart of one sign tile.
__global__ __launch_bounds__(256) void dbf_admm_operands_kernel(const float* __restrict__ Minv, uint8_t* __restrict__ Minv_planes, int q_blocks,
                                                               const float* __restrict__ C, const float* __restrict__ U, float rho,
                                                               const float* __restrict__ a, const float* __restrict__ m,
                                                               const uint8_t* __restrict__ bits, int q, int r, int n_ct,
                                                               uint8_t* __restrict__ planes) {
    if ((int)blockIdx.y < q_blocks) {
        sg_split_dense<true>(Minv, q, q, q, nullptr, Minv_planes, blockIdx.y);
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
// G^-1 = Y^T Y is one more contraction.  Block row jb in two launches:
//   panel    [R | Y][jb, :] = R_jj^-T [G | Y][jb, :], all columns at once            dbf_chol_panel_kernel
//   update   [G | Y][i, :] -= R[jb, i]^T [R | Y][jb, :] for the block rows i > jb    dbf_chol_update_kernel
// and the workgroup of the update that makes diagonal block jb + 1 factors it and inverts its factor right there: that
// chain of 128 pivots, the longest of the whole, runs beside the other blocks' updates.
// G and Y share one q x q matrix: block (i, c) is G's for c >= i and Y's for c < i (an update starts it at zero at c = jb), and
// row jb of R is dead after its own update.  A finished row is written as the fp16 planes that the update and the last
// contraction read (R's for c > jb, Y's for c <= jb) and nowhere else.
// What bounds it: the chain.  Per block row 2 launches and 4 x 32 pivots; the update's products take 3 us of it.  Measured at
// q = 2048 (16 block rows): panel 5.6 us, update 31.6 us of which the pivots 25 while every entry of a pivot row went through a scalar register and
// the pivot's root stood in the chain; now 6.2 and 23.8.  With p = r = 4096 the constants took 890 us so, now 736.
// ---------------------------------------------------------------------------------------------
constexpr int NB = 128;        // block size: the contraction's tile
constexpr int CH_LD = NB + 4;  // LDS row length of a diagonal block: rows start on 16 bytes
constexpr int CH_LDT = 36;
constexpr int CH_LDS = 4 * (NB * CH_LD + 32 * CH_LDT);

// d -= P^T Q (or d = -P^T Q) for 32 x 32 blocks in LDS, 32 values of k: lane l supplies P[k][l % 32] and Q[k][l % 32], k = 2 kk + l / 32.
// (What is there is read with the operands, but subtracted from at the end: starting the sums from it rounds it 32 times.)
__device__ __forceinline__ void chol_update32(float* d, const float* P, const float* Q, bool fresh, int lane) {
    const int l32 = lane & 31, h = lane >> 5;
    float a[16], b[16];
    v16f acc, old;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
        a[kk] = P[(2 * kk + h) * CH_LD + l32];
        b[kk] = Q[(2 * kk + h) * CH_LD + l32];
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) old[v] = d[(8 * (v >> 2) + 4 * h + (v & 3)) * CH_LD + l32];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kk], b[kk], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) d[(8 * (v >> 2) + 4 * h + (v & 3)) * CH_LD + l32] = (fresh ? 0.f : old[v]) - acc[v];
}

// The operand of 16 x 16 outputs for 32 values of k: lane l supplies P[k][l % 16], k = 16 (kk / 4) + 4 (l / 16) + kk % 4 (rows four apart start 16 banks
// apart); register v of the result is row 4 (l / 16) + v, column l % 16.
__device__ __forceinline__ void chol_load16(const float* P, int ld, int lane, float (&x)[8]) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) x[kk] = P[(16 * (kk >> 2) + 4 * (lane >> 4) + (kk & 3)) * ld + (lane & 15)];
}

// x -= (lane N of each 16 of v) * t.  (Written out: the compiler makes two instructions of it.)
template <int N>
__device__ __forceinline__ void chol_sub(float& x, float v, float t) {
    asm("v_fmac_f32_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(x) : "v"(v), "v"(t), "n"(N));
}
template <int C, int... R>
__device__ __forceinline__ void chol_rows(float (&x)[32], float v0, float v1, float t, std::integer_sequence<int, R...>) {
    (chol_sub<(C + 1 + R) & 15>(x[C + 1 + R], C + 1 + R < 16 ? v0 : v1, t), ...);
}
// Pivot C, its value to lane C of piv: the rows below lose their multiples of row C.  t = x[C] / pivot (reciprocal and one Newton step), and lanes 0-15
// of x[C] in every 16 lanes of v0, lanes 16-31 in every 16 of v1.  (One block, so that what the instructions want between a write and a
// use is the work itself as far as it goes: one other before a lane read of a fresh register, two between the lane read and a use of its scalar
// register, two before a lane swap of a fresh register and before a lane broadcast of one, one behind the reciprocal.  The
// build checks the assembly for them: _wait_states_report in build.py.)
template <int C>
__device__ __forceinline__ void chol_pivot(float (&x)[32], float& piv) {
    float v0, v1, t, r, p;
    asm("v_mov_b32 %0, %6\n\t"
        "v_readlane_b32 %4, %6, %7\n\t"
        "v_mov_b32 %1, %6\n\t"
        "s_nop 0\n\t"
        "v_rcp_f32 %3, %4\n\t"
        "v_permlane32_swap_b32 %0, %1\n\t"
        "v_mov_b32 %1, %0\n\t"
        "v_fma_f32 %2, -%4, %3, 1.0\n\t"
        "v_fma_f32 %3, %2, %3, %3\n\t"
        "v_permlane16_swap_b32 %0, %1\n\t"
        "v_mul_f32 %2, %6, %3\n\t"
        "v_writelane_b32 %5, %4, %7"
        : "=&v"(v0), "=&v"(v1), "=&v"(t), "=&v"(r), "=&s"(p), "+v"(piv)
        : "v"(x[C]), "n"(C));
    chol_rows<C>(x, v0, v1, t, std::make_integer_sequence<int, 31 - C>());
}
template <int... C>
__device__ __forceinline__ void chol_pivots(float (&x)[32], float& piv, std::integer_sequence<int, C...>) {
    (chol_pivot<C>(x, piv), ...);
}

// The same for any pivots, in LDS and at leisure, with roots alone: pivots down to subnormal numbers (the instructions take none: a scaled copy) and up
// to the largest, rows of pivots that are not positive set to zero.  Returns whether there was one of the latter.
__device__ __forceinline__ int chol_factor32_any(float* H, float* T, int lane) {
    const int l32 = lane & 31;
    volatile float* X = lane < 32 ? H + l32 : T + l32;   // column l of the block or of the identity
    const int ld = lane < 32 ? CH_LD : CH_LDT;
    volatile float* G = H;
    int bad = 0;
    if (lane >= 32)
        for (int r = 0; r < 32; ++r) X[r * ld] = r == l32 ? 1.f : 0.f;
#pragma unroll 1
    for (int c = 0; c < 32; ++c) {
        const float piv = G[c * CH_LD + c];
        const bool tiny = piv < 0x1p-64f, pos = piv > 0.f;
        const float ps = tiny ? piv * 0x1p64f : piv;
        float y = __builtin_amdgcn_rsqf(ps);
        y = fmaf(0.5f * y, fmaf(-ps * y, y, 1.f), y);
        y = tiny ? y * 0x1p32f : y;
        bad |= !pos;
        const float xc = X[c * ld] * (pos ? y : 0.f);
        X[c * ld] = xc;
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int r = c + 1; r < 32; ++r) X[r * ld] = fmaf(-G[c * CH_LD + r], xc, X[r * ld]);
        __builtin_amdgcn_wave_barrier();
    }
    float x[32];
#pragma unroll
    for (int r = 0; r < 32; ++r) x[r] = X[r * ld];
    __builtin_amdgcn_wave_barrier();
    if (lane >= 32) {
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            G[r * CH_LD + l32] = x[r];
            T[l32 * CH_LDT + r] = x[r];
        }
    }
    return bad;
}

// One wavefront: the 32 x 32 diagonal block at H (leading dimension CH_LD, upper triangle read) is replaced by Y = R^-T
// (lower triangular, zeros above), and T (leading dimension CH_LDT) receives Y^T = R^-1.  Lane l < 32 holds column l of
// the block, lane 32 + l column l of the identity.  A pivot row's entries reach the other rows through lane broadcasts that are part
// of the multiplication; the rows are scaled by 1 / sqrt(pivot) at the end, all roots at once.  What bounds it: a wavefront on its own issues one
// instruction in four cycles, here 12 and one per row below for a pivot.  (With every entry through a scalar register, two
// instructions a row, and the root in the chain from pivot to pivot 8300 cycles; so 4400 with 11 instructions a pivot.)  Returns whether a pivot was not positive.
__device__ __forceinline__ int chol_factor32(float* H, float* T, int lane) {
    const int l32 = lane & 31;
    const bool right = lane >= 32;
    float x[32], piv = 1.f;
#pragma unroll
    for (int r = 0; r < 32; ++r) {
        x[r] = H[r * CH_LD + l32];
        asm("" : "+v"(x[r]));  // (loaded by all lanes, not in a branch of its own)
    }
#pragma unroll
    for (int r = 0; r < 32; ++r) x[r] = right ? (r == l32 ? 1.f : 0.f) : x[r];
    chol_pivots(x, piv, std::make_integer_sequence<int, 32>());
    // (below 2^-126, whose reciprocal and root the instructions do not take, 2^126 and more, whose reciprocal they do not return, or not positive)
    if (__any(__builtin_bit_cast(unsigned, piv) - 0x00800000u >= 0x7e000000u)) return chol_factor32_any(H, T, lane);
    float y = __builtin_amdgcn_rsqf(piv);
    y = fmaf(0.5f * y, fmaf(-piv * y, y, 1.f), y);
#pragma unroll
    for (int r = 0; r < 32; ++r) x[r] *= __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, y), r));
    if (right) {
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            H[r * CH_LD + l32] = x[r];
            T[l32 * CH_LDT + r] = x[r];
        }
    }
    return 0;
}

// One workgroup (256 threads): the 128 x 128 block in LDS (upper triangle; identity where it is padded) is factored, and tinv
// (128 x 128, row major, device memory) receives Y = R^-T, the inverse of the transposed factor: its 32 x 32 blocks on and below the diagonal.  *fail is raised if
// a pivot is not positive.  The elimination above, once more, with blocks of 32: all wavefronts bring the
// next diagonal block up to date, wavefront 0 factors it while the others update the rest.
__device__ __forceinline__ void chol_block(float* H, float* T, float* __restrict__ tinv, int* __restrict__ fail) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto blk = [&](int i, int c) { return H + 32 * i * CH_LD + 32 * c; };
    const int r16 = w & 1, c16 = w >> 1, at16 = (16 * r16 + 4 * (lane >> 4)) * CH_LD + 16 * c16 + (lane & 15);   // a wavefront's 16 x 16 of a block
    int bad = 0;
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
        // beside the pivots of block (s, s): what else row s - 1 takes from the rows i >= s, columns c >= i (G) and c < s (Y)
        if (w == 0) {
            bad |= chol_factor32(blk(s, s), T, lane);
        } else if (s > 0) {
            int n = 0;
            for (int i = s; i < 4; ++i)
                for (int c = 0; c < 4; ++c) {
                    if ((c >= s && c < i) || (i == s && c == s)) continue;
                    if (++n % 3 == w - 1) chol_update32(blk(i, c), blk(s - 1, i), blk(s - 1, c), c == s - 1, lane);   // (Y starts at c = s - 1)
                }
        }
        __syncthreads();
        // row s, the three blocks beside the diagonal, 16 x 16 of each to a wavefront
        {
            float t[8], d[3][8];
            chol_load16(T + 16 * r16, CH_LDT, lane, t);
#pragma unroll
            for (int n = 0; n < 3; ++n) chol_load16(blk(s, n + (n >= s)) + 16 * c16, CH_LD, lane, d[n]);
            __syncthreads();   // (in place)
            v4f o[3];
#pragma unroll
            for (int n = 0; n < 3; ++n) o[n] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
#pragma unroll
                for (int n = 0; n < 3; ++n) o[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[kk], d[n][kk], o[n], 0, 0, 0);
#pragma unroll
            for (int n = 0; n < 3; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) blk(s, n + (n >= s))[at16 + v * CH_LD] = o[n][v];
        }
        __syncthreads();
        // the next diagonal block, 16 x 16 to a wavefront
        if (s < 3) {
            float a[8], b[8];
            chol_load16(blk(s, s + 1) + 16 * r16, CH_LD, lane, a);
            chol_load16(blk(s, s + 1) + 16 * c16, CH_LD, lane, b);
            float* d = blk(s + 1, s + 1) + at16;
            v4f old, o[2];   // (two sums: half the chain)
#pragma unroll
            for (int v = 0; v < 4; ++v) old[v] = d[v * CH_LD];
            o[0] = o[1] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) o[kk & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], b[kk], o[kk & 1], 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) d[v * CH_LD] = old[v] - (o[0][v] + o[1][v]);
            __syncthreads();
        }
    }
    if (bad && tid == 0) atomicAdd(fail, 1);
    // (32 x 32 blocks above the diagonal are not read)
#pragma unroll
    for (int n = 0; n < NB * NB / 4 / 256; ++n) {
        const int e = tid + 256 * n, i = e / (NB / 4), k = 4 * (e % (NB / 4));
        if (k / 32 <= i / 32) *reinterpret_cast<v4f*>(tinv + NB * i + k) = *reinterpret_cast<const v4f*>(H + i * CH_LD + k);
    }
}

// Diagonal block 0.
__global__ __launch_bounds__(256) void dbf_chol_first_kernel(const float* __restrict__ G, int q, float* __restrict__ tinv,
                                                           int* __restrict__ fail) {
    __shared__ __align__(16) uint8_t lds[CH_LDS];
    float* H = reinterpret_cast<float*>(lds);
    const int w = min(q, NB);
#pragma unroll 16
    for (int e = threadIdx.x; e < NB * NB; e += 256) {
        const int i = e / NB, j = e % NB;
        const float v = G[(size_t)min(min(i, j), w - 1) * q + min(max(i, j), w - 1)];
        H[i * CH_LD + j] = (i < w && j < w) ? v : (i == j ? 1.f : 0.f);
    }
    __syncthreads();
    chol_block(H, H + NB * CH_LD, tinv, fail);
}

// Row jb, 32 columns per workgroup: the planes of R_jj^-T [G | Y][jb, :].  Wavefront w makes rows 32 w .. + 31; every load is
// issued before anything waits.  (Columns of the diagonal block itself: Y there is R_jj^-T, the product with the identity.)
__global__ __launch_bounds__(256) void dbf_chol_panel_kernel(const float* __restrict__ G, int q, int jb, const float* __restrict__ tinv,
                                                           uint8_t* __restrict__ planes) {
    __shared__ float Q[NB][33], part[4][32];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j0 = jb * NB, wb = min(NB, q - j0), c0 = 32 * blockIdx.x, n_kb = sg_kblocks(q);
    const bool diag = (c0 / NB) == jb;
    const int rk = tid >> 5, cc = c0 + (tid & 31);
    float qv[16];
    v4f a[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) qv[e] = G[(size_t)(j0 + min(rk + 8 * e, wb - 1)) * q + min(cc, q - 1)];
    // (register e of a[m] is k = 8 m + 4 h + e of row 32 w + l32; k >= 32 (w + 1) is not used)
#pragma unroll
    for (int m = 0; m < 16; ++m) a[m] = *reinterpret_cast<const v4f*>(tinv + (32 * w + l32) * NB + 8 * m + 4 * h);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int k = rk + 8 * e;
        Q[k][tid & 31] = (k >= wb || cc >= q) ? 0.f : diag ? (j0 + k == cc ? 1.f : 0.f) : qv[e];
    }
    __syncthreads();
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b > w) break;
#pragma unroll
        for (int m = 4 * b; m < 4 * b + 4; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m][e], Q[8 * m + 4 * h + e][l32], acc, 0, 0, 0);
    }
    // the largest magnitude of each column: its scale
    float mx = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, fabsf(acc[v]));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (lane < 32) part[w][lane] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(part[0][l32], part[1][l32]), fmaxf(part[2][l32], part[3][l32]));
    const SgScale scale = sg_scale(mx);
    if (tid < 32) reinterpret_cast<float*>(planes + sg_scales_at(2, q, q))[(size_t)jb * sg_lines(q) + c0 + tid] = scale.up;
    // register v of lane (h, l32) is row 8 (v / 4) + 4 h + v % 4; a plane wants rows 8 h .. + 7 of each 16
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = acc[8 * t + e], hi = acc[8 * t + 4 + e];
            const float got = __shfl_xor(h ? lo : hi, 32, 64);
            x[e] = h ? got : lo;
            x[4 + e] = h ? hi : got;
        }
        const int kb = j0 / 16 + 2 * w + t;
        sg_store2(planes + (((size_t)(c0 / NB) * n_kb + kb) * 8 + ((c0 >> 5) & 3)) * SG_FRAG + lane * 16, x, scale);
    }
}

// The products of one chunk for a workgroup of 128 x 128 outputs (dbf_split_gemm.h has the layout of the operands): acc = their sums, scaled.
// 32 k per step, through registers into two LDS buffers.  `meanwhile` runs beside the last step's products.  Ends with a barrier behind the last read of `lds`.
struct CholTile {
    uint8_t frags[2][32 * SG_FRAG];
    float up[256];
};
template <class F>
__device__ __forceinline__ void chol_tile(CholTile& lds, const SgOperand P, const SgOperand Q, v16f (&acc)[2][2], F meanwhile) {
    constexpr int STEPS = NB / 32;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), fi = 2 * (w & 1), fj = 2 * (w >> 1);
    v4f st[8];
    v16f low[2][2];   // the products with a low piece (dbf_split_gemm.h)
    // (an operand's 32 k are 16 KiB in one run: [k / 16][piece][32-block])
    auto fetch = [&](int s) {
#pragma unroll
        for (int n = 0; n < 8; ++n) st[n] = *reinterpret_cast<const v4f*>((n < 4 ? P.frags : Q.frags) + (size_t)s * 16 * SG_FRAG + 4096 * (n & 3) + 16 * tid);
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int n = 0; n < 8; ++n) *reinterpret_cast<v4f*>(&lds.frags[buf][4096 * n + 16 * tid]) = st[n];
    };
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bi][bj][v] = low[bi][bj][v] = 0.f;
    fetch(0);
    const float up = tid < 128 ? P.up[tid] : Q.up[tid - 128];
    stage(0);
    lds.up[tid] = up;
    fetch(1);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        if (s + 1 < STEPS) stage((s + 1) & 1);
        if (s + 2 < STEPS) fetch(s + 2);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 == STEPS) meanwhile();
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const uint8_t* base = &lds.frags[s & 1][8 * sub * SG_FRAG + 16 * lane];
            v8h a[2][2], b[2][2];
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    a[x][p] = *reinterpret_cast<const v8h*>(base + (4 * p + fi + x) * SG_FRAG);
                    b[x][p] = *reinterpret_cast<const v8h*>(base + (16 + 4 * p + fj + x) * SG_FRAG);
                }
#pragma unroll
            for (int p = 1; p >= 0; --p)
#pragma unroll
                for (int q = 1 - p; q >= 0; --q)
#pragma unroll
                    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                        for (int bj = 0; bj < 2; ++bj) {
                            v16f& sum = p + q == 0 ? acc[bi][bj] : low[bi][bj];
                            sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[bi][p], b[bj][q], sum, 0, 0, 0);
                        }
        }
        __syncthreads();
    }
    // (P's scale first, unlike sg_scaled in dbf_split_gemm.h: P is R, whose entries are below the root of one of G's, 2^64)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            const float uq = lds.up[128 + 32 * (fj + bj) + (lane & 31)];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const v4f ur = *reinterpret_cast<const v4f*>(&lds.up[32 * (fi + bi) + 8 * c + 4 * (lane >> 5)]);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[bi][bj][4 * c + e] = fmaf(low[bi][bj][4 * c + e], 1.f / SG_LOW, acc[bi][bj][4 * c + e]) * ur[e] * uq;
            }
        }
    __syncthreads();
}

// Rows i > jb: [G | Y][i, :] -= R[jb, i]^T [R | Y][jb, :], a workgroup per 128 x 128 block.  Workgroup (0, 0) has diagonal block jb + 1: it keeps it in LDS
// and factors it; being the first of the launch it starts with it.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_chol_update_kernel(
    float* __restrict__ G, int q, int jb, const uint8_t* __restrict__ planes, float* __restrict__ tinv_next, int* __restrict__ fail) {
    __shared__ __align__(16) uint8_t lds[CH_LDS > sizeof(CholTile) ? CH_LDS : sizeof(CholTile)];
    const int nblk = gridDim.x, it = jb + 1 + blockIdx.y, jt = (int)((jb + 1 + blockIdx.x) % nblk);
    if (jt > jb && jt < it) return;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), fi = 2 * (w & 1), fj = 2 * (w >> 1);
    const bool factor = blockIdx.x == 0 && blockIdx.y == 0;
    v16f acc[2][2];
    float old[2][2][16];
    // (block row jb is whole: only the last can be short, and it has nothing to update)
    chol_tile(*reinterpret_cast<CholTile*>(lds), sg_operand(planes, 2, q, q, it, jb), sg_operand(planes, 2, q, q, jt, jb), acc, [&]() {
#pragma unroll
                           for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                               for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                                   for (int v = 0; v < 16; ++v) {
                                       const int row = NB * it + 32 * (fi + bi) + 8 * (v >> 2) + 4 * h + (v & 3);
                                       const int col = NB * jt + 32 * (fj + bj) + l32;
                                       old[bi][bj][v] = G[(size_t)min(row, q - 1) * q + min(col, q - 1)];
                                   }
                       });
    float* H = reinterpret_cast<float*>(lds);   // (the tile's last barrier is behind every read of the operands)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = 32 * (fi + bi) + 8 * (v >> 2) + 4 * h + (v & 3), j = 32 * (fj + bj) + l32;
                const int row = NB * it + i, col = NB * jt + j;
                const bool in = row < q && col < q;
                const float val = (jt == jb ? 0.f : old[bi][bj][v]) - acc[bi][bj][v];
                if (factor) H[i * CH_LD + j] = in ? val : (i == j ? 1.f : 0.f);
                else if (in) G[(size_t)row * q + col] = val;
            }
    if (!factor) return;
    __syncthreads();
    chol_block(H, H + NB * CH_LD, tinv_next, fail);
}

// M[j][i] = M[i][j] for i < j: the lower triangle of a symmetric matrix whose upper blocks were computed.
// One workgroup per 32 x 32 block on or above the diagonal, through LDS so that both sides are coalesced.
__global__ __launch_bounds__(256) void dbf_chol_mirror_kernel(float* __restrict__ M, int q) {
    __shared__ float t[32][33];
    const int bi = blockIdx.y, bj = blockIdx.x;
    if (bi > bj) return;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int rr = ty; rr < 32; rr += 8) {
        const int i = 32 * bi + rr, j = 32 * bj + tx;
        t[rr][tx] = (i < q && j < q) ? M[(size_t)i * q + j] : 0.f;
    }
    __syncthreads();
    for (int rr = ty; rr < 32; rr += 8) {
        const int j = 32 * bj + rr, i = 32 * bi + tx;   // writes M[j][i] = t[i - 32 bi][j - 32 bj]
        if (i < q && j < q && i < j) M[(size_t)j * q + i] = t[tx][rr];
    }
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
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 255) || workspace_bytes < w.total)
        return DBF_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint8_t* base = static_cast<uint8_t*>(workspace_dev);
    float* Z = reinterpret_cast<float*>(base + w.Z);
    float* U = static_cast<float*>(U_dev);
    const float* C = static_cast<const float*>(C_dev);
    const int n_rt = dbf_row_tiles(q), n_ct = dbf_col_tiles(r);
    const int vec_r = ((r & 3) == 0 && (reinterpret_cast<uintptr_t>(U) & 15) == 0) ? 1 : 0;  // (Z is 256-byte aligned)

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
    const int rc = dbf_svid(Z, q, r, svid_iters, a_dev, m_dev, bits_dev, base + w.svid, workspace_bytes - w.svid, st);
    if (rc != DBF_OK) return rc;
    hipLaunchKernelGGL(dbf_admm_dual_kernel, dim3(n_ct, n_rt), dim3(256), 0, st, Z, static_cast<const float*>(a_dev),
                       static_cast<const float*>(m_dev),
                       static_cast<const uint8_t*>(bits_dev), q, r, n_ct, vec_r, U);
    if (hipGetLastError() != hipSuccess) return DBF_EHIP;
    return DBF_OK;
}

// ---- forming the constant matrices of the update on the device ---------------------------------
namespace {
struct PrepWorkspace {
    size_t tinv, fail, S, V, total;
    int nblk;
};
inline PrepWorkspace prep_workspace(int p, int q, int r) {
    PrepWorkspace w;
    w.nblk = (q + NB - 1) / NB;
    size_t off = 0;
    w.tinv = off;  off = up256(off + 4 * (size_t)w.nblk * NB * NB);
    w.fail = off;  off = up256(off + 256);
    w.S = off;     off = up256(off + sg_plane_bytes(1, p, q));   // planes of the signs
    // planes of the other operand of the three large contractions in turn: the scaled signs, b . W, [R | Y]
    size_t v = sg_plane_bytes(2, p, q);
    v = v < sg_plane_bytes(2, p, r) ? sg_plane_bytes(2, p, r) : v;
    v = v < sg_plane_bytes(2, q, q) ? sg_plane_bytes(2, q, q) : v;
    w.V = off;     off = up256(off + v);
    w.total = off;
    return w;
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
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 255) || workspace_bytes < w.total)
        return DBF_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint8_t* base = static_cast<uint8_t*>(workspace_dev);
    float* tinv = reinterpret_cast<float*>(base + w.tinv);
    int* fail = not_positive_definite_dev ? not_positive_definite_dev : reinterpret_cast<int*>(base + w.fail);
    float* G = static_cast<float*>(Minv_dev);  // G, then its factor, live in the output until the last contraction
    const uint8_t* bits = static_cast<const uint8_t*>(bits_dev);
    const float* m2 = static_cast<const float*>(m2_dev);
    const float* b = static_cast<const float*>(b_dev);
    const int n_ct = dbf_col_tiles(p);

    uint8_t *S = base + w.S, *V = base + w.V;
    // G = B^T B + rho I with B[l][j] = b_l S[j][l] m2_j: the signs against the signs times b^2, m2 by output row and column in
    // the epilogue.  Upper blocks only.
    hipLaunchKernelGGL(dbf_split_signs_kernel, sg_plane_grid(p, q), dim3(256), 0, st, bits, n_ct, p, q, b, S, V, fail);
    {
        SplitGemmArgs g = {};
        g.P = S;  g.Q = V;  g.out = G;  g.ldo = q;  g.M = q;  g.N = q;  g.K = p;
        g.rs = m2;  g.cs = m2;  g.diag = rho;  g.upper = 1;
        launch_split_gemm<1>(g, st);
    }
    // C = B^T W: the signs against b . W
    {
        hipLaunchKernelGGL(dbf_split_dense_kernel, sg_plane_grid(p, r), dim3(256), 0, st, static_cast<const float*>(W_dev), (size_t)r, p, r, b,
                           V);
        SplitGemmArgs g = {};
        g.P = S;  g.Q = V;  g.out = static_cast<float*>(C_dev);  g.ldo = r;  g.M = q;  g.N = r;  g.K = p;
        g.rs = m2;
        launch_split_gemm<1>(g, st);
    }
    // [G | I] -> [R | Y], the planes of Y (and of R, row by row) in V
    hipLaunchKernelGGL(dbf_chol_first_kernel, dim3(1), dim3(256), 0, st, G, q, tinv, fail);
    for (int jb = 0; jb < w.nblk; ++jb) {
        const bool last = jb + 1 == w.nblk;
        float* tj = tinv + (size_t)jb * NB * NB;
        hipLaunchKernelGGL(dbf_chol_panel_kernel, dim3(4 * w.nblk), dim3(256), 0, st, G, q, jb, tj, V);
        if (!last)
            hipLaunchKernelGGL(dbf_chol_update_kernel, dim3(w.nblk, w.nblk - 1 - jb), dim3(256), 0, st, G, q, jb, V, tj + NB * NB,
                               fail);
    }
    // G^-1 = Y^T Y (overwrites G): upper blocks, the sums starting where both operands can be non-zero,
    // then the mirror image
    {
        SplitGemmArgs g = {};
        g.P = V;  g.Q = V;  g.out = G;  g.ldo = q;  g.M = q;  g.N = q;  g.K = q;
        g.upper = 1;  g.ktri = 1;
        launch_split_gemm<2>(g, st);
        hipLaunchKernelGGL(dbf_chol_mirror_kernel, dim3((q + 31) / 32, (q + 31) / 32), dim3(256), 0, st, G, q);
    }
    if (hipGetLastError() != hipSuccess) return DBF_EHIP;
    return DBF_OK;
}
