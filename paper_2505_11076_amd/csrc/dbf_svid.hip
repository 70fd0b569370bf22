// SVID projection (paper, section 3.2): SVID(Z) = a . Sign(Z) . m^T, where a m^T is the rank-one
// decomposition of |Z| obtained by power iteration.  It is the projection step of the ADMM iteration
// that computes the factorisation; here it produces the sign matrix directly in the packed device
// tile layout of this library (what a layer stores), and the two scale vectors in fp32.
//
// Readings of what the paper leaves open (the same as the CPU oracle's): Sign(0) = +1; the iteration
// starts from the constant unit vector and runs `iters` rounds of
//     u <- |Z| v / ||.||,   v <- |Z|^T u,   sigma <- ||v||,   v <- v / sigma;      a = sigma u,  m = v.
//
// Everything is bound by reading Z (fp32, rows x cols, row major).  A round needs u = |Z| v before any of
// v' = |Z|^T u -- but only row by row: the term of row i in v' needs u_i alone, and u_i needs row i alone.  So
// ONE pass over Z does a whole round (dbf_svid_round_kernel): a workgroup holds batches of whole rows in registers,
// forms their dots with v, and adds the rows, weighted by those dots, into its partial column sums; a second, small
// launch sums the partial sums over the workgroups.  Rows of up to 4096 columns are dealt to workgroups in groups of the
// eight that share a byte of the sign tiles, so that the first pass writes the signs as well.  Rows too long for one pass (more than
// 24576 columns, 12288 where they cannot be read in 16-byte pieces) take two passes per round (row dots, column dots) and the same
// reduce launch.  In both forms the normalisations are not passes of their own.  The iterate is kept unnormalised (u_raw =
// |Z| v, v_raw = |Z|^T u_raw; the length of u cancels in v / ||v||), the column reduction leaves the squared length of v_raw
// as one partial sum per workgroup, and the next row pass scales by 1 / ||v_raw|| on the fly; the last kernel forms
// m = v_raw / ||v_raw|| and a = sigma u = u_raw ||v_raw|| / ||u_raw||^2.  All reductions have a fixed
// order, so the result does not depend on scheduling:
//   row dots     one wavefront per row, 16-byte loads, butterfly reduction;
//   column dots  workgroup = 256 columns x 64 rows (4 row lanes x 16 rows, combined in LDS in lane
//                order), partial sums per 64-row chunk, then summed over the chunks in a fixed order;
//   norms        partial sums of squares per 32 or 64 columns (v) or per thread stride (u), combined in a fixed tree;
//   signs        one workgroup per 128 x 64 tile, a thread per four bytes of the tile.
// And where Z has room in the registers of the whole device and the rounds are several, one launch does all of them (dbf_svid_held_kernel).
#include "dbf_kernels.h"
#include "dbf_wave.h"

#include <climits>
#include <type_traits>

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int COL_CHUNK_ROWS = 64;   // rows per partial sum of the column pass
constexpr int COL_BLOCK = 256;       // columns per workgroup of the column pass
constexpr int ROUND_WGS = 256;       // workgroups of the one-pass round: one per compute unit

__device__ inline float wave_sum_f(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of n partial sums in a fixed order (lane-strided, then butterfly); every lane gets the result.
__device__ inline float wave_total(const float* __restrict__ part, int n, int lane) {
    float s = 0.f;
    for (int i = lane; i < n; i += 64) s += part[i];
    return wave_sum_f(s);
}

// u_raw[i] = (sum_j |Z[i][j]| v_raw[j]) / ||v_raw||, with ||v_raw||^2 = sum of ss_part[0 .. n_ss).
// FIRST: the start vector, v = 1 / sqrt(cols) everywhere (v_raw and ss_part are not read).
template <bool FIRST>
__global__ __launch_bounds__(256) void dbf_svid_row_dots_kernel(const float* __restrict__ Z, int rows, int cols,
                                                               const float* __restrict__ v,
                                                               const float* __restrict__ ss_part, int n_ss,
                                                               float* __restrict__ u, int vec_ok) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float* z = Z + (size_t)row * cols;
    float s = 0.f;
    if (vec_ok) {
        for (int c = 4 * lane; c < cols; c += 256) {
            const v4f a = *reinterpret_cast<const v4f*>(z + c);
            if (FIRST) {
                s += (fabsf(a.x) + fabsf(a.y)) + (fabsf(a.z) + fabsf(a.w));
            } else {
                const v4f b = *reinterpret_cast<const v4f*>(v + c);
                s += fabsf(a.x) * b.x + fabsf(a.y) * b.y + fabsf(a.z) * b.z + fabsf(a.w) * b.w;
            }
        }
    } else {
        for (int c = lane; c < cols; c += 64) s += FIRST ? fabsf(z[c]) : fabsf(z[c]) * v[c];
    }
    s = wave_sum_f(s);
    float inv;
    if (FIRST) {
        inv = 1.0f / sqrtf((float)cols);
    } else {
        const float nrm = sqrtf(wave_total(ss_part, n_ss, lane));
        inv = nrm > 0.f ? 1.0f / nrm : 0.f;
    }
    if (lane == 0) u[row] = s * inv;
}

// The sums of N values (8 or 4) over the wavefront, N / 4 to a lane: entry i of the result, in every lane of the row rho of 16 lanes, is the
// sum of value i + N / 4 (2 (rho / 2) + rho % 2).  Halves and rows of lanes change places, so that every addition serves two values:
// 28 instructions for eight values, where a reduction each takes 150.
template <int N>
__device__ __forceinline__ void wave_sums(const float (&x)[N], float (&sum)[N / 4]) {
    float s[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x[i]), __builtin_bit_cast(unsigned, x[i + N / 2]), false, false);
        s[i] = __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);   // (lanes 0-31: value i, 32-63: i + N / 2)
    }
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, s[i]), __builtin_bit_cast(unsigned, s[i + N / 4]), false, false);
        sum[i] = dbf_row16_sum_f(__builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]));
    }
}

// One round in one pass, a workgroup of W wavefronts per compute unit.  Rows come in groups of eight, group 16 q + r being the rows
// 128 q + 16 s + r, s = 0 .. 7 (one byte column of a sign tile); a workgroup has `groups_per_wg` consecutive groups and takes RB rows
// of one at a time.  Thread t holds, of every row of the batch, the CPL float4s at columns 4 t + 256 W k (k < CPL), so a
// wavefront's load of a row segment is 1 KiB contiguous.  Per batch: the next batch's loads are issued first (register double
// buffer), then every wavefront forms its part of the RB row dots (register-to-register reduction) and leaves it in LDS; the
// parts are summed by RB rows of 16 lanes, scaled by 1 / ||v_raw|| -> u_raw, and every thread adds |z| u_raw of its columns
// into its CPL float4 accumulators.  At the end the accumulators are the workgroup's partial column sums: partial[workgroup][column].
// FIRST: v = 1 / sqrt(cols) everywhere, v_raw is not read; and with CPL == 1 the signs are written.  All sums have a fixed order.
// What bounds it: at 4096 x 4096 reading Z from the last-level cache, 67 MB in two batches per workgroup.
template <int W, int CPL, bool FIRST, bool VEC>
__global__ __launch_bounds__(64 * W) void dbf_svid_round_kernel(const float* __restrict__ Z, int rows, int cols,
                                                              const float* __restrict__ v,
                                                              const float* __restrict__ ss_part, int n_ss,
                                                              float* __restrict__ u, float* __restrict__ partial,
                                                              int groups_per_wg, int n_groups, uint8_t* __restrict__ bits, int n_ct) {
    constexpr int RB = CPL == 1 ? 8 : CPL == 2 ? 4 : CPL == 3 ? 2 : 1;  // rows per batch: about 32 registers per buffer
    constexpr int NB = 8 / RB;                                         // batches per group
    constexpr bool SIGNS = FIRST && CPL == 1 && VEC;
    __shared__ float dots[2][RB][16];
    __shared__ __align__(16) float us[2][RB];
    __shared__ float inv_s;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int b_lo = blockIdx.x * groups_per_wg * NB, b_hi = min(n_groups, (int)(blockIdx.x + 1) * groups_per_wg) * NB;
    v4f vv[CPL], acc[CPL];
    // element e of the thread's k-th float4: column 4 tid + 256 W k + e, or, where rows cannot be read in 16-byte pieces, tid + 64 W (4 k + e)
    auto col_of = [&](int k, int e) { return VEC ? 4 * tid + 256 * W * k + e : tid + 64 * W * (4 * k + e); };
    auto live = [&](int k, int e) { return col_of(k, VEC ? 0 : e) < cols; };   // (VEC: cols is a multiple of 4)
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        vv[k] = (v4f){0.f, 0.f, 0.f, 0.f};
        if (!FIRST && VEC && live(k, 0)) vv[k] = *reinterpret_cast<const v4f*>(v + col_of(k, 0));
        if (!FIRST && !VEC) {
#pragma unroll
            for (int e = 0; e < 4; ++e) vv[k][e] = live(k, e) ? v[col_of(k, e)] : 0.f;
        }
        acc[k] = (v4f){0.f, 0.f, 0.f, 0.f};
    }
    // row i of batch b
    auto row_of = [&](int b, int i) {
        const int g = b / NB;
        return 128 * (g >> 4) + 16 * (RB * (b % NB) + i) + (g & 15);
    };
    // (no branch around a load: rows beyond the matrix are read as its last row and get weight zero below,
    //  columns beyond the matrix are read as the row's first and get v = 0 / are masked, so that all loads of a
    //  batch are in flight together)
    auto load_batch = [&](v4f (&z)[RB][CPL], int b) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int row = min(row_of(b, r), rows - 1);
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const float* zr = Z + (size_t)row * cols;
                if (VEC) {
                    z[r][k] = *reinterpret_cast<const v4f*>(zr + (live(k, 0) ? col_of(k, 0) : 0));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) z[r][k][e] = zr[live(k, e) ? col_of(k, e) : 0];
                }
            }
        }
    };
    auto abs4 = [](v4f a) { return (v4f){fabsf(a.x), fabsf(a.y), fabsf(a.z), fabsf(a.w)}; };
    v4f za[RB][CPL], zb[RB][CPL];
    load_batch(za, b_lo);
    load_batch(zb, min(b_lo + 1, b_hi - 1));
    if (tid < 2 * RB * 16) (&dots[0][0][0])[tid] = 0.f;   // (the parts of wavefronts that a narrower workgroup does not have)
    if (w == 0) {
        float inv;
        if (FIRST) {
            inv = 1.0f / sqrtf((float)cols);
        } else {
            const float nrm = sqrtf(wave_total(ss_part, n_ss, lane));
            inv = nrm > 0.f ? 1.0f / nrm : 0.f;
        }
        if (lane == 0) inv_s = inv;
    }
    __syncthreads();
    int buf = 0;
    // (two batches per trip, so that the two register buffers keep their names)
    auto process = [&](v4f (&z)[RB][CPL], int b) {
        float part[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            float sdot = 0.f;
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const v4f a = abs4(z[r][k]);
                if (FIRST) sdot += ((live(k, 0) ? a.x : 0.f) + (live(k, 1) ? a.y : 0.f)) + ((live(k, 2) ? a.z : 0.f) + (live(k, 3) ? a.w : 0.f));
                else sdot += a.x * vv[k].x + a.y * vv[k].y + a.z * vv[k].z + a.w * vv[k].w;
            }
            part[r] = RB >= 4 ? sdot : dbf_wave_sum_f(sdot);
        }
        if constexpr (RB >= 4) {
            float sum[RB / 4];
            wave_sums<RB>(part, sum);
            if ((lane & 15) == 0) {
#pragma unroll
                for (int i = 0; i < RB / 4; ++i) dots[buf][i + RB / 4 * (lane >> 4)][w] = sum[i];
            }
        } else if (lane == 0) {
#pragma unroll
            for (int r = 0; r < RB; ++r) dots[buf][r][w] = part[r];
        }
        if (SIGNS) {
            const int g = b, col = 4 * tid;
            unsigned out = 0;
#pragma unroll
            for (int s = 0; s < RB; ++s) {
                const v4f a = z[s][0];
                const unsigned four = (unsigned)(a.x >= 0.f) | (unsigned)(a.y >= 0.f) << 8 | (unsigned)(a.z >= 0.f) << 16 | (unsigned)(a.w >= 0.f) << 24;
                out |= (live(0, 0) && row_of(b, s) < rows) ? four << s : 0u;
            }
            if (col < n_ct * DBF_TILE_COLS)
                *reinterpret_cast<unsigned*>(bits + ((size_t)(g >> 4) * n_ct + (col >> 6)) * DBF_TILE_BYTES + 256 * ((col >> 4) & 3) +
                                             16 * (g & 15) + (col & 15)) = out;
        }
        __syncthreads();
        if (tid < 16 * RB) {
            const float tot = dbf_row16_sum_f((&dots[buf][0][0])[tid]);
            if ((tid & 15) == 0) {
                const int row = row_of(b, tid >> 4);
                const float ur = row < rows ? tot * inv_s : 0.f;
                us[buf][tid >> 4] = ur;
                if (row < rows) u[row] = ur;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const float ur = us[buf][r];
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const v4f a = abs4(z[r][k]);
                acc[k].x += a.x * ur;  acc[k].y += a.y * ur;  acc[k].z += a.z * ur;  acc[k].w += a.w * ur;  // (dead columns: never stored)
            }
        }
        buf ^= 1;
    };
    for (int b = b_lo; b < b_hi; b += 2) {
        process(za, b);
        if (b + 2 < b_hi) load_batch(za, b + 2);
        if (b + 1 < b_hi) {
            process(zb, b + 1);
            if (b + 3 < b_hi) load_batch(zb, b + 3);
        }
    }
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        float* out = partial + (size_t)blockIdx.x * cols;
        if (VEC) {
            if (live(k, 0)) *reinterpret_cast<v4f*>(out + col_of(k, 0)) = acc[k];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (live(k, e)) out[col_of(k, e)] = acc[k][e];
        }
    }
}

// partial[chunk][j] = sum over the chunk's rows i of |Z[i][j]| u[i]
__global__ __launch_bounds__(256) void dbf_svid_col_dots_kernel(const float* __restrict__ Z, int rows, int cols,
                                                               const float* __restrict__ u,
                                                               float* __restrict__ partial) {
    __shared__ float part[4][COL_BLOCK];
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;       // column quad, row lane
    const int col = blockIdx.x * COL_BLOCK + 4 * cl;
    const int row0 = blockIdx.y * COL_CHUNK_ROWS;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    const bool vec = (cols & 3) == 0 && col + 4 <= cols;
    if (vec) {
        // rows beyond the matrix are read as the last row with weight zero: no branch in the loop, so
        // the loads of several rounds are in flight together
        static_assert(COL_CHUNK_ROWS % 4 == 0, "four row lanes share a chunk evenly");
#pragma unroll
        for (int ii = 0; ii < COL_CHUNK_ROWS / 4; ++ii) {
            const int row = row0 + rl + 4 * ii;
            const int rc = min(row, rows - 1);
            const float w = row < rows ? u[rc] : 0.f;
            const v4f a = *reinterpret_cast<const v4f*>(Z + (size_t)rc * cols + col);
            s[0] += fabsf(a.x) * w;  s[1] += fabsf(a.y) * w;  s[2] += fabsf(a.z) * w;  s[3] += fabsf(a.w) * w;
        }
    } else {
        for (int i = rl; i < COL_CHUNK_ROWS; i += 4) {
            const int row = row0 + i;
            if (row >= rows) break;
            const float w = u[row];
            const float* z = Z + (size_t)row * cols + col;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (col + q < cols) s[q] += fabsf(z[q]) * w;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[rl][4 * cl + q] = s[q];
    __syncthreads();
    const int c = threadIdx.x;
    if (blockIdx.x * COL_BLOCK + c < cols)
        partial[(size_t)blockIdx.y * cols + blockIdx.x * COL_BLOCK + c] = ((part[0][c] + part[1][c]) + part[2][c]) + part[3][c];
}

// v_raw[j] = sum over chunks of partial[chunk][j]: S interleaved running sums (chunks c = 0, S, 2 S, ... in the first, and so on), added up in
// order; and ss_part[workgroup] = sum of v_raw[j]^2 over the workgroup's COLS columns (butterfly order).  Workgroup = COLS columns x S running
// sums, 256 chunks in one memory round trip (with four sums and a load at a time 64 chunks took 6.6 us, so 4).  32 columns a workgroup while that is
// one workgroup per compute unit: calls of 8 rounds, 64 / 32 columns, 1024 x 1024 54.0 / 49.9 us, 4096 x 4096 136.1 / 134.4; 4 rounds of
// 4096 x 11008 163.5 / 167.8.  Summed in 64 bits: up to 256 partial sums in 32 bits, against
// 64 of the two passes, left m 20 % further from the exact factor (7.7e-8 against 6.5e-8 at 4096 x 4096, means of 12 inputs; 4.7e-8 with
// these sums, 3.9e-8 with those of the last kernel too).  The 64-bit sums of both cost a call of 8 rounds 2.5 us of 154.
constexpr int REDUCE_THREADS = 1024;
inline int reduce_cols(int cols) { return cols <= 8192 ? 32 : 64; }
template <int COLS>
__global__ __launch_bounds__(REDUCE_THREADS) void dbf_svid_col_reduce_kernel(const float* __restrict__ partial, int chunks, int cols,
                                                               float* __restrict__ v, float* __restrict__ ss_part) {
    constexpr int S = REDUCE_THREADS / COLS, LOADS = 256 / S, H = 64 / COLS;
    __shared__ double part[S][COLS];
    const int c = threadIdx.x % COLS, q = threadIdx.x / COLS;
    const int j = blockIdx.x * COLS + c, jc = min(j, cols - 1);
    double s = 0.;
    for (int c0 = q; c0 < chunks; c0 += LOADS * S) {
        float p[LOADS];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) p[i] = partial[(size_t)min(c0 + S * i, chunks - 1) * cols + jc];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) s += (double)(c0 + S * i < chunks ? p[i] : 0.f);
    }
    part[q][c] = s;
    __syncthreads();
    if (threadIdx.x < 64) {   // (COLS = 32: half of the running sums to each half of the wavefront)
        double sum = part[q][c];
#pragma unroll
        for (int i = 1; i < S / H; ++i) sum += part[q + H * i][c];
        if (H == 2) sum += __shfl_xor(sum, 32, 64);
        const float vj = (float)sum;
        if (j < cols && q == 0) v[j] = vj;
        const float ss = wave_sum_f(j < cols && q == 0 ? vj * vj : 0.f);
        if (threadIdx.x == 0) ss_part[blockIdx.x] = ss;
    }
}
template <class... A>
void launch_reduce(int cols, hipStream_t st, A... a) {
    const int per = reduce_cols(cols);
    hipLaunchKernelGGL(per == 32 ? dbf_svid_col_reduce_kernel<32> : dbf_svid_col_reduce_kernel<64>, dim3((cols + per - 1) / per), dim3(REDUCE_THREADS),
                       0, st, a...);
}

// The two factors from the unnormalised iterate: m = v_raw / ||v_raw|| (in place) and
// a = sigma u = u_raw ||v_raw|| / ||u_raw||^2 (sigma = ||v_raw|| / ||u_raw||, u = u_raw / ||u_raw||).
// Every workgroup forms both lengths itself, in 64 bits and the same fixed order, and then writes its 1024 entries of each.  Bound by its chain of
// latencies: one memory round trip for both lengths, then sixteen partial sums of each from LDS.
constexpr int FINISH = 1024;
__global__ __launch_bounds__(FINISH) void dbf_svid_finish_kernel(const float* __restrict__ u_raw, int rows,
                                                             const float* __restrict__ ss_part, int n_ss,
                                                             float* __restrict__ m, int cols, float* __restrict__ a) {
    __shared__ double part[2][FINISH / 64];
    const int tid = threadIdx.x, lane = tid & 63, i = blockIdx.x * FINISH + tid;
    const float ui = u_raw[min(i, rows - 1)], mi = m[min(i, cols - 1)];
    double s[2] = {0., 0.};
    for (int j0 = tid; j0 < rows; j0 += 4 * FINISH) {
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = u_raw[min(j0 + FINISH * e, rows - 1)];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[0] += j0 + FINISH * e < rows ? (double)p[e] * (double)p[e] : 0.;
    }
    for (int j = tid; j < n_ss; j += FINISH) s[1] += (double)ss_part[j];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s[k] += __shfl_xor(s[k], off, 64);
        if (lane == 0) part[k][tid >> 6] = s[k];
    }
    __syncthreads();
    double ssu = part[0][0], ssv = part[1][0];
#pragma unroll
    for (int w = 1; w < FINISH / 64; ++w) {
        ssu += part[0][w];
        ssv += part[1][w];
    }
    const double nv = sqrt(ssv);
    if (i < rows) a[i] = ssu > 0. ? (float)(ui * (nv / ssu)) : 0.f;
    if (i < cols && nv > 0.) m[i] = (float)(mi / nv);
}

// Sign(Z) into the tile layout: tile = 128 rows x 64 columns, byte 256 g + 16 r + j, bit s = sign of
// (row 16 s + r, column 16 g + j), a set bit meaning +1.  Thread t makes bytes 4t .. 4t+3.
__global__ __launch_bounds__(256) void dbf_svid_signs_kernel(const float* __restrict__ Z, int rows, int cols, int n_ct,
                                                            uint8_t* __restrict__ bits) {
    const int t = threadIdx.x;
    const int g = t >> 6, r = (t >> 2) & 15, j0 = 4 * (t & 3);
    const int col = blockIdx.x * DBF_TILE_COLS + 16 * g + j0;
    const bool vec = (cols & 3) == 0 && col + 4 <= cols;
    unsigned out = 0;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int row = blockIdx.y * DBF_TILE_ROWS + 16 * s + r;
        if (row >= rows) continue;
        const float* z = Z + (size_t)row * cols + col;
        if (vec) {
            const v4f a = *reinterpret_cast<const v4f*>(z);
            out |= (unsigned)(a.x >= 0.f) << s;
            out |= (unsigned)(a.y >= 0.f) << (8 + s);
            out |= (unsigned)(a.z >= 0.f) << (16 + s);
            out |= (unsigned)(a.w >= 0.f) << (24 + s);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (col + q < cols) out |= (unsigned)(z[q] >= 0.f) << (8 * q + s);
        }
    }
    reinterpret_cast<unsigned*>(bits + ((size_t)blockIdx.y * n_ct + blockIdx.x) * DBF_TILE_BYTES)[t] = out;
}

// ---- all rounds in one launch -------------------------------------------------------------------------------------------
// Z held in registers from round to round: 256 compute units have 128 MB of them.  The rows are cut into parts, G groups of eight rows each (the groups of
// the one-pass round), a part to a workgroup of 512 threads, one workgroup to a compute unit.  A round: every workgroup forms its rows' dots with v and its
// partial column sums, as there, and writes the sums to memory; each then adds up some columns of all parts, in 64 bits, and publishes
// their v; when it has every column, a workgroup goes on to the next round.
// What passes between workgroups is written through to memory and read from there (agent scope).  All of it is sums of magnitudes, so the sign is free to tell
// a round from the one before: words of round i (from 1) have the sign i % 2, all are +0 to begin with, and a word is written again only
// when everyone has read it (who writes sums of round i + 1 has all of v of round i, which nobody publishes without all the sums of round i; who publishes v of
// round i + 1 has everyone's sums of that round, which nobody forms without v of round i).  So a reader polls the values themselves, and a step from
// workgroup to workgroup is one way to memory and one back.  (With a flag behind the values: 13.6 us a round of 4096 x 4096.)
// Who is there: a workgroup takes a ticket and clears its words, and goes on when all have; the last ticket closes the door.  If others keep the device busy, the first one closes it:
// workgroups that come later leave at once, and those inside share out the parts among them, reading Z anew for each part and round.  So
// nobody waits for a workgroup that is not running, and the sums are the same, bit for bit, whoever made them: their order is that of the parts.
// When: a part of another workgroup takes 1.5 us and its bytes at 75 GB/s, each round.  The door stays open until that, for those inside now, would have been
// done (HELD_DOOR_US at most, twice that in all), and a fourth of it from when the last one came in, for the others may be right behind: unless they come
// one by one, the call takes about twice what it would have with the right choice at worst.  4096 x 4096, 8 rounds, with place for 8 at first and for
// all after 300 us: closed after 50 us 1635 us, so 405, a launch a round 451; with place for 64 throughout 325, 435, 243.  (6 rounds with 1 / 4 / 16 / 64 / 128 / 255
// inside 9980 / 2270 / 600 / 189 / 140 / 144 us, with all 70.)
// What bounds it: those steps, two a round.  At 4096 x 4096 7.7 us a round: 1.3 of arithmetic, two
// steps of 2 to 2.5, the adding up; 24 us besides, 14 of them the one read of Z.  (A launch a round: 13.9 for the read from the last-level cache, 4.1 for the
// reduction.)
constexpr int HELD_THREADS = 512, HELD_WAVES = HELD_THREADS / 64;
constexpr int HELD_PARTS = 256;
constexpr unsigned HELD_CLOSED = 0x80000000u;
constexpr int HELD_DOOR_US = 100000;                // (twice this is less than HELD_SPINS polls)
// Polls of a wait: seconds.  A wait this long is a mistake; it ends, and what it waited for is no number from there on: in all that comes of it, in this
// workgroup and in those that read its sums.  Every entry of the product a m^T is then no number, or right.
constexpr int HELD_SPINS = 1 << 21;
struct HeldSync {                                   // cleared before the launch
    unsigned state, inside, cleared, pad[61];
};
struct HeldArgs {
    const float* Z;
    float *u, *partial, *a, *m;
    HeldSync* sync;
    float* v;                                       // [cols]: v_raw as published
    double* ss;                                     // [part]: squared length of its part of u
    uint8_t* bits;
    int rows, cols, iters, n_parts, n_ct;
    int lanes;                                      // a workgroup adds up 4 << lanes columns at a time
    unsigned share_ticks;                           // of the constant clock, 100 MHz: what one part takes those who are without it, all rounds
    int door_spins, spins;                          // HELD_SPINS: of the wait for all to be in, of the others
    int door;                                       // tickets (n_parts, or fewer in a test: the others are outside)
};
template <class T>
__device__ __forceinline__ T held_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T>
__device__ __forceinline__ void held_store(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// 16 bytes, written through to memory and read from there (the policy of an agent-scope access)
constexpr int HELD_MEMORY = 16;   // sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t held_buffer(const void* p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)std::min(bytes, (size_t)0x7fffffff), 0x00020000);
}
__device__ __forceinline__ v4f held_load4(__amdgpu_buffer_rsrc_t b, unsigned at) {
    return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, HELD_MEMORY));
}
__device__ __forceinline__ void held_store4(__amdgpu_buffer_rsrc_t b, unsigned at, v4f v) {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), b, at, 0, HELD_MEMORY);
}

__global__ __launch_bounds__(256) void dbf_svid_clear_kernel(unsigned long long* __restrict__ words, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) words[i] = 0;
}

// v plus what other lanes hold of it: all whose number is the same modulo 2^LANES, register to register.
template <int CTRL>
__device__ __forceinline__ double held_dpp(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    return __builtin_bit_cast(double, (unsigned long long)(unsigned)dbf_dpp_move<CTRL>((int)b) | (unsigned long long)(unsigned)dbf_dpp_move<CTRL>((int)(b >> 32)) << 32);
}
template <int LANES>
__device__ __forceinline__ double held_sum(double v) {
    if (LANES <= 3) v += held_dpp<0x128>(v);   // row_ror:8
    if (LANES <= 2) v += held_dpp<0x124>(v);   // row_ror:4
    auto add = [](auto lo, auto hi) {
        return __builtin_bit_cast(double, (unsigned)lo[0] | (unsigned long long)(unsigned)hi[0] << 32) +
               __builtin_bit_cast(double, (unsigned)lo[1] | (unsigned long long)(unsigned)hi[1] << 32);
    };
    unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    v = add(__builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false), __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false));
    b = __builtin_bit_cast(unsigned long long, v);
    return add(__builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false), __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false));
}

template <int CPL, int G>
__global__ __launch_bounds__(HELD_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_svid_held_kernel(const HeldArgs A) {
    __shared__ float dots[8 * G][HELD_WAVES];
    __shared__ float us[8 * G];
    __shared__ float lengths[HELD_WAVES];
    __shared__ double sums[HELD_WAVES][64], total[2];
    __shared__ int enter[2], any_lost, spins;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = A.rows, cols = A.cols, n_parts = A.n_parts;
    HeldSync* const sync = A.sync;
    v4f z[8 * G][CPL], v[CPL], acc[CPL];
    auto col_of = [&](int k) { return 4 * tid + 4 * HELD_THREADS * k; };
    auto live = [&](int k) { return col_of(k) < cols; };   // (cols is a multiple of 4)
    auto row_of = [&](int part, int r) {
        const int g = part * G + (r >> 3);
        return 128 * (g >> 4) + 16 * (r & 7) + (g & 15);
    };
    auto load_part = [&](int part) {   // (rows and columns beyond the matrix: others in their place, no branch around a load)
#pragma unroll
        for (int r = 0; r < 8 * G; ++r) {
            const float* zr = A.Z + (size_t)min(row_of(part, r), rows - 1) * cols;
#pragma unroll
            for (int k = 0; k < CPL; ++k) z[r][k] = *reinterpret_cast<const v4f*>(zr + (live(k) ? col_of(k) : 0));
        }
    };
    const int chunk_cols = 4 << A.lanes, n_chunks = (cols + chunk_cols - 1) / chunk_cols;
    const auto partial_of = [&](int part) { return held_buffer(A.partial + (size_t)part * cols, 4 * (size_t)cols); };
    const auto v_buffer = held_buffer(A.v, 4 * (size_t)cols);
    bool lost = false;   // (a wait has not ended)
    // One wavefront clears a part's words and those of every step-th chunk from there on, and when they are in memory and `times` that many have come from
    // everyone inside, it has the number of these, or -1 if they have not come in time; 0 if the door was closed before (nothing may be touched then).
    auto clear = [&](int part, int step) {
        const v4f zero = {0.f, 0.f, 0.f, 0.f};
        for (int col = 4 * lane; col < cols; col += 256) held_store4(partial_of(part), 4 * (unsigned)col, zero);
        for (int chunk = part; chunk < n_chunks; chunk += step)
            if (4 * lane < chunk_cols) held_store4(v_buffer, 4 * (unsigned)(chunk * chunk_cols + 4 * lane), zero);   // (nothing beyond the last column)
        if (lane == 0) held_store(reinterpret_cast<unsigned long long*>(A.ss + part), 0ull);
    };
    auto all_cleared = [&](int ticket, int times) {
        __builtin_amdgcn_s_waitcnt(0);
        int n = 0;
        if (lane == 0) {
            auto close = [&] {
                const unsigned old = __hip_atomic_fetch_or(&sync->state, HELD_CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (!(old & HELD_CLOSED)) held_store(&sync->inside, std::min(old, (unsigned)A.door));
            };
            __hip_atomic_fetch_add(&sync->cleared, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (ticket == A.door - 1) close();
            const unsigned long long t0 = wall_clock64();
            unsigned long long last = t0;   // when someone came in, and how many that made
            unsigned seen = 0;
            bool all = false;
            for (int spin = 0; spin < A.door_spins && !all; ++spin) {
                n = (int)held_load(&sync->inside);
                all = n > 0 && held_load(&sync->cleared) >= (unsigned)(n * times);
                if (n == 0 && ticket == 0 && wall_clock64() - t0 >= A.share_ticks) {   // (not before: a load more a poll)
                    const unsigned in = held_load(&sync->state) & ~HELD_CLOSED, share = std::min(A.share_ticks * ((n_parts + in - 1) / in), 100u * HELD_DOOR_US);
                    const unsigned long long now = wall_clock64();
                    if (in != seen) last = now;
                    seen = in;
                    if ((now - t0 >= share && now - last >= share / 4) || now - t0 >= 200u * HELD_DOOR_US) close();
                }
            }
            if (!all) n = -1;
        }
        return __builtin_amdgcn_readfirstlane(n);
    };
    if (w == 0) {   // (before its loads of Z, or every answer would come behind them)
        int mine = 0, n = 0;
        if (lane == 0) mine = (int)__hip_atomic_fetch_add(&sync->state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mine = __builtin_amdgcn_readfirstlane(mine);
        if ((unsigned)mine < (unsigned)A.door) {   // (HELD_CLOSED is the sign)
            clear(blockIdx.x, n_parts);
            n = all_cleared(mine, 1);
            if (n > 0 && n < n_parts) {   // the parts and columns of those outside
                for (int part = mine; part < n_parts; part += n) clear(part, n);
                n = all_cleared(mine, 2);
            }
        }
        if (lane == 0) {
            enter[0] = mine;
            enter[1] = n;
            any_lost = 0;
            spins = A.spins;
        }
    }
    load_part(blockIdx.x);
    __syncthreads();
    const int inside = __builtin_amdgcn_readfirstlane(enter[1]);
    if (inside == 0) return;   // (too late)
    if (inside < 0) {          // (the others, if they go on, do without its sums: nothing of theirs is a number either)
        for (int i = tid; i < rows; i += HELD_THREADS) A.a[i] = __builtin_nanf("");
        for (int j = tid; j < cols; j += HELD_THREADS) A.m[j] = __builtin_nanf("");
        return;
    }
    const bool held = inside == n_parts;
    const int ticket = held ? (int)blockIdx.x : __builtin_amdgcn_readfirstlane(enter[0]);   // (all are inside: the part that is in the registers)
    // 16 bytes of round `it`, once they are there; no numbers, of this and all later ones, if they do not come
    auto await4 = [&](__amdgpu_buffer_rsrc_t b, unsigned at, int it) {
        v4f x;
        for (int spin = 0;; ++spin) {
            asm volatile("" ::: "memory");   // (another load each time)
            x = held_load4(b, at);
            bool all = true;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float one = x[e];
                all = all && __builtin_bit_cast(unsigned, one) >> 31 == (unsigned)(it & 1);
            }
            if (all) break;
            lost = lost || spin >= spins;
            if (lost) {
                x.x = x.y = x.z = x.w = __builtin_nanf("");
                break;
            }
        }
        return (v4f){fabsf(x.x), fabsf(x.y), fabsf(x.z), fabsf(x.w)};
    };
    auto of_round = [](float x, int it) { return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, x) & 0x7fffffffu) | (unsigned)it << 31); };
    // this thread's columns of v as of round `it` (from 1), and the sum of their squares to lengths[]
    auto take_v = [&](int it) {
        float ss = 0.f;
#pragma unroll
        for (int k = 0; k < CPL; ++k) v[k] = live(k) ? await4(v_buffer, 4 * (unsigned)col_of(k), it) : (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < CPL; ++k) ss += (v[k].x * v[k].x + v[k].y * v[k].y) + (v[k].z * v[k].z + v[k].w * v[k].w);
        ss = dbf_wave_sum_f(ss);
        if (lane == 0) lengths[w] = ss;
    };
    for (int it = 0; it < A.iters; ++it) {
        if (it > 0) take_v(it);
        for (int part = ticket; part < n_parts; part += inside) {
            if (!held) load_part(part);
            if (it == 0) {
                // the signs: a group of eight rows is a byte column of a tile
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int group = part * G + g;
                    if (group >= (rows + DBF_TILE_ROWS - 1) / DBF_TILE_ROWS * 16) break;
#pragma unroll
                    for (int k = 0; k < CPL; ++k) {
                        unsigned out = 0;
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const v4f x = z[8 * g + r][k];
                            const unsigned four = (unsigned)(x.x >= 0.f) | (unsigned)(x.y >= 0.f) << 8 | (unsigned)(x.z >= 0.f) << 16 | (unsigned)(x.w >= 0.f) << 24;
                            out |= (live(k) && row_of(part, 8 * g + r) < rows) ? four << r : 0u;
                        }
                        const int col = col_of(k);
                        if (col < A.n_ct * DBF_TILE_COLS)
                            *reinterpret_cast<unsigned*>(A.bits + ((size_t)(group >> 4) * A.n_ct + (col >> 6)) * DBF_TILE_BYTES + 256 * ((col >> 4) & 3) +
                                                         16 * (group & 15) + (col & 15)) = out;
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float part_dot[8], sum[2];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    float d = 0.f;
#pragma unroll
                    for (int k = 0; k < CPL; ++k) {
                        const v4f x = z[8 * g + r][k];
                        if (it == 0) d += live(k) ? (fabsf(x.x) + fabsf(x.y)) + (fabsf(x.z) + fabsf(x.w)) : 0.f;
                        else d += (fabsf(x.x) * v[k].x + fabsf(x.y) * v[k].y) + (fabsf(x.z) * v[k].z + fabsf(x.w) * v[k].w);
                    }
                    part_dot[r] = d;
                }
                wave_sums<8>(part_dot, sum);
                if ((lane & 15) == 0) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) dots[8 * g + i + 2 * (lane >> 4)][w] = sum[i];
                }
            }
            __syncthreads();
            if (tid < 8 * G * HELD_WAVES) {
                static_assert(HELD_WAVES == 8, "eight neighbouring lanes have a row's parts");
                const float tot = dbf_row8_sum_f((&dots[0][0])[tid]);
                if ((tid & 7) == 0) {
                    float inv;
                    if (it == 0) {
                        inv = 1.f / sqrtf((float)cols);
                    } else {
                        float ss = lengths[0];
#pragma unroll
                        for (int i = 1; i < HELD_WAVES; ++i) ss += lengths[i];
                        const float nrm = sqrtf(ss);
                        inv = nrm > 0.f ? 1.f / nrm : 0.f;
                    }
                    const int row = row_of(part, tid >> 3);
                    const float ur = row < rows ? tot * inv : 0.f;
                    us[tid >> 3] = ur;
                    if (it + 1 == A.iters && row < rows) A.u[row] = ur;
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < CPL; ++k) acc[k] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 8 * G; ++r) {
                const float ur = us[r];
#pragma unroll
                for (int k = 0; k < CPL; ++k) {
                    const v4f x = z[r][k];
                    acc[k].x += fabsf(x.x) * ur;  acc[k].y += fabsf(x.y) * ur;  acc[k].z += fabsf(x.z) * ur;  acc[k].w += fabsf(x.w) * ur;
                }
            }
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const v4f out = {of_round(acc[k].x, it + 1), of_round(acc[k].y, it + 1), of_round(acc[k].z, it + 1), of_round(acc[k].w, it + 1)};
                held_store4(partial_of(part), 4 * (unsigned)col_of(k), out);   // (nothing beyond the last column)
            }
            if (it + 1 == A.iters && w == 0) {
                double ss = 0.;
                if (lane < 8 * G) ss = (double)us[lane] * (double)us[lane];
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
                if (lane == 0) held_store(reinterpret_cast<unsigned long long*>(A.ss + part), __builtin_bit_cast(unsigned long long, ss) | 1ull << 63);
            }
        }
        // the columns of all parts: four columns to a lane, a part to 2^LANES of them
        auto add_up = [&](auto lanes) {
            constexpr int LANES = decltype(lanes)::value, PER = HELD_THREADS >> LANES, COLS = 4 << LANES;
            const auto all = held_buffer(A.partial, 4 * (size_t)cols * n_parts);
            const int c4 = 4 * (tid & ((1 << LANES) - 1)), first = tid >> LANES;
            for (int chunk = ticket; chunk < n_chunks; chunk += inside) {
                const unsigned at = 4 * min((unsigned)(chunk * COLS + c4), (unsigned)cols - 4);
                v4f p[HELD_PARTS / PER < 4 ? HELD_PARTS / PER : 4];
                double s[4] = {0., 0., 0., 0.};
#pragma unroll
                for (int i = 0; i < (int)(sizeof(p) / sizeof(p[0])); ++i)
                    p[i] = await4(all, at + 4 * (unsigned)cols * (unsigned)min(first + PER * i, n_parts - 1), it + 1);
#pragma unroll
                for (int i = 0; i < (int)(sizeof(p) / sizeof(p[0])); ++i)
                    if (first + PER * i < n_parts) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) s[e] += (double)p[i][e];
                    }
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = held_sum<LANES>(s[e]);
                if (lane < 1 << LANES) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sums[w][c4 + e] = s[e];
                }
                __syncthreads();
                if (tid < COLS && chunk * COLS + tid < cols) {
                    double sum = sums[0][tid];
#pragma unroll
                    for (int i = 1; i < HELD_WAVES; ++i) sum += sums[i][tid];
                    held_store(A.v + chunk * COLS + tid, of_round((float)sum, it + 1));
                }
                __syncthreads();
            }
        };
        if (A.lanes == 2) add_up(std::integral_constant<int, 2>());
        else if (A.lanes == 3) add_up(std::integral_constant<int, 3>());
        else add_up(std::integral_constant<int, 4>());
    }
    // both lengths, in 64 bits; m = v_raw / ||v_raw|| and a = u_raw ||v_raw|| / ||u_raw||^2
    take_v(A.iters);
    double s[2] = {0., 0.};
#pragma unroll
    for (int k = 0; k < CPL; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[1] += (double)v[k][e] * (double)v[k][e];
    if (tid < n_parts) {
        unsigned long long ss = 0;
        for (int spin = 0; !(ss = held_load(reinterpret_cast<const unsigned long long*>(A.ss + tid))) && !lost; ++spin) lost = spin >= spins;
        s[0] = __builtin_bit_cast(double, ss & ~(1ull << 63));
    }
    if (lost) any_lost = 1;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s[i] += __shfl_xor(s[i], off, 64);
        if (lane == 0) sums[w][i] = s[i];
    }
    __syncthreads();
    if (tid < 2) {
        double sum = sums[0][tid];
#pragma unroll
        for (int i = 1; i < HELD_WAVES; ++i) sum += sums[i][tid];
        total[tid] = sum;
    }
    __syncthreads();
    // (lengths that are no numbers, as in the other last kernels: a is zero and m as it is, no numbers with a Z like that)
    const double ssu = total[0], nv = sqrt(total[1]);
    const bool none = any_lost;
#pragma unroll
    for (int k = 0; k < CPL; ++k)
        if (live(k) && (col_of(k) / chunk_cols) % inside == ticket) {
#pragma unroll
            for (int e = 0; e < 4; ++e) A.m[col_of(k) + e] = none ? __builtin_nanf("") : nv > 0. ? (float)(v[k][e] / nv) : v[k][e];
        }
    for (int part = ticket; part < n_parts; part += inside)
        if (tid < 8 * G && row_of(part, tid) < rows) {
            const int row = row_of(part, tid);
            A.a[row] = none ? __builtin_nanf("") : ssu > 0. ? (float)(A.u[row] * (nv / ssu)) : 0.f;   // (written by this workgroup)
        }
}

// The dual of the ADMM update behind the projection: U = Z - a_i m_j s_ij.  One workgroup per 128 x 64 tile of the sign matrix; thread t takes the four
// columns 4 (t % 16) .. + 3 of rows 16 s + t / 16, s = 0 .. 7.  Their eight sign quadruples are the
// eight bits of the four bytes of ONE 32-bit word of the tile (byte 256 g + 16 r + j, bit s = sign of
// row 16 s + r, column 16 g + j), and a wavefront touches four rows of 256 contiguous bytes per pass.  Bound by memory.
// FINISH: a and m are made on the way (dbf_svid_finish_kernel; u_raw and v_raw in their place), every workgroup forming both lengths from L2: a
// launch of 5 us less.  An update of 2048 x 4096 179.5 / 177.1 us, 1024 x 4096 75.5 / 72.3, 512 x 2000 44.5 / 42.7.
template <bool FINISH>
__global__ __launch_bounds__(256) void dbf_svid_dual_kernel(const float* __restrict__ Z, const float* __restrict__ a_or_u, const float* __restrict__ m_or_v,
                                                           const float* __restrict__ ss_part, int n_ss, const uint8_t* __restrict__ bits, int rows, int cols,
                                                           int n_ct, int vec_ok, float* __restrict__ a, float* __restrict__ m, float* __restrict__ out) {
    __shared__ double part[2][4];
    const int tid = threadIdx.x, lane = tid & 63, rr = tid >> 4, cq = tid & 15;
    const int row0 = blockIdx.y * DBF_TILE_ROWS + rr, col = blockIdx.x * DBF_TILE_COLS + 4 * cq;
    const unsigned w = reinterpret_cast<const unsigned*>(bits + ((size_t)blockIdx.y * n_ct + blockIdx.x) * DBF_TILE_BYTES)[64 * (cq >> 2) + 4 * rr + (cq & 3)];
    const bool vec = vec_ok && col + 4 <= cols;
    float mj[4], ai[8];
    v4f z[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) mj[e] = m_or_v[min(col + e, cols - 1)];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int row = min(row0 + 16 * s, rows - 1);
        const float* at = Z + (size_t)row * cols;
        ai[s] = a_or_u[row];
        if (vec) {
            z[s] = *reinterpret_cast<const v4f*>(at + col);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) z[s][e] = at[min(col + e, cols - 1)];
        }
    }
    if (FINISH) {
        double s[2] = {0., 0.};
        for (int j0 = tid; j0 < rows; j0 += 4 * 256) {
            float p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = a_or_u[min(j0 + 256 * e, rows - 1)];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[0] += j0 + 256 * e < rows ? (double)p[e] * (double)p[e] : 0.;
        }
        for (int j = tid; j < n_ss; j += 256) s[1] += (double)ss_part[j];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            s[k] = held_sum<2>(s[k]);   // (lanes equal modulo 4; the rest below)
            s[k] += held_dpp<0xB1>(s[k]);
            s[k] += held_dpp<0x4E>(s[k]);
            if (lane == 0) part[k][tid >> 6] = s[k];
        }
        __syncthreads();
        const double ssu = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]), ssv = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
        const double nv = sqrt(ssv), of_u = nv / ssu;
#pragma unroll
        for (int s = 0; s < 8; ++s) ai[s] = ssu > 0. ? (float)(ai[s] * of_u) : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) mj[e] = nv > 0. ? (float)(mj[e] / nv) : mj[e];
        if (blockIdx.x == 0 && cq == 0) {
#pragma unroll
            for (int s = 0; s < 8; ++s)
                if (row0 + 16 * s < rows) a[row0 + 16 * s] = ai[s];
        }
        if (blockIdx.y == 0 && rr == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < cols) m[col + e] = mj[e];
        }
    }
    if (col >= cols) return;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int row = row0 + 16 * s;
        if (row >= rows) break;
        const size_t at = (size_t)row * cols + col;
        v4f res;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float am = ai[s] * mj[e];
            res[e] = z[s][e] - (((w >> (8 * e + s)) & 1u) ? am : -am);
        }
        if (vec) {
            *reinterpret_cast<v4f*>(out + at) = res;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < cols) out[at + e] = res[e];
        }
    }
}

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }
// Groups of eight rows per workgroup of the one-pass round.
inline int round_groups_per_wg(int rows) { return (16 * dbf_row_tiles(rows) + ROUND_WGS - 1) / ROUND_WGS; }
struct RoundArgs {
    const float *Z, *v, *ss_part;
    float *u, *partial;
    uint8_t* bits;
    int rows, cols, n_ss, n_ct;
};
template <int W, int CPL, bool VEC>
int launch_round(bool first, hipStream_t st, const RoundArgs& a) {
    const int per = round_groups_per_wg(a.rows), n_groups = 16 * dbf_row_tiles(a.rows), n_wg = (n_groups + per - 1) / per;
    if (first)
        hipLaunchKernelGGL((dbf_svid_round_kernel<W, CPL, true, VEC>), dim3(n_wg), dim3(64 * W), 0, st, a.Z, a.rows, a.cols, a.v, a.ss_part,
                           a.n_ss, a.u, a.partial, per, n_groups, a.bits, a.n_ct);
    else
        hipLaunchKernelGGL((dbf_svid_round_kernel<W, CPL, false, VEC>), dim3(n_wg), dim3(64 * W), 0, st, a.Z, a.rows, a.cols, a.v, a.ss_part,
                           a.n_ss, a.u, a.partial, per, n_groups, a.bits, a.n_ct);
    return n_wg;
}
// Whether the rounds run in one launch: groups of eight rows per part, or 0.  (16-byte pieces; at most 192 values a thread, 160
// of long rows.  Less than 64 K entries: too little for a workgroup on each of a few compute units.  With 160 and more the compiler keeps 9 to 32 registers
// of a thread in scratch; a launch a round is the slower there too, us, a launch a round / one launch: 12288 x 2048 6 rounds 126.1 / 77.8, 6144 x 4096 3 68.4 / 62.0,
// 3000 x 6144 3 68.7 / 55.7, 2048 x 10240 3 77.2 / 73.7, 8 177.5 / 145.5.)
inline int held_cpl(int cols) { return (cols + 4 * HELD_THREADS - 1) / (4 * HELD_THREADS); }
inline int held_groups(int rows, int cols) {
    if ((cols & 3) || (long long)rows * cols < 1 << 16 || cols > 24576 || rows > 1 << 15) return 0;
    const int per = (16 * dbf_row_tiles(rows) + HELD_PARTS - 1) / HELD_PARTS, cpl = held_cpl(cols);
    if (per * cpl > (cpl > 3 ? 5 : 6)) return 0;
    return cpl == 1 && per == 5 ? 6 : per;
}
inline int held_parts(int rows, int groups) { return (16 * dbf_row_tiles(rows) + groups - 1) / groups; }
// 16 or 32 columns to a workgroup at a time, 64 if there are no more than 128 parts: all at once where that does it
inline int held_chunks(int cols, int lanes) { return (cols + (4 << lanes) - 1) / (4 << lanes); }
inline int held_lanes(int cols, int parts) { return held_chunks(cols, 2) <= parts ? 2 : held_chunks(cols, 3) <= parts || parts > 128 ? 3 : 4; }
// From how many rounds on one launch is the faster: its head and end cost more than two or three launches, its rounds less.  us, a launch a
// round / one launch: 4096 x 4096 3 rounds 54.5 / 47.9, 8 135.6 / 84.9; 2048 x 6144 3 52.7 / 47.6; 1640 x 10240 3 70.7 / 70.0; 1240 x 10240 3 58.4 / 61.7, 4 74.1 / 74.2; 3000 x 2048 6
// 47.7 / 45.7; 768 x 768 6 37.5 / 32.4; 1500 x 4000 6 56.0 / 56.4, 7 64.6 / 62.9; 4000 x 900 6 45.5 / 41.9.
// Few parts of long rows have the columns to add up in two or more turns, each as long as the first: two, 256 x 4096 6 46.3 / 47.3, 12 88.7 / 83.9; 384 x 4096 6
// 46.5 / 50.7, 12 88.9 / 89.8; 512 x 8192 6 60.6 / 64.4, 8 78.5 / 80.9, 12 114.3 / 113.9; 768 x 10240 6 86.0 / 80.7; three, 256 x 6144 6 53.7 / 64.2, 16 133.7 / 149.9; eight,
// 128 x 8192 6 55.3 / 122.
inline int held_rounds(int rows, int cols) {
    const int parts = held_parts(rows, held_groups(rows, cols)), turns = (held_chunks(cols, held_lanes(cols, parts)) + parts - 1) / parts;
    if (turns > 2) return INT_MAX;
    if (turns == 2 && parts < 96) return parts < 64 ? 12 : 8;
    const long long entries = (long long)rows * cols;
    return entries < 12 << 20 ? 6 : held_cpl(cols) == 5 && entries < 16 << 20 ? 4 : 3;
}
struct SvidWorkspace {
    size_t u, v, partial, scalars, least, sync, ss, total;   // `least`: what a call can do with, a launch per round
};
inline SvidWorkspace svid_workspace(int rows, int cols) {
    SvidWorkspace w;
    size_t chunks = ((size_t)rows + COL_CHUNK_ROWS - 1) / COL_CHUNK_ROWS;
    const size_t per = round_groups_per_wg(rows), n_wg = (16 * (size_t)dbf_row_tiles(rows) + per - 1) / per;
    if (n_wg > chunks) chunks = n_wg;  // partial sums: one row per 64-row chunk or per workgroup of the one-pass round
    size_t off = 0;
    w.u = off;        off = up256(off + 4 * (size_t)rows);
    w.v = off;        off = up256(off + 4 * (size_t)cols);
    w.partial = off;  off = up256(off + 4 * chunks * (size_t)cols);
    w.scalars = off;  off = up256(off + 4 * (((size_t)cols + reduce_cols(cols) - 1) / reduce_cols(cols)));   // squared length of v_raw per workgroup of the column reduction
    w.least = off;
    w.sync = w.ss = off;
    if (held_groups(rows, cols)) {
        off = up256(off + sizeof(HeldSync));
        w.ss = off;  off = up256(off + sizeof(double) * HELD_PARTS);
    }
    w.total = off;
    return w;
}
template <int CPL, int G>
void launch_held(HeldArgs a, hipStream_t st) {
    a.n_parts = held_parts(a.rows, G);
    a.door = std::min(a.door, a.n_parts);
    const int n_words = (int)(sizeof(HeldSync) / 8);
    a.lanes = held_lanes(a.cols, a.n_parts);
    a.share_ticks = (unsigned)std::min((long long)a.iters * (150 + 32ll * G * a.cols / 750), 100ll * HELD_DOOR_US);
    hipLaunchKernelGGL(dbf_svid_clear_kernel, dim3((n_words + 255) / 256), dim3(256), 0, st, reinterpret_cast<unsigned long long*>(a.sync), n_words);
    hipLaunchKernelGGL((dbf_svid_held_kernel<CPL, G>), dim3(a.n_parts), dim3(HELD_THREADS), 0, st, a);
}
void launch_held_any(int groups, const HeldArgs& a, hipStream_t st) {
    switch (10 * held_cpl(a.cols) + groups) {
        case 11: return launch_held<1, 1>(a, st);
        case 12: return launch_held<1, 2>(a, st);
        case 13: return launch_held<1, 3>(a, st);
        case 14: return launch_held<1, 4>(a, st);
        case 16: return launch_held<1, 6>(a, st);
        case 21: return launch_held<2, 1>(a, st);
        case 22: return launch_held<2, 2>(a, st);
        case 23: return launch_held<2, 3>(a, st);
        case 31: return launch_held<3, 1>(a, st);
        case 32: return launch_held<3, 2>(a, st);
        case 41: return launch_held<4, 1>(a, st);
        default: return launch_held<5, 1>(a, st);
    }
}

}  // namespace

namespace {
// The projection, and with U the dual behind it.  (The polls: of the waits of the one launch.)
int svid_run(const void* Z_dev, int rows, int cols, int iters, void* a_dev, void* m_dev, void* bits_dev, void* workspace_dev, size_t workspace_bytes, float* U,
             hipStream_t st, int door_spins = HELD_SPINS, int spins = HELD_SPINS, int door = HELD_PARTS) {
    const SvidWorkspace w = svid_workspace(rows, cols);
    const float* Z = static_cast<const float*>(Z_dev);
    uint8_t* base = static_cast<uint8_t*>(workspace_dev);
    float* u = reinterpret_cast<float*>(base + w.u);
    float* partial = reinterpret_cast<float*>(base + w.partial);
    float* ss_part = reinterpret_cast<float*>(base + w.scalars);
    const int n_rt = dbf_row_tiles(rows), n_ct = dbf_col_tiles(cols), n_ss = (cols + reduce_cols(cols) - 1) / reduce_cols(cols);
    // The last kernel's work in the dual's while every workgroup reading u is little (2048 x 4096: 1024 of 8 KiB).  An update by size, us, apart / in the
    // dual: 512 x 2000 44.5 / 42.7, 2048 x 4096 179.5 / 177.1, 4096 x 4096 516 / 516, 8192 x 4096 1918 / 1916: nothing left to gain beyond 4096 x 4096.
    const bool finish_in_dual = U && (size_t)n_rt * n_ct * rows <= 8u << 20;
    // the right factor is iterated in place in the caller's buffer, or where the dual's workgroups read it while others write m
    float* const v = finish_in_dual ? reinterpret_cast<float*>(base + w.v) : static_cast<float*>(m_dev);
    const int vec_ok = ((cols & 3) == 0 && (reinterpret_cast<uintptr_t>(Z_dev) & 15) == 0 && (reinterpret_cast<uintptr_t>(v) & 15) == 0) ? 1 : 0;
    const int vec_u = ((cols & 3) == 0 && (reinterpret_cast<uintptr_t>(Z_dev) & 15) == 0 && (reinterpret_cast<uintptr_t>(U) & 15) == 0) ? 1 : 0;
    auto dual = [&](bool finish) {
        float *a = static_cast<float*>(a_dev), *m = static_cast<float*>(m_dev);
        hipLaunchKernelGGL(finish ? dbf_svid_dual_kernel<true> : dbf_svid_dual_kernel<false>, dim3(n_ct, n_rt), dim3(256), 0, st, Z, finish ? u : a, finish ? v : m,
                           ss_part, n_ss, static_cast<const uint8_t*>(bits_dev), rows, cols, n_ct, vec_u, a, m, U);
    };
    const int chunks = (rows + COL_CHUNK_ROWS - 1) / COL_CHUNK_ROWS;

    // One pass per round wherever rows can be held: up to 24576 columns in 16-byte pieces, 12288 in single values.  8 rounds, us, two
    // passes / one: 4096 x 4096 247 / 157, now 134 (the row sums of a batch reduced together, 15.6 -> 13.7 us a round; 32 columns to a workgroup of
    // the reduction; the last kernel 6.7 -> 3.8); 2048 x 4096 161 / 93, now 83; 4 rounds of 8192 x 8192 262, now 252.
    if (const int groups = held_groups(rows, cols); groups && vec_ok && iters >= held_rounds(rows, cols) && workspace_bytes >= w.total) {
        const HeldArgs h = {Z, u, partial, static_cast<float*>(a_dev), static_cast<float*>(m_dev), reinterpret_cast<HeldSync*>(base + w.sync),
                            reinterpret_cast<float*>(base + w.v), reinterpret_cast<double*>(base + w.ss), static_cast<uint8_t*>(bits_dev),
                            rows, cols, iters, 0, n_ct, 0, 0, door_spins, spins, door};
        launch_held_any(groups, h, st);
        if (U) dual(false);
        return hipGetLastError() == hipSuccess ? DBF_OK : DBF_EHIP;
    }
    const int cpl = (cols + 4095) / 4096;  // float4s per thread and row of a workgroup of 1024
    const bool one_pass = cpl <= (vec_ok ? 6 : 3);
    if (!(one_pass && cpl == 1 && vec_ok))   // (else the first pass writes the signs)
        hipLaunchKernelGGL(dbf_svid_signs_kernel, dim3(n_ct, n_rt), dim3(256), 0, st, Z, rows, cols, n_ct,
                           static_cast<uint8_t*>(bits_dev));
    const RoundArgs ra = {Z, v, ss_part, u, partial, static_cast<uint8_t*>(bits_dev), rows, cols, n_ss, n_ct};
    for (int it = 0; it < iters; ++it) {
        if (one_pass) {
            int n_wg;
            const bool first = it == 0;
            if (vec_ok) {
                switch (cpl) {
                    case 1: n_wg = cols <= 1024 ? launch_round<4, 1, true>(first, st, ra) : cols <= 2048 ? launch_round<8, 1, true>(first, st, ra)
                                                                                          : launch_round<16, 1, true>(first, st, ra); break;
                    case 2: n_wg = launch_round<16, 2, true>(first, st, ra); break;
                    case 3: n_wg = launch_round<16, 3, true>(first, st, ra); break;
                    case 4: n_wg = launch_round<16, 4, true>(first, st, ra); break;
                    case 5: n_wg = launch_round<16, 5, true>(first, st, ra); break;
                    default: n_wg = launch_round<16, 6, true>(first, st, ra); break;
                }
            } else {
                switch (cpl) {
                    case 1: n_wg = cols <= 1024 ? launch_round<4, 1, false>(first, st, ra) : cols <= 2048 ? launch_round<8, 1, false>(first, st, ra)
                                                                                           : launch_round<16, 1, false>(first, st, ra); break;
                    case 2: n_wg = launch_round<16, 2, false>(first, st, ra); break;
                    default: n_wg = launch_round<16, 3, false>(first, st, ra); break;
                }
            }
            launch_reduce(cols, st, partial, n_wg, cols, v, ss_part);
            continue;
        }
        if (it == 0)
            hipLaunchKernelGGL(dbf_svid_row_dots_kernel<true>, dim3((rows + 3) / 4), dim3(256), 0, st, Z, rows, cols, v,
                               ss_part, n_ss, u, vec_ok);
        else
            hipLaunchKernelGGL(dbf_svid_row_dots_kernel<false>, dim3((rows + 3) / 4), dim3(256), 0, st, Z, rows, cols, v,
                               ss_part, n_ss, u, vec_ok);
        hipLaunchKernelGGL(dbf_svid_col_dots_kernel, dim3((cols + COL_BLOCK - 1) / COL_BLOCK, chunks), dim3(256), 0, st,
                           Z, rows, cols, u, partial);
        launch_reduce(cols, st, partial, chunks, cols, v, ss_part);
    }
    if (finish_in_dual) {
        dual(true);
    } else {
        const int longest = rows > cols ? rows : cols;
        hipLaunchKernelGGL(dbf_svid_finish_kernel, dim3((longest + FINISH - 1) / FINISH), dim3(FINISH), 0, st, u, rows, ss_part, n_ss, v,
                           cols, static_cast<float*>(a_dev));
        if (U) dual(false);
    }
    if (hipGetLastError() != hipSuccess) return DBF_EHIP;
    return DBF_OK;
}
}  // namespace

extern "C" size_t dbf_svid_workspace_bytes(int rows, int cols) {
    if (rows < 1 || cols < 1 || rows > DBF_MAX_DIM || cols > DBF_MAX_DIM) return 0;
    return svid_workspace(rows, cols).total;
}

size_t dbf_svid_least_workspace(int rows, int cols) { return svid_workspace(rows, cols).least; }

extern "C" int dbf_svid(const void* Z_dev, int rows, int cols, int iters, void* a_dev, void* m_dev, void* bits_dev,
                        void* workspace_dev, size_t workspace_bytes, void* hip_stream) {
    if (!Z_dev || !a_dev || !m_dev || !bits_dev || rows < 1 || cols < 1 || iters < 1) return DBF_EINVAL;
    if (rows > DBF_MAX_DIM || cols > DBF_MAX_DIM) return DBF_EINVAL;
    if ((reinterpret_cast<uintptr_t>(Z_dev) & 3) || (reinterpret_cast<uintptr_t>(a_dev) & 3) ||
        (reinterpret_cast<uintptr_t>(m_dev) & 3) || (reinterpret_cast<uintptr_t>(bits_dev) & 3))
        return DBF_EINVAL;
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 255) || workspace_bytes < svid_workspace(rows, cols).least)
        return DBF_EWORKSPACE;
    return svid_run(Z_dev, rows, cols, iters, a_dev, m_dev, bits_dev, workspace_dev, workspace_bytes, nullptr, static_cast<hipStream_t>(hip_stream));
}

int dbf_svid_dual(const void* Z_dev, int rows, int cols, int iters, void* a_dev, void* m_dev, void* bits_dev, void* workspace_dev, size_t workspace_bytes,
                  float* U_dev, hipStream_t stream) {
    return svid_run(Z_dev, rows, cols, iters, a_dev, m_dev, bits_dev, workspace_dev, workspace_bytes, U_dev, stream);
}

int dbf_svid_forced(const void* Z_dev, int rows, int cols, int iters, void* a_dev, void* m_dev, void* bits_dev, void* workspace_dev, size_t workspace_bytes,
                    int door, int door_spins, int spins, void* hip_stream) {
    if (!held_groups(rows, cols) || iters < held_rounds(rows, cols) || (reinterpret_cast<uintptr_t>(Z_dev) & 15) || (reinterpret_cast<uintptr_t>(m_dev) & 15) ||
        (reinterpret_cast<uintptr_t>(workspace_dev) & 255) || workspace_bytes < svid_workspace(rows, cols).total || door < 1 || door_spins < 0 || spins < 0)
        return DBF_EINVAL;
    return svid_run(Z_dev, rows, cols, iters, a_dev, m_dev, bits_dev, workspace_dev, workspace_bytes, nullptr, static_cast<hipStream_t>(hip_stream), door_spins, spins,
                    door);
}
