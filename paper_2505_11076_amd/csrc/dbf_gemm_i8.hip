// Prefill with the int8 matrix cores as the adder: the decode trick (dbf_gemv_mfma.hip) for T tokens.
//
//   quantise:  u = X . b per token, rounded once to 16-bit fixed point, split into two int8 planes
//   stage 1:   mid = ((X . b) B^T) . m      (T x k, fp32)   contraction over n_in
//   quantise:  mid per token -> two int8 planes
//   stage 2:   Y   = (mid A^T) . a          (T x n_out, fp16) contraction over k
//
// (forward-pass expression of the paper, section 3; the paper times batch 1 only, so this design
// is not taken from it).  Compared with a path on the fp16 matrix cores:
//   * the A operand of v_mfma_i32_16x16x64_i8 is the masked sign bytes, one AND per register
//     (0.25 vector-ALU operations per sign instead of 1), and one instruction covers 64 columns;
//   * the sums are exact integers: acc_s = 2^s * sum over set bits of q, so
//     sum(+-q) = 2 (acc_s >> s) - sum(q); the only roundings left are the two 16-bit
//     quantisations (relative 2^-16 of the row maximum) and the fp16 output;
//   * hi and lo planes are separate instructions with separate accumulators: twice the
//     instructions at twice the int8 rate.
//
// Three kernels by size, all with the same bits: up to a few dozen tokens those of dbf_gemv_few.hip (no quantising launch), then
// 128 rows x 32 tokens per workgroup (dbf_gemm_i8_mid_kernel), then the one that this describes (the rules: dbf_gemm_i8_launch,
// mid_waves).
//
// Work split of a stage of many tokens: workgroup = 256 rows x 64 tokens, 4 wavefronts; wavefront w owns row tile
// (w & 1) and the token half (w >> 1): 128 rows x 32 tokens = 8 planes x 2 token blocks x
// {hi, lo} = 32 accumulator tiles (128 registers).  Twice as many workgroups as compute units at
// 4096 rows x 2048 tokens, i.e. two wavefronts per SIMD.  The 64-token slice of the quantised
// operand (2 planes x 64 tokens x 64 bytes per step) is staged in LDS, double buffered; sign
// tiles and operand columns of step kt + 4 are requested while step kt is computed, by loads
// issued and waited for by hand (see the stage kernel).
#include "dbf_kernels.h"
#include "dbf_wave.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr float QMAX = 32512.f;     // 127*256: largest |q| so that hi and lo fit int8
constexpr int QI_TOKENS = 64;       // tokens per workgroup
constexpr int QI_ROWTILES = 2;      // 128-row tiles per workgroup
constexpr int QI_STEP = 2 * QI_TOKENS * 64;  // operand bytes of a step: two planes
constexpr int QI_DEPTH = 4;         // steps requested ahead
constexpr int QI_TB = 2;            // 16-token blocks per wavefront: 8 planes x 2 x {hi, lo} = 128 accumulator registers
constexpr int QI_TSPLIT = QI_TOKENS / (16 * QI_TB);       // token slices of a row tile
// 1: workgroups that read the same operand slice are renumbered onto one compute die (one L2); 0: launch order
#ifndef DBF_QI_XCD_REMAP
#define DBF_QI_XCD_REMAP 1
#endif

constexpr int QI_WAVES = QI_ROWTILES * QI_TSPLIT;
constexpr int QI_OCC = 2;           // wavefronts per SIMD (the accumulators leave room for no more)
constexpr int QI_THREADS = 64 * QI_WAVES;
constexpr int QI_STAGE_BYTES = 2 * QI_TOKENS * 64 / QI_THREADS;  // operand bytes a thread stages per step
static_assert(QI_STAGE_BYTES == 32, "staging is two 16-byte pieces per thread");


// ---------------------------------------------------------------------------------------------
// Quantisation of token rows: q = rint(u * 32512 / max|u|), hi/lo int8 planes.
//   FROM_F32 = false: u = x (fp16) * col_scale (fp16, zero padded)      (input of stage 1)
//   FROM_F32 = true:  u = src (fp32, leading dimension ld)               (input of stage 2)
// Output layout: the 16 tokens x 64 columns that are one operand of a matrix instruction are 1 KiB in the order of its lanes
// (lane 16 g + c: token c, columns 16 g .. + 15), fragments ordered [column step kt][16-token block][plane (0 = hi, 1 = lo)]; Tp = T rounded
// up to 64.  Loads and LDS reads of a fragment are 16 bytes per lane in lane order (with the 64 bytes of a token in one run, as
// this layout once had them, neighbouring lanes read different cache lines: 64 tag look-ups per load, which bounded
// any kernel that loads its operand straight into registers), and the 64 tokens of a stage workgroup are 8 KiB per step.
// A token's bytes are 16 apart in lines shared with seven others: workgroups are numbered so that those run on one die.
// Zeros beyond `cols`; scale[token] = max|u| / 32512, sigma[token] = sum of q.
// ---------------------------------------------------------------------------------------------
struct QuantArgs {
    const void* src;
    const uint16_t* col_scale;
    signed char* dst;
    float* scale;
    int* sigma;
    int T, Tp, cols, kp;
    long long ld;     // elements between token rows of src
    int vec_ok;       // rows can be read in 16-byte (fp16) / 32-byte (fp32) pieces
};

template <bool FROM_F32>
__device__ inline void load8(const QuantArgs& a, int token, int v, float (&u)[8]) {
    // columns 8v .. 8v+7 (v < kp/8); zero beyond `cols`
    const int c0 = 8 * v;
    if (FROM_F32) {
        const float* row = static_cast<const float*>(a.src) + (size_t)token * a.ld;
        if (a.vec_ok && c0 + 8 <= a.cols) {
            const v4f f0 = *reinterpret_cast<const v4f*>(row + c0), f1 = *reinterpret_cast<const v4f*>(row + c0 + 4);
            u[0] = f0.x;  u[1] = f0.y;  u[2] = f0.z;  u[3] = f0.w;
            u[4] = f1.x;  u[5] = f1.y;  u[6] = f1.z;  u[7] = f1.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) u[i] = c0 + i < a.cols ? row[c0 + i] : 0.f;
        }
    } else {
        const uint16_t* row = static_cast<const uint16_t*>(a.src) + (size_t)token * a.ld;
        if (a.vec_ok && c0 + 8 <= a.cols) {
            const h8 xv = *reinterpret_cast<const h8*>(row + c0);
            const h8 bv = *reinterpret_cast<const h8*>(a.col_scale + c0);
            u[0] = (float)xv.s0 * (float)bv.s0;  u[1] = (float)xv.s1 * (float)bv.s1;
            u[2] = (float)xv.s2 * (float)bv.s2;  u[3] = (float)xv.s3 * (float)bv.s3;
            u[4] = (float)xv.s4 * (float)bv.s4;  u[5] = (float)xv.s5 * (float)bv.s5;
            u[6] = (float)xv.s6 * (float)bv.s6;  u[7] = (float)xv.s7 * (float)bv.s7;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                u[i] = c0 + i < a.cols ? (float)__builtin_bit_cast(_Float16, row[c0 + i]) *
                                             (float)__builtin_bit_cast(_Float16, a.col_scale[c0 + i])
                                       : 0.f;
        }
    }
}

__device__ inline signed char* plane_at(const QuantArgs& a, int token, int v) {  // columns 8 v .. + 7 of plane 0; plane 1 is 1 KiB on
    return a.dst + ((size_t)(v >> 3) * (a.Tp >> 4) + (token >> 4)) * 2048 + 256 * ((v & 7) >> 1) + 16 * (token & 15) + 8 * (v & 1);
}
// Token of a workgroup that has one: eight neighbouring tokens to a compute die (the launch has Tp workgroups).
__device__ inline int own_token() { return (int)((blockIdx.x & ~63u) + 8 * (blockIdx.x & 7) + ((blockIdx.x >> 3) & 7)); }

// Quantises eight values and stores their two planes; returns the sum of the q.
__device__ inline int quantise_store(const QuantArgs& a, int token, int v, const float (&u)[8], float inv) {
    unsigned hi4[2] = {0, 0}, lo4[2] = {0, 0};
    int sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float f = rintf(u[i] * inv);
        f = fminf(fmaxf(f, -QMAX), QMAX);
        const int q = (int)f;
        const int lo = ((q + 128) & 255) - 128;
        const int hi = (q - lo) >> 8;
        hi4[i >> 2] |= (unsigned)(hi & 255) << (8 * (i & 3));
        lo4[i >> 2] |= (unsigned)(lo & 255) << (8 * (i & 3));
        sum += q;
    }
    signed char* d = plane_at(a, token, v);
    *reinterpret_cast<uint2*>(d) = make_uint2(hi4[0], hi4[1]);
    *reinterpret_cast<uint2*>(d + 1024) = make_uint2(lo4[0], lo4[1]);
    return sum;
}

// One wavefront per token (four tokens per workgroup, no LDS, no barriers).  Rows of up to 4096
// columns are held in registers between the max pass and the quantisation; longer rows are read
// twice (the second read hits in L2).
template <bool FROM_F32>
__global__ __launch_bounds__(256) void dbf_quantise_rows_kernel(const QuantArgs a) {
    constexpr int HOLD = 8;  // vectors of 8 columns a lane can hold
    const int lane = threadIdx.x & 63;
    const int token = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (token >= a.T) return;
    const int nvec = a.kp >> 3;
    float mx = 0.f;
    int local = 0;
    if (nvec <= 64 * HOLD) {
        float u[HOLD][8];
#pragma unroll
        for (int r = 0; r < HOLD; ++r) {
            const int v = lane + 64 * r;
            if (v < nvec) {
                load8<FROM_F32>(a, token, v, u[r]);
#pragma unroll
                for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(u[r][i]));
            }
        }
        mx = dbf_wave_max(mx);
        const float inv = mx > 0.f ? QMAX / mx : 0.f;
#pragma unroll
        for (int r = 0; r < HOLD; ++r) {
            const int v = lane + 64 * r;
            if (v < nvec) local += quantise_store(a, token, v, u[r], inv);
        }
    } else {
        for (int v = lane; v < nvec; v += 64) {
            float u[8];
            load8<FROM_F32>(a, token, v, u);
#pragma unroll
            for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(u[i]));
        }
        mx = dbf_wave_max(mx);
        const float inv = mx > 0.f ? QMAX / mx : 0.f;
        for (int v = lane; v < nvec; v += 64) {
            float u[8];
            load8<FROM_F32>(a, token, v, u);
            local += quantise_store(a, token, v, u, inv);
        }
    }
    local = dbf_wave_sum(local);
    if (lane == 0) {
        a.scale[token] = mx / QMAX;
        a.sigma[token] = local;
    }
}

// Rows held in registers: a workgroup of 1024 threads has four tokens, a quarter of every wavefront each (so that a store of a plane
// writes the 16 bytes of four neighbouring tokens next to each other; with a workgroup per token it wrote 16 bytes to a cache
// line, and 2048 tokens of 11008 columns took 23.8 us), HOLD vector items of 8 columns per thread: rows of up to 2048 * HOLD columns
// that can be read in 16-byte pieces.  Straight-line: every load of the row is issued before anything waits (vector items
// beyond the row are read as its last one and zeroed afterwards); the wavefronts exchange their maxima and sums through LDS.
// With many wavefronts of little work the launch is as long as one memory round trip and a little arithmetic.
template <bool FROM_F32, int HOLD>
__global__ __launch_bounds__(1024) void dbf_quantise_rows_held_kernel(const QuantArgs a) {
    __shared__ __align__(16) float wmax[4][16];
    __shared__ __align__(16) int wsum[4][16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, tau = lane >> 4;
    // (two workgroups share the lines they write: the same die)
    const int token = 4 * (int)((blockIdx.x & ~15u) + 2 * (blockIdx.x & 7) + ((blockIdx.x >> 3) & 1)) + tau;
    const bool live = token < a.T;
    const int v0 = 16 * w + (lane & 15);
    const int nvec = a.kp >> 3, nreal = a.cols >> 3;
    float u[HOLD][8];
    if (FROM_F32) {
        const float* row = static_cast<const float*>(a.src) + (size_t)min(token, a.T - 1) * a.ld;
        v4f f0[HOLD], f1[HOLD];
#pragma unroll
        for (int r = 0; r < HOLD; ++r) {
            const int c0 = 8 * min(v0 + 256 * r, nreal - 1);
            f0[r] = *reinterpret_cast<const v4f*>(row + c0);
            f1[r] = *reinterpret_cast<const v4f*>(row + c0 + 4);
        }
#pragma unroll
        for (int r = 0; r < HOLD; ++r) {
            const bool in = v0 + 256 * r < nreal;
            u[r][0] = in ? f0[r].x : 0.f;  u[r][1] = in ? f0[r].y : 0.f;
            u[r][2] = in ? f0[r].z : 0.f;  u[r][3] = in ? f0[r].w : 0.f;
            u[r][4] = in ? f1[r].x : 0.f;  u[r][5] = in ? f1[r].y : 0.f;
            u[r][6] = in ? f1[r].z : 0.f;  u[r][7] = in ? f1[r].w : 0.f;
        }
    } else {
        const uint16_t* row = static_cast<const uint16_t*>(a.src) + (size_t)min(token, a.T - 1) * a.ld;
        h8 xv[HOLD], bv[HOLD];
#pragma unroll
        for (int r = 0; r < HOLD; ++r) {
            const int c0 = 8 * min(v0 + 256 * r, nreal - 1);
            xv[r] = *reinterpret_cast<const h8*>(row + c0);
            bv[r] = *reinterpret_cast<const h8*>(a.col_scale + c0);
        }
#pragma unroll
        for (int r = 0; r < HOLD; ++r) {
            const bool in = v0 + 256 * r < nreal;
#pragma unroll
            for (int i = 0; i < 8; ++i) u[r][i] = in ? (float)xv[r][i] * (float)bv[r][i] : 0.f;
        }
    }
    float mx = 0.f;
#pragma unroll
    for (int r = 0; r < HOLD; ++r)
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(u[r][i]));
    mx = dbf_row16_max(mx);
    if ((lane & 15) == 0) wmax[tau][w] = mx;
    __syncthreads();
    mx = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) mx = fmaxf(mx, wmax[tau][q]);
    const float inv = mx > 0.f ? QMAX / mx : 0.f;
    int local = 0;
#pragma unroll
    for (int r = 0; r < HOLD; ++r) {
        const int v = v0 + 256 * r;
        if (live && v < nvec) local += quantise_store(a, token, v, u[r], inv);
    }
    local = dbf_row16_sum(local);
    if ((lane & 15) == 0) wsum[tau][w] = local;
    __syncthreads();
    if (w == 0 && (lane & 15) == 0 && live) {
        int sum = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) sum += wsum[tau][q];
        a.scale[token] = mx / QMAX;
        a.sigma[token] = sum;
    }
}

// One workgroup per token: for rows too long to hold in a wavefront's registers.
template <bool FROM_F32>
__global__ __launch_bounds__(256) void dbf_quantise_rows_block_kernel(const QuantArgs a) {
    __shared__ float wmax[4];
    __shared__ int wsum[4];
    const int token = own_token();
    if (token >= a.T) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int nvec = a.kp >> 3;
    float mx = 0.f;
    for (int v = tid; v < nvec; v += 256) {
        float u[8];
        load8<FROM_F32>(a, token, v, u);
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(u[i]));
    }
    mx = dbf_wave_max(mx);
    if (lane == 0) wmax[w] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    const float inv = mx > 0.f ? QMAX / mx : 0.f;
    int local = 0;
    for (int v = tid; v < nvec; v += 256) {
        float u[8];
        load8<FROM_F32>(a, token, v, u);   // second read of the row: L2 resident
        unsigned hi4[2] = {0, 0}, lo4[2] = {0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float f = rintf(u[i] * inv);
            f = fminf(fmaxf(f, -QMAX), QMAX);
            const int q = (int)f;
            const int lo = ((q + 128) & 255) - 128;
            const int hi = (q - lo) >> 8;
            hi4[i >> 2] |= (unsigned)(hi & 255) << (8 * (i & 3));
            lo4[i >> 2] |= (unsigned)(lo & 255) << (8 * (i & 3));
            local += q;
        }
        signed char* d = plane_at(a, token, v);
        *reinterpret_cast<uint2*>(d) = make_uint2(hi4[0], hi4[1]);
        *reinterpret_cast<uint2*>(d + 1024) = make_uint2(lo4[0], lo4[1]);
    }
    local = dbf_wave_sum(local);
    if (lane == 0) wsum[w] = local;
    __syncthreads();
    if (tid == 0) {
        a.scale[token] = mx / QMAX;
        a.sigma[token] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    }
}

// Rows of eight values and more that start anywhere, read twice (the second read hits in L2 or the last-level cache): a workgroup of 1024
// threads has eight tokens, a wavefront every 16th column step of theirs, a token eight of its lanes.  So a wavefront's load is
// whole cache lines of eight rows (128 bytes of fp16 each) and its store of a plane whole lines too (eight tokens x 16 bytes, four
// times): what bounds the kernels above at many tokens is writing a line in eight pieces.  (Of a FROM_F32 row every column is there.)
template <bool FROM_F32>
__global__ __launch_bounds__(1024) void dbf_quantise_rows_twice_kernel(const QuantArgs a) {
    constexpr int UN = 4;   // steps of a wavefront whose loads are in flight together
    __shared__ __align__(16) float wmax[8][16];
    __shared__ __align__(16) int wsum[8][16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, tau = lane >> 3;
    const int token = 8 * blockIdx.x + tau, n_steps = a.kp >> 6;
    const bool live = token < a.T;
    const char* row = static_cast<const char*>(a.src) + (size_t)min(token, a.T - 1) * a.ld * (FROM_F32 ? 4 : 2);
    // eight values of every step kt0 + 16 i (steps past the row: its last one again)
    auto load = [&](int kt0, float (&u)[UN][8]) {
        v4u r0[UN], r1[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int v = 8 * min(kt0 + 16 * i, n_steps - 1) + (lane & 7);
            if (FROM_F32) {
                r0[i] = *reinterpret_cast<const v4u*>(row + 32 * (size_t)v);
                r1[i] = *reinterpret_cast<const v4u*>(row + 32 * (size_t)v + 16);
            } else {
                r0[i] = dbf_half8_load(reinterpret_cast<const uint16_t*>(row), v, a.cols);
                r1[i] = *reinterpret_cast<const v4u*>(a.col_scale + 8 * (size_t)v);
            }
        }
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            const int v = 8 * min(kt0 + 16 * i, n_steps - 1) + (lane & 7);
            if (FROM_F32) {
                const v4f f0 = __builtin_bit_cast(v4f, r0[i]), f1 = __builtin_bit_cast(v4f, r1[i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    u[i][e] = f0[e];
                    u[i][4 + e] = f1[e];
                }
            } else {
                const h8 xv = __builtin_bit_cast(h8, dbf_half8_place(r0[i], v, a.cols)), bv = __builtin_bit_cast(h8, r1[i]);
#pragma unroll
                for (int e = 0; e < 8; ++e) u[i][e] = (float)xv[e] * (float)bv[e];
            }
        }
    };
    float mx = 0.f;
    for (int kt0 = w; kt0 < n_steps; kt0 += 16 * UN) {
        float u[UN][8];
        load(kt0, u);
#pragma unroll
        for (int i = 0; i < UN; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(u[i][e]));
    }
    mx = dbf_row8_max(mx);
    if ((lane & 7) == 0) wmax[tau][w] = mx;
    __syncthreads();
    mx = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) mx = fmaxf(mx, wmax[tau][q]);
    const float inv = mx > 0.f ? QMAX / mx : 0.f;
    int local = 0;
    for (int kt0 = w; kt0 < n_steps; kt0 += 16 * UN) {
        float u[UN][8];
        load(kt0, u);
#pragma unroll
        for (int i = 0; i < UN; ++i)
            if (live && kt0 + 16 * i < n_steps) local += quantise_store(a, token, 8 * (kt0 + 16 * i) + (lane & 7), u[i], inv);
    }
    local = dbf_row8_sum(local);
    if ((lane & 7) == 0) wsum[tau][w] = local;
    __syncthreads();
    if (w == 0 && (lane & 7) == 0 && live) {
        int sum = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) sum += wsum[tau][q];
        a.scale[token] = mx / QMAX;
        a.sigma[token] = sum;
    }
}

// ---------------------------------------------------------------------------------------------
// One stage: out[token][row] = rscale[row] * scale[token] * sum_col sign(row, col) * q[token][col]
// ---------------------------------------------------------------------------------------------
struct StageArgs {
    const uint8_t* bits;        // tiled sign matrix: n_rt x n_ct tiles
    const uint16_t* row_scale;  // fp16 [n_rt*128] (m or a, zero padded)
    const signed char* xq;      // [n_ct][Tp / 16][2][1024] quantised operand (see above)
    const float* scale;         // [T]
    const int* sigma;           // [T]
    void* out;                  // OUT_F32: float [T][ldo]; else fp16 [T][ldo]
    int n_rt, n_ct, T, Tp, ldo;
    int n_valid;                // output rows to store
};

// Four consecutive outputs of a token.
template <bool OUT_F32>
__device__ inline void store4(const StageArgs& a, int token, int n0, const float (&v)[4]) {
                if (OUT_F32) {
                    float* dst = static_cast<float*>(a.out) + (size_t)token * a.ldo + n0;
                    if (n0 + 4 <= a.n_valid) {
                        *reinterpret_cast<v4f*>(dst) = (v4f){v[0], v[1], v[2], v[3]};
                    } else {
    #pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (n0 + i < a.n_valid) dst[i] = v[i];
                    }
                } else {
                    uint16_t* dst = static_cast<uint16_t*>(a.out) + (size_t)token * a.ldo + n0;
                    const bool vec_ok = (a.ldo & 3) == 0 && (reinterpret_cast<uintptr_t>(a.out) & 7) == 0;
                    if (vec_ok && n0 + 4 <= a.n_valid) {
                        typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                        *reinterpret_cast<h4*>(dst) = (h4){(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
                    } else {
    #pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (n0 + i < a.n_valid) dst[i] = __builtin_bit_cast(uint16_t, (_Float16)v[i]);
                    }
                }
}

template <bool OUT_F32>
__global__ __launch_bounds__(QI_THREADS) __attribute__((amdgpu_waves_per_eu(QI_OCC, QI_OCC)))
void dbf_gemm_i8_stage_kernel(const StageArgs a) {
    __shared__ __align__(16) unsigned char xs[2][QI_STEP];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    // Workgroups are handed to the 8 compute dies in turn (linear id modulo 8) and each die has its own L2.
    // All workgroups of a token block read the same operand slice, so they are renumbered to share a die:
    // die d takes a contiguous range of the (token block, row group) pairs, row group fastest.
#if DBF_QI_XCD_REMAP
    const unsigned n_wg = gridDim.x * gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
    const unsigned die = lin & 7, slot = lin >> 3, per = n_wg >> 3, extra = n_wg & 7;
    const unsigned vid = die * per + (die < extra ? die : extra) + slot;
    const int bx = (int)(vid % gridDim.x), by = (int)(vid / gridDim.x);
#else
    const int bx = blockIdx.x, by = blockIdx.y;
#endif
    const int token0 = by * QI_TOKENS;
    const int th = w / QI_ROWTILES;                          // token slice of this wavefront
    int rt = bx * QI_ROWTILES + (w % QI_ROWTILES);           // its row tile
    const bool active = rt < a.n_rt;                         // beyond the matrix: compute on tile 0, store nothing
    if (!active) rt = 0;

    // staging: the 8 KiB of a step are contiguous in memory and in LDS; thread t takes bytes 16 t and 4096 + 16 t
    constexpr int SB = QI_STAGE_BYTES;
    // (tokens in [T, Tp) hold whatever the workspace held: they are computed and never stored)
    const size_t s_step = (size_t)a.Tp * 128;                // bytes between steps
    unsigned char* s_dst0 = xs[0] + 16 * tid;
    unsigned char* s_dst1 = xs[1] + 16 * tid;

    v4i acc[8][QI_TB][2];  // [plane s][token block][hi, lo]
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int tb = 0; tb < QI_TB; ++tb) {
            acc[s][tb][0] = (v4i){0, 0, 0, 0};
            acc[s][tb][1] = (v4i){0, 0, 0, 0};
        }

    // Software pipeline with hand-issued loads.  The sign tile and the operand bytes of step kt + QI_DEPTH are
    // requested at the end of step kt by inline assembly and waited for by hand: the compiler does not see
    // these loads, so it cannot drain the whole pipeline with a vmcnt(0) wait at the loop's back edge (which
    // it does for loads it tracks: once per QI_DEPTH steps every wavefront then sits out a full memory
    // latency).  Loads complete in issue order.  A step's group is issued as (x0, x1, bq); at the top of step
    // kt the groups of steps kt+1 .. kt+3 are in flight behind bq of step kt, and the step needs bq(kt),
    // x0(kt+1), x1(kt+1): bq(kt+1) and the two younger groups may stay outstanding = 1 + 3 + 3 loads.
    static_assert(QI_DEPTH == 4 && SB == 32, "the wait counts below are written for this pipeline");
    v4u bq[QI_DEPTH], x0[QI_DEPTH], x1[QI_DEPTH];
    const int last_ct = a.n_ct - 1;
    const unsigned x_voff = (unsigned)(16 * tid), t_voff = (unsigned)(lane * 16);
    const signed char* x_base = a.xq + (size_t)token0 * 128;
    const uint8_t* t_base = a.bits + (size_t)rt * a.n_ct * DBF_TILE_BYTES;
    auto request = [&](int j, int kt) {  // kt is the same for all lanes: the step's part of the address is scalar
        const signed char* xs_ = x_base + (size_t)kt * s_step;
        const uint8_t* ts_ = t_base + (size_t)kt * DBF_TILE_BYTES;
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(x0[j]) : "v"(x_voff), "s"(xs_) : "memory");
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(x1[j]) : "v"(x_voff + 4096u), "s"(xs_) : "memory");
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(bq[j]) : "v"(t_voff), "s"(ts_) : "memory");
    };
#pragma unroll
    for (int j = 0; j < QI_DEPTH; ++j) request(j, min(j, last_ct));
    asm volatile("s_waitcnt vmcnt(10)" : "+v"(x0[0]), "+v"(x1[0]) : : "memory");
    *reinterpret_cast<v4u*>(s_dst0) = x0[0];
    *reinterpret_cast<v4u*>(s_dst0 + 4096) = x1[0];
    __syncthreads();

    const unsigned char* xlane = xs[0] + QI_TB * th * 2048 + 16 * lane;

    for (int kt0 = 0; kt0 < a.n_ct; kt0 += QI_DEPTH) {
#pragma unroll
        for (int j = 0; j < QI_DEPTH; ++j) {
            const int kt = kt0 + j;
            const int jn = (j + 1) % QI_DEPTH;
            asm volatile("s_waitcnt vmcnt(7)" : "+v"(x0[jn]), "+v"(x1[jn]), "+v"(bq[j]) : : "memory");
            // stage step kt + 1 into the other buffer
            {
                unsigned char* d = (j & 1) ? s_dst0 : s_dst1;
                *reinterpret_cast<v4u*>(d) = x0[jn];
                *reinterpret_cast<v4u*>(d + 4096) = x1[jn];
            }
            // A step beyond the matrix contributes nothing if its sign operand is zero (no branch around
            // the matrix instructions); `live` is the same for all lanes and is folded into the plane masks.
            const unsigned live = kt < a.n_ct ? 0xFFFFFFFFu : 0u;
            const unsigned char* xb = xlane + (j & 1) * QI_STEP;
            v4i xop[QI_TB][2];
#pragma unroll
            for (int tb = 0; tb < QI_TB; ++tb) {
                xop[tb][0] = *reinterpret_cast<const v4i*>(xb + tb * 2048);
                xop[tb][1] = *reinterpret_cast<const v4i*>(xb + tb * 2048 + 1024);
            }
            v4i av[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const unsigned msk = (0x01010101u << s) & live;
                av[s].x = (int)(bq[j].x & msk);
                av[s].y = (int)(bq[j].y & msk);
                av[s].z = (int)(bq[j].z & msk);
                av[s].w = (int)(bq[j].w & msk);
                if (s == 7) {
                    // every register of slot j has been read: request step kt + QI_DEPTH into it
                    asm volatile("" : "+v"(av[s]), "+v"(bq[j]), "+v"(x0[j]), "+v"(x1[j]));
                    request(j, min(kt + QI_DEPTH, last_ct));
                }
#pragma unroll
                for (int tb = 0; tb < QI_TB; ++tb) {
                    acc[s][tb][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[s], xop[tb][0], acc[s][tb][0], 0, 0, 0);
                    acc[s][tb][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[s], xop[tb][1], acc[s][tb][1], 0, 0, 0);
                }
            }
            __syncthreads();
        }
    }
    // the requests of the last QI_DEPTH steps are still in flight: let them land before their registers are reused
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int j = 0; j < QI_DEPTH; ++j) asm volatile("" : "+v"(bq[j]), "+v"(x0[j]), "+v"(x1[j]));

    // ---- epilogue: acc[s][tb][p][i] of lane (g, c) is row 16*s + 4*g + i, token 32*th + 16*tb + c ----
    if (!active) return;
#pragma unroll
    for (int tb = 0; tb < QI_TB; ++tb) {
        const int token = token0 + 16 * QI_TB * th + 16 * tb + c;
        if (token >= a.T) continue;
        const float tscale = a.scale[token];
        const int tsigma = a.sigma[token];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int n0 = rt * DBF_TILE_ROWS + 16 * s + 4 * g;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int vh = acc[s][tb][0][i] >> s, vl = acc[s][tb][1][i] >> s;
                if (s == 7) {  // the mask 0x80 is -128 as an int8
                    vh = -vh;
                    vl = -vl;
                }
                const int set_sum = vh * 256 + vl;   // the sum of q over the set bits of the row, exact
                // (2 * the sum of the set bits' q may pass 2^31 on the way to a total that fits: modular arithmetic)
                const int total = (int)(2u * (unsigned)set_sum - (unsigned)tsigma);
                const float rs = (float)__builtin_bit_cast(_Float16, a.row_scale[n0 + i]);
                v[i] = (float)total * tscale * rs;
            }
            store4<OUT_F32>(a, token, n0, v);
        }
    }
}

// The same stage for calls of a few hundred tokens, where workgroups of 256 rows x 64 tokens leave compute units idle or alone with
// one wavefront per SIMD: a workgroup of 128 rows x 32 tokens whose WAVES wavefronts take an equal share of the column steps each.
// Every wavefront has 128 rows x 32 tokens of its own (the accumulators of the kernel above), loads its sign tiles and operand
// bytes straight into registers, MID_DEPTH steps ahead, and meets the others only at the end: exact integer sums through LDS.
// No barrier and no LDS traffic per step; the matrix pipe with its ANDs and the loads bound it together: at 411 tokens of 4096 -> 11008,
// k = 4477, the A stage (1118 workgroups, 52 us) keeps the matrix pipes 48 % busy and brings 400 MB (5 KiB per wavefront and step) to
// registers, 7.7 TB/s, 79 % of the requests hitting L2; the B stage (611 workgroups, 24 us) 38 %.  The kernel above: 62-65 % busy.
constexpr int MID_TOKENS = 32, MID_DEPTH = 3;
constexpr int MID_LDS = 16 * 64 * 16;   // per wavefront
template <bool OUT_F32, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_gemm_i8_mid_kernel(const StageArgs a) {
    extern __shared__ __align__(16) unsigned char mid_lds[];   // [WAVES][16 blocks of 8 rows][64 lanes][16 bytes]
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (workgroups of a token block on one compute die: see the kernel above)
    const unsigned n_x = a.n_rt, n_wg = n_x * ((a.T + MID_TOKENS - 1) / MID_TOKENS), lin = blockIdx.x;
    const unsigned die = lin & 7, slot = lin >> 3, per = n_wg >> 3, extra = n_wg & 7;
    const unsigned vid = die * per + (die < extra ? die : extra) + slot;
    const int rt = (int)(vid % n_x), token0 = (int)(vid / n_x) * MID_TOKENS;
    const int lo = a.n_ct * w / WAVES, hi = a.n_ct * (w + 1) / WAVES;

    const auto signs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.bits + (size_t)rt * a.n_ct * DBF_TILE_BYTES), 0,
                                                         a.n_ct * DBF_TILE_BYTES, 0x00020000);
    const unsigned step = (unsigned)a.Tp * 128;   // operand bytes from one column step to the next
    const auto operand = __builtin_amdgcn_make_buffer_rsrc(const_cast<signed char*>(a.xq), 0, (int)(step * a.n_ct), 0x00020000);
    // (32 x 32 x 32: lane l supplies row l % 32, columns 16 (l / 32) .. + 15 of the signs -- r-row l % 16 of bit plane 2 sp + (l / 16) % 2,
    //  so lanes 16 apart hold the same bytes and differ in the mask -- and token l % 32, the same columns, of a plane of the operand)
    const int h = lane >> 5, l32 = lane & 31;
    const unsigned t_off = 256u * h + 16u * (lane & 15), x_off = (unsigned)token0 * 128 + 2048u * ((lane >> 4) & 1) + 256u * h + 16u * (lane & 15);
    unsigned mask[4];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) mask[sp] = 0x01010101u << (2 * sp + ((lane >> 4) & 1));
    v4u tl[MID_DEPTH][2], x[MID_DEPTH][2][2];   // [half of the 64 columns], [half][hi, lo]
    auto fetch = [&](int j, int kt) {        // (steps past the wavefront's share: offsets out of range, no memory traffic)
        const unsigned k = kt < hi ? (unsigned)kt : 0u, gone = kt < hi ? 0u : 0x80000000u;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) tl[j][kh] = __builtin_amdgcn_raw_buffer_load_b128(signs, t_off + gone + 512 * kh, k * DBF_TILE_BYTES, 0);
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int p = 0; p < 2; ++p) x[j][kh][p] = __builtin_amdgcn_raw_buffer_load_b128(operand, x_off + gone + 512 * kh + 1024 * p, k * step, 0);
    };
    v16i acc[4][2];   // [planes 2 sp, 2 sp + 1][hi, lo]
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[sp][p][v] = 0;
#pragma unroll
    for (int j = 0; j < MID_DEPTH; ++j) {
        fetch(j, lo + j);
        __builtin_amdgcn_sched_barrier(0);
    }
    auto multiply = [&](int j) {
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int sp = 0; sp < 4; ++sp) {
                const v4i av = {(int)(tl[j][kh].x & mask[sp]), (int)(tl[j][kh].y & mask[sp]), (int)(tl[j][kh].z & mask[sp]),
                                (int)(tl[j][kh].w & mask[sp])};
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    acc[sp][p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, __builtin_bit_cast(v4i, x[j][kh][p]), acc[sp][p], 0, 0, 0);
            }
    };
    // (whole rounds of the ring, then the rest without new requests: with a way out in the middle of a round the compiler
    //  cannot tell which loads are still under way at its start, and waits for all of them)
    int k0 = lo;
    for (; k0 + MID_DEPTH <= hi; k0 += MID_DEPTH) {
#pragma unroll
        for (int j = 0; j < MID_DEPTH; ++j) {
            multiply(j);
            fetch(j, k0 + j + MID_DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int j = 0; j < MID_DEPTH - 1; ++j) {
        if (k0 + j >= hi) break;
        multiply(j);
    }
    // register v of acc[sp][p] of lane (h, l32): row 32 sp + 8 (v / 4) + 4 h + v % 4 (bit plane 2 sp + v / 8), token l32.  The two
    // planes of the operand become one sum per output.
    v4i* mine = reinterpret_cast<v4i*>(mid_lds) + (size_t)w * 16 * 64 + lane;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int s = 2 * sp + (b >> 1);
            v4i v;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = (int)(((unsigned)(acc[sp][0][4 * b + i] >> s) << 8) + (unsigned)(acc[sp][1][4 * b + i] >> s));
                v[i] = s == 7 ? -q : q;   // (the mask 0x80 is -128 as an int8)
            }
            mine[(4 * sp + b) * 64] = v;
        }
    __syncthreads();
    const int token = token0 + l32;
    if (token >= a.T) return;
    const float tscale = a.scale[token];
    const int tsigma = a.sigma[token];
#pragma unroll
    for (int e = 0; e < 16 / WAVES; ++e) {
        const int idx = w + WAVES * e, n0 = rt * DBF_TILE_ROWS + 8 * idx + 4 * h;
        v4i sum = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < WAVES; ++q) sum += reinterpret_cast<const v4i*>(mid_lds)[((size_t)q * 16 + idx) * 64 + lane];
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int total = (int)(2u * (unsigned)sum[i] - (unsigned)tsigma);
            v[i] = (float)total * tscale * (float)__builtin_bit_cast(_Float16, a.row_scale[n0 + i]);
            asm("" : "+v"(v[i]));   // (rounded to fp32 before anything else, as in every kernel of the layer product)
        }
        store4<OUT_F32>(a, token, n0, v);
    }
}

// The quantiser for a row length: rows held in registers where they can be read in 16-byte pieces (up to 4096 and up to 12288 padded
// columns); longer ones by a workgroup per token, or by eight tokens a workgroup where that gives 160 workgroups and the planes (48 MB
// and more) are beyond the L2s, so that pieces of a line no longer meet there.  Rows that cannot be read in 16-byte pieces: up to 2048
// columns by a wavefront per token, up to 4096 by eight tokens a workgroup, beyond by the latter from 384 tokens on.
// Launches, us, a workgroup per token / eight tokens: 28672 columns  1024 tokens 34 / 47   1280: 48 / 47   1536: 88 / 58   4096: 269 / 137;
// 14336  1024: 17.7 / 26.2   1536: 26.1 / 28.4   2048: 39 / 31   4096: 95 / 64;   11007  777: 45 / 22   4096: 179 / 50 (calls of
// 11007 -> 4096 at 64 / 256 / 384 tokens 41.1, 64.0, 80.4 / 44.3, 66.6, 78.3);   a wavefront per token / eight tokens: 4095  256: 16.4 / 9.8
// 777: 14.3 / 12.0   4096: 59 / 21;   1001  777: 5.2 / 8.4   4096: 14.8 / 16.0.
template <bool FROM_F32>
void launch_quantise(const QuantArgs& q, size_t kp, int T, hipStream_t stream) {
    const bool straight = q.vec_ok && (q.cols & 7) == 0 && q.cols >= 8;
    if (straight && kp <= 4096)
        hipLaunchKernelGGL((dbf_quantise_rows_held_kernel<FROM_F32, 2>), dim3(q.Tp / 4), dim3(1024), 0, stream, q);
    else if (straight && kp <= 12288)
        hipLaunchKernelGGL((dbf_quantise_rows_held_kernel<FROM_F32, 6>), dim3(q.Tp / 4), dim3(1024), 0, stream, q);
    else if (straight ? T >= 1280 && T * kp >= 24u << 20 : kp > 4096 ? T >= 384 : kp > 2048)
        hipLaunchKernelGGL(dbf_quantise_rows_twice_kernel<FROM_F32>, dim3(q.Tp / 8), dim3(1024), 0, stream, q);
    else if (kp <= 4096)
        hipLaunchKernelGGL(dbf_quantise_rows_kernel<FROM_F32>, dim3((T + 3) / 4), dim3(256), 0, stream, q);
    else
        hipLaunchKernelGGL(dbf_quantise_rows_block_kernel<FROM_F32>, dim3(q.Tp), dim3(256), 0, stream, q);
}

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Which kernel a stage takes, by their measured times on a full chip: the 256 x 64 kernel 0.43 us per column step while a compute unit
// has one workgroup and 0.68 with two, in rounds of 512 workgroups; the 128 x 32 kernel 0.44 us per 1024 workgroups and step, in whatever
// number there are.  Calls, us, 256 x 64 / 128 x 32:  4096 x 4096, k = 4096  64 tokens 50.8 / 22.6   256: 65.3 / 26.1   512: 70.4 / 40.8
//   1024: 74.1 / 69.5   2048: 112.7 / 130.9;   4096 -> 11008, k = 5970  128: 77.3 / 34.8   411: 105.5 / 78.5   800: 152.9 / 131.5
//   1024: 154.4 / 159.9   2048: 269.8 / 310.6.  Eight wavefronts for up to 256 workgroups of the latter (22.6 against 23.5 at 64 tokens), else
// four, two workgroups to a compute unit (78.5 against 85.7 at 411 tokens).
int mid_waves(int n_rt, int n_ct, int T) {
    const int forced = dbf_tune(DBF_TUNE_GEMM_SPLITS);
    if (forced == 1 || (long long)((T + 63) & ~63) * 128 * n_ct >= 1LL << 31) return 0;   // (32-bit buffer offsets)
    const long long n = (long long)n_rt * ((T + MID_TOKENS - 1) / MID_TOKENS);
    if (forced > 1) return forced < 8 ? 4 : 8;
    const long long wgs = (long long)((n_rt + QI_ROWTILES - 1) / QI_ROWTILES) * ((T + QI_TOKENS - 1) / QI_TOKENS);
    const long long rounds = wgs / 512, rest = wgs % 512;
    const double big = 0.68 * (double)rounds + (rest > 256 ? 0.68 : rest > 0 ? 0.43 : 0.);
    if (0.44 * (double)n / 1024 > big) return 0;
    return n <= 256 ? 8 : 4;
}

// workspace carve-up (all sections 256-byte aligned)
struct I8Workspace {
    size_t xq1, sc1, sg1, mid, xq2, sc2, sg2, total;
};
inline I8Workspace i8_workspace(const dbf_layer* L, int T) {
    const size_t kp1 = (size_t)dbf_col_tiles(L->n_in) * DBF_TILE_COLS;
    const size_t kp2 = (size_t)dbf_col_tiles(L->k) * DBF_TILE_COLS;
    const size_t ks = (size_t)dbf_row_tiles(L->k) * DBF_TILE_ROWS;
    const size_t Tp = ((size_t)T + 63) & ~(size_t)63;
    I8Workspace w;
    size_t off = 0;
    w.xq1 = off;  off = align256(off + Tp * 2 * kp1);
    w.sc1 = off;  off = align256(off + (size_t)T * 4);
    w.sg1 = off;  off = align256(off + (size_t)T * 4);
    w.mid = off;  off = align256(off + (size_t)T * ks * 4);
    w.xq2 = off;  off = align256(off + Tp * 2 * kp2);
    w.sc2 = off;  off = align256(off + (size_t)T * 4);
    w.sg2 = off;  off = align256(off + (size_t)T * 4);
    w.total = off;
    return w;
}

template <bool OUT_F32>
void launch_stage(const StageArgs& s, hipStream_t stream) {
    const int waves = mid_waves(s.n_rt, s.n_ct, s.T);
    const dim3 mid_grid(s.n_rt * ((s.T + MID_TOKENS - 1) / MID_TOKENS));
    if (waves == 8)
        hipLaunchKernelGGL((dbf_gemm_i8_mid_kernel<OUT_F32, 8>), mid_grid, dim3(512), 8 * MID_LDS, stream, s);
    else if (waves == 4)
        hipLaunchKernelGGL((dbf_gemm_i8_mid_kernel<OUT_F32, 4>), mid_grid, dim3(256), 4 * MID_LDS, stream, s);
    else
        hipLaunchKernelGGL((dbf_gemm_i8_stage_kernel<OUT_F32>), dim3((s.n_rt + QI_ROWTILES - 1) / QI_ROWTILES, (s.T + QI_TOKENS - 1) / QI_TOKENS),
                           dim3(QI_THREADS), 0, stream, s);
}

}  // namespace

size_t dbf_gemm_i8_workspace_bytes(const dbf_layer* L, int T) { return i8_workspace(L, T).total; }

// More than 64 KiB of LDS per workgroup has to be asked for, once per process (see dbf_mfma_prepare).
hipError_t dbf_gemm_i8_prepare() {
    static const hipError_t raised = [] {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dbf_gemm_i8_mid_kernel<true, 8>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           8 * MID_LDS);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dbf_gemm_i8_mid_kernel<false, 8>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    8 * MID_LDS);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }();
    return raised;
}

// Launches the two stages on `stream`: each as one launch whose workgroups round their own input, where there are few of
// them (dbf_few_takes), else as quantise -> stage.  Arguments are validated by the caller (dbf_gemm); `ws` holds
// dbf_gemm_i8_workspace_bytes(L, T) bytes.
hipError_t dbf_gemm_i8_launch(const dbf_layer* L, const void* X_dev, void* Y_dev, int T, void* ws, hipStream_t stream) {
    const hipError_t raised = dbf_gemm_i8_prepare();
    if (raised != hipSuccess) return raised;
    const I8Workspace w = i8_workspace(L, T);
    uint8_t* base = static_cast<uint8_t*>(ws);
    const int ks = dbf_row_tiles(L->k) * DBF_TILE_ROWS;
    const int kp1 = dbf_col_tiles(L->n_in) * DBF_TILE_COLS, kp2 = dbf_col_tiles(L->k) * DBF_TILE_COLS;
    float* mid = reinterpret_cast<float*>(base + w.mid);
    const bool forced = dbf_tune(DBF_TUNE_GEMM_SPLITS) > 0;   // (the knob names the kernels below)

    if (!forced && dbf_few_takes(L->plan, false, T)) {
        const hipError_t e = dbf_launch_few(L->plan, false, X_dev, Y_dev, mid, T, stream);
        if (e != hipSuccess) return e;
    } else {
        QuantArgs q1;
        q1.src = X_dev;  q1.col_scale = L->db;
        q1.dst = reinterpret_cast<signed char*>(base + w.xq1);
        q1.scale = reinterpret_cast<float*>(base + w.sc1);  q1.sigma = reinterpret_cast<int*>(base + w.sg1);
        q1.T = T;  q1.Tp = (T + 63) & ~63;  q1.cols = L->n_in;  q1.kp = kp1;  q1.ld = L->n_in;
        q1.vec_ok = ((L->n_in & 7) == 0 && (reinterpret_cast<uintptr_t>(X_dev) & 15) == 0) ? 1 : 0;
        launch_quantise<false>(q1, kp1, T, stream);
        StageArgs s1;
        s1.bits = L->dB;  s1.row_scale = L->dm;
        s1.xq = q1.dst;  s1.scale = q1.scale;  s1.sigma = q1.sigma;
        s1.out = mid;
        s1.n_rt = dbf_row_tiles(L->k);  s1.n_ct = dbf_col_tiles(L->n_in);  s1.T = T;  s1.Tp = q1.Tp;  s1.ldo = ks;
        s1.n_valid = ks;  // padded rows have m = 0 and are written as zeros: the second quantisation reads them
        launch_stage<true>(s1, stream);
    }
    if (!forced && dbf_few_takes(L->plan, true, T)) {
        const hipError_t e = dbf_launch_few(L->plan, true, X_dev, Y_dev, mid, T, stream);
        if (e != hipSuccess) return e;
    } else {
        QuantArgs q2;
        q2.src = mid;  q2.col_scale = nullptr;
        q2.dst = reinterpret_cast<signed char*>(base + w.xq2);
        q2.scale = reinterpret_cast<float*>(base + w.sc2);  q2.sigma = reinterpret_cast<int*>(base + w.sg2);
        q2.T = T;  q2.Tp = (T + 63) & ~63;  q2.cols = kp2 < ks ? kp2 : ks;  q2.kp = kp2;  q2.ld = ks;
        q2.vec_ok = 1;
        launch_quantise<true>(q2, kp2, T, stream);
        StageArgs s2;
        s2.bits = L->dA;  s2.row_scale = L->da;
        s2.xq = q2.dst;  s2.scale = q2.scale;  s2.sigma = q2.sigma;
        s2.out = Y_dev;
        s2.n_rt = dbf_row_tiles(L->n_out);  s2.n_ct = dbf_col_tiles(L->k);  s2.T = T;  s2.Tp = q2.Tp;  s2.ldo = L->n_out;
        s2.n_valid = L->n_out;
        launch_stage<false>(s2, stream);
    }
    return hipGetLastError();
}
