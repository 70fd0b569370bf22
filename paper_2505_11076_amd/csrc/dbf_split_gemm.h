// fp32 contractions on the fp16 matrix cores, for the ADMM kernels (dbf_admm.hip): out = P^T Q in fp32 accuracy.
//
// An fp32 value is taken as (h + l / 2048) 2^e: h the fp16 value nearest to x 2^-e, l the fp16 value nearest to 2048 times the rest.  e belongs
// to an output line of an operand and a chunk of 128 summation indices: it puts the largest magnitude of those 128 values into
// [2^14, 2^15).  (Minv has a factor in place of 2^e that makes it 2^15: sg_scale_largest.)  h and l have 22 significant bits and a sign between them: x is met
// to 2^-23 of itself, 2^-24.5 on average, down to 2^-27 of the chunk's largest, and smaller values to 2^-50 of that one.  A product of two such values is taken as
// h h + (h l + l h) / 2048, the two in sums of their own; l l, left out, is at most 2^-22 of the product (2^-24.5 on average), of either sign, but never
// negative where a line meets itself (the diagonal of Y^T Y).  Products of two fp16 are exact in the matrix cores, the
// sums of a chunk are kept in fp32, 16 products entering a sum at once, and are scaled and added to the total chunk by chunk.
// An operand that is a matrix of signs is one fp16 plane of +-1, and two products suffice.
//
// Why: v_mfma_f32_32x32x16_f16 does 16 k in 8 passes where v_mfma_f32_32x32x2_f32 does 2 k in 16; three of the former per 16 k
// are half of what three bf16 parts per value need (six products, of 8 significant bits a part).
#ifndef DBF_SPLIT_GEMM_H
#define DBF_SPLIT_GEMM_H

#include "dbf_kernels.h"

#include <algorithm>

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------------------
// Operand planes.  The operand element (k, i) -- summation index k, output index i -- lives in a fragment of 16 k by 32 i, the
// operand of one matrix instruction: lane l of a wavefront holds i = l % 32, k = 8 (l / 32) .. + 7, 16 bytes, 1 KiB in all.
// Order in memory: [i / 128][k / 16][piece][(i / 32) % 4][lane][8], so that what a workgroup of 128 outputs stages per step is
// one contiguous run, every load and LDS access of it is 16 bytes per lane in lane order, and no operand is transposed
// anywhere but in the kernels below, which make the planes.  Zeros beyond K (up to whole chunks) and beyond M.  Behind the planes of a
// two-piece operand the 2^e: [k / 128][M rounded up to 128].
// ---------------------------------------------------------------------------------------------
constexpr int SG_FRAG = 1024;                 // bytes of a fragment
constexpr float SG_LOW = 2048.f;              // what l is scaled by
constexpr int SG_STEP = 16;                   // summation indices per step of the contraction
constexpr int SG_CHUNK = 128;                 // summation indices that share a line's scale
constexpr int SG_CHUNK_STEPS = SG_CHUNK / SG_STEP;
__host__ __device__ inline int sg_kblocks(int K) { return (K + SG_CHUNK - 1) / SG_CHUNK * (SG_CHUNK / 16); }
__host__ __device__ inline int sg_lines(int M) { return (M + 127) & ~127; }
__host__ __device__ inline size_t sg_scales_at(int pieces, int K, int M) { return (size_t)(sg_lines(M) >> 7) * sg_kblocks(K) * pieces * 4 * SG_FRAG; }
inline size_t sg_plane_bytes(int pieces, int K, int M) {
    return sg_scales_at(pieces, K, M) + (pieces == 1 ? 0 : sizeof(float) * (size_t)((K + SG_CHUNK - 1) / SG_CHUNK) * sg_lines(M));
}

// 2^-e and 2^e for a line's chunk whose largest magnitude is mx.  (Chunks of tiny values are not brought all the way up, so that both are
// normal numbers: h + l is then exact below 2^-126.  Infinities: any scale does, their products are not numbers.)
struct SgScale {
    float down, up;
};
__device__ __forceinline__ SgScale sg_scale(float mx) {
    const int e = (int)(__builtin_bit_cast(unsigned, mx) >> 23);              // (mx >= 0: its biased exponent)
    const int b = min(max(e, 15), 254) - 14;                                  // biased exponent of `up`: 1 .. 240
    SgScale s;
    s.up = __builtin_bit_cast(float, (unsigned)b << 23);
    s.down = __builtin_bit_cast(float, (unsigned)(254 - b) << 23);
    return s;
}

// The same, but no power of two: up = mx / 2^15, so that the largest value is met exactly, h = 2^15 and l = 0 (a power of two where that would be below
// 2^-115, which is enough for subnormal numbers).  For Minv, whose diagonal outweighs the rest of a line: an error of that entry would be common to a
// whole row of the result, and the row's factor keeps all of it (deviation of the factor from 64 bits, over sizes: 7.0e-8 with a power of two, 5.4e-8 so;
// three bf16 parts left 5.5e-8).
__device__ __forceinline__ SgScale sg_scale_largest(float mx) {
    SgScale s;
    s.up = fmaxf(mx * 0x1p-15f, 0x1p-115f);
    s.down = __builtin_amdgcn_rcpf(s.up);   // (need not be exact)
    return s;
}

// The two pieces of eight values to a fragment of piece 0 (`at`) and, NEXT bytes on, of piece 1.  (LARGEST: a scale that is no power of two; the rest is taken
// before it is scaled, so that only the rounding of l remains.)
template <bool LARGEST = false, int NEXT = 4 * SG_FRAG>
__device__ __forceinline__ void sg_store2(uint8_t* at, const float (&x)[8], const SgScale& c) {
    v8h h, l;
    if (LARGEST) {
        const float low = c.down * SG_LOW;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = x[e] * c.down;
            asm("" : "+v"(v));   // (one value: the compiler rounds the product for h and for its use below by different instructions, once and twice)
            h[e] = (_Float16)v;
            l[e] = (_Float16)(fmaf(-(float)h[e], c.up, x[e]) * low);
        }
    } else {
        // (v SG_LOW - h SG_LOW: both exact, four instructions an element)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const float v[2] = {x[e] * c.down, x[e + 1] * c.down};
            v2h two = {(_Float16)v[0], (_Float16)v[1]};
            asm("" : "+v"(two));   // (or the compiler rounds it a second time for the rest)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                h[e + i] = two[i];
                l[e + i] = (_Float16)fmaf((float)two[i], -SG_LOW, v[i] * SG_LOW);
            }
        }
    }
    *reinterpret_cast<v8h*>(at) = h;
    *reinterpret_cast<v8h*>(at + NEXT) = l;
}

// The plane kernels: 256 threads have a chunk of 128 k and 32 lines, a wavefront two fragments of it.  (A workgroup of their own, blockIdx.x the chunk;
// or half of a larger one.)
struct SgSite {
    int i, k0[2];    // this lane's output index (of the ib-th 32) and the first k of its two fragments
    size_t off[2];   // byte offset of the lane's 16 bytes in piece 0 (pieces are 4 fragments apart)
};
__device__ inline SgSite sg_site(int K, int pieces, int ib, int chunk, int t) {
    const int lane = t & 63, n_kb = sg_kblocks(K);
    SgSite s;
    s.i = 32 * ib + (lane & 31);
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int kb = chunk * (SG_CHUNK / 16) + 2 * (t >> 6) + n;
        s.k0[n] = 16 * kb + 8 * (lane >> 5);
        s.off[n] = (((size_t)(ib >> 2) * n_kb + kb) * (4 * pieces) + (ib & 3)) * SG_FRAG + lane * 16;
    }
    return s;
}
__device__ inline SgSite sg_site(int K, int pieces, int ib) { return sg_site(K, pieces, ib, blockIdx.x, threadIdx.x); }
inline dim3 sg_plane_grid(int K, int M) { return dim3((K + SG_CHUNK - 1) / SG_CHUNK, sg_lines(M) / 32); }

// Scales the values of a workgroup's chunk and lines and stores their pieces and scales.  x: zero where k or i is out of range.
template <bool LARGEST = false>
__device__ __forceinline__ void sg_split_chunk(uint8_t* planes, int K, int M, const SgSite& s, const float (&x)[2][8], int chunk, int t, float (*part)[32]) {
    const int lane = t & 63, l32 = lane & 31, w = t >> 6;
    float mx = 0.f;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(x[n][e]));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (lane < 32) part[w][lane] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(part[0][l32], part[1][l32]), fmaxf(part[2][l32], part[3][l32]));
    const SgScale c = LARGEST ? sg_scale_largest(mx) : sg_scale(mx);
#pragma unroll
    for (int n = 0; n < 2; ++n)
        sg_store2<LARGEST>(planes + s.off[n], x[n], c);
    if (t < 32) reinterpret_cast<float*>(planes + sg_scales_at(2, K, M))[(size_t)chunk * sg_lines(M) + s.i] = c.up;
}
template <bool LARGEST = false>
__device__ __forceinline__ void sg_split_chunk(uint8_t* planes, int K, int M, const SgSite& s, const float (&x)[2][8]) {
    __shared__ float part[4][32];
    sg_split_chunk<LARGEST>(planes, K, M, s, x, blockIdx.x, threadIdx.x, part);
}

// Planes of a dense k-major matrix src [K][ld >= M], its rows scaled by kscale (or NULL).  A wavefront's load of one k is two
// runs of 128 bytes.  Bound by memory: 4 bytes read and 4 written per element.
template <bool LARGEST = false>
__device__ __forceinline__ void sg_split_dense(const float* __restrict__ src, size_t ld, int K, int M, const float* __restrict__ kscale,
                                               uint8_t* __restrict__ planes, int ib, int chunk, int t, float (*part)[32]) {
    const SgSite s = sg_site(K, 2, ib, chunk, t);
    float x[2][8];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(s.k0[n] + e, K - 1), i = min(s.i, M - 1);   // (clamped, not branched around: sixteen loads in flight)
            x[n][e] = src[(size_t)k * ld + i] * (kscale ? kscale[k] : 1.f);
        }
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            asm("" : "+v"(x[n][e]));   // (or the compiler puts each load behind a branch and waits for it)
            x[n][e] = (s.k0[n] + e < K && s.i < M) ? x[n][e] : 0.f;
        }
    sg_split_chunk<LARGEST>(planes, K, M, s, x, chunk, t, part);
}
// blockIdx.y: 32 lines.  (Those from `first` on.)
__global__ __launch_bounds__(256) void dbf_split_dense_kernel(const float* __restrict__ src, size_t ld, int K, int M, const float* __restrict__ kscale,
                                                             uint8_t* __restrict__ planes, int first) {
    __shared__ float part[4][32];
    sg_split_dense(src, ld, K, M, kscale, planes, first + blockIdx.y, blockIdx.x, threadIdx.x, part);
}

// Planes of a packed sign matrix S (rows = output index i, columns = k) in the 128 x 64 tile layout: `signs`, one plane of +-1, and `scaled`, two
// planes of +-kscale[k]^2.  A lane's eight signs are bit (i % 128) / 16 of eight consecutive bytes.  (One launch for both, which also clears
// *flag: as three they took 6.5, 9.3 and 5 us.)
__global__ __launch_bounds__(256) void dbf_split_signs_kernel(const uint8_t* __restrict__ bits, int n_ct, int K, int M,
                                                             const float* __restrict__ kscale, uint8_t* __restrict__ signs,
                                                             uint8_t* __restrict__ scaled, int* __restrict__ flag) {
    const SgSite s = sg_site(K, 2, blockIdx.y), s1 = sg_site(K, 1, blockIdx.y);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *flag = 0;
    const int i = min(s.i, sg_lines(M) - 1), ir = i & 127;
    float x[2][8];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int k0 = min(s.k0[n], 64 * n_ct - 8);   // (a fragment that does not exist reads the row's last columns)
        const unsigned* b = reinterpret_cast<const unsigned*>(bits + ((size_t)(i >> 7) * n_ct + (k0 >> 6)) * DBF_TILE_BYTES +
                                                              256 * ((k0 >> 4) & 3) + 16 * (ir & 15) + (k0 & 15));   // (a caller's: 4-byte aligned)
        const unsigned b0 = b[0], b1 = b[1];
        v8h h;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned bit = ((e < 4 ? b0 : b1) >> (8 * (e & 3) + (ir >> 4))) & 1u;
            const float c = kscale[min(s.k0[n] + e, K - 1)], sign = (s.k0[n] + e < K && s.i < M) ? (bit ? 1.f : -1.f) : 0.f;
            h[e] = (_Float16)sign;
            x[n][e] = sign != 0.f ? sign * (c * c) : 0.f;   // (a scale past the end may be no number)
        }
        *reinterpret_cast<v8h*>(signs + s1.off[n]) = h;
    }
    sg_split_chunk(scaled, K, M, s, x);
}

// ---------------------------------------------------------------------------------------------
// out[i][j] = sum_k P[k][i] Q[k][j] + add[i][j] from the planes of P (PA = 2 pieces) and Q (2 pieces), or, P being signs (PA = 1),
// rs[i] * cs[j] * sum_k P[k][i] Q[k][j] + (i == j ? diag : 0).  Workgroup = 128 x 128 outputs (BI = 2; BI = 1: 64 x 128), 4
// wavefronts of 64 x 64 (2 x 2 blocks of 32 x 32: 64 registers for each of the three sums; BI = 1: 32 x 64), 16 values of k per step:
// 12 matrix instructions of 32 cycles per wavefront (8 with PA = 1) against 8 (6) LDS reads of 1 KiB.  A step's 16 (12) KiB come straight
// from memory into one of four LDS buffers, three steps ahead (two where the next step's operands are read early: AHEAD), one barrier per step; two workgroups per compute unit cover each
// other's barriers.  A chunk's last products are made block by block, each block being scaled and added to the total while the next is multiplied.
// KS = 2: eight wavefronts, two such halves that take every other chunk and add up through LDS at the end.
// What bounds it: the matrix pipes, at the rate that a plain bf16 product of 8192^3 reaches on the same card (1.24 PFLOP/s).  2048 x 4096
// outputs, K = 2048 (PA = 2): through registers into two LDS buffers of 32 k 130 us, so 96 (1.07 PFLOP/s; without the LDS traffic and
// the loads 89); a workgroup of four wavefronts with 64 x 128 outputs each, 12 LDS reads per 24 instructions, 132.
// ---------------------------------------------------------------------------------------------
struct SplitGemmArgs {
    const uint8_t* P;
    const uint8_t* Q;
    const float* add;      // PA = 2: [M][N] with leading dimension lda, or NULL
    const float* rs;       // PA = 1: [M]
    const float* cs;       // PA = 1: [N], or NULL (and diag is 0)
    float* out;            // [M][N], leading dimension ldo
    size_t lda, ldo;
    float diag;
    int M, N, K;
    int upper;             // symmetric output (M = N): only the blocks that meet the upper triangle are made, a workgroup in x for each
    int ktri;              // (upper) both operands are zero for k < output index: sums start at the first chunk that can contribute; both triangles are written
    int vec;               // ktri: out may be written 16 bytes at a time
};

// One operand of a workgroup's block: its fragments from a chunk on, its lines' scales from that chunk on (two pieces).
struct SgOperand {
    const uint8_t* frags;
    const float* up;
    int lines;       // scales from one chunk to the next
};
__device__ inline SgOperand sg_operand(const uint8_t* planes, int pieces, int K, int M, int block, int chunk) {
    SgOperand o;
    o.frags = planes + ((size_t)block * sg_kblocks(K) + chunk * SG_CHUNK_STEPS) * (4 * pieces) * SG_FRAG;
    o.lines = sg_lines(M);
    o.up = reinterpret_cast<const float*>(planes + sg_scales_at(pieces, K, M)) + (size_t)chunk * o.lines + 128 * block;
    return o;
}

// The sums of a chunk reach 2^37: scaled by P's `up` (2^113 at most) and then by Q's they overflow where the result does not, from
// entries of P of 1e31 on.  So Q's goes first as far as it is below 1, then P's, then the rest of Q's: no product leaves the range at the top
// unless the result does.  What is lost at its bottom, 2^-150 times the scales that are still to come, is less than 2^-24 of the product of the
// lines' largest entries (down to entries of 2^-140).  (A multiplication more per sum and chunk: an update of 2048 x 4096 187.7 us, so 189.5.)
__device__ __forceinline__ float sg_scaled(float a, float l, float p_up, float q_below) { return fmaf(l, q_below / SG_LOW, a * q_below) * p_up; }

// 1 KiB of a wavefront, 16 bytes (or 256 bytes, 4) per lane in lane order, from memory into LDS.
typedef const __attribute__((address_space(1))) unsigned* SgGlobal;
typedef __attribute__((address_space(3))) unsigned* SgShared;
__device__ __forceinline__ void sg_load16_lds(const void* src, void* dst) { __builtin_amdgcn_global_load_lds((SgGlobal)src, (SgShared)dst, 16, 0, 0); }
__device__ __forceinline__ void sg_load4_lds(const void* src, void* dst) { __builtin_amdgcn_global_load_lds((SgGlobal)src, (SgShared)dst, 4, 0, 0); }
// Waits until at most LEFT of this wavefront's loads are under way and its LDS reads have arrived, then for the workgroup's other wavefronts.
// (The wait is the builtin one: the compiler counts with it and adds none of its own before the LDS reads of a buffer.)
template <int LEFT>
__device__ __forceinline__ void sg_barrier() {
    static_assert(LEFT < 16, "the low four bits of the count");
    __builtin_amdgcn_s_waitcnt(0x0070 | LEFT);   // vmcnt <= LEFT, lgkmcnt = 0
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Planes made beside a contraction whose blocks leave compute units idle, by workgroups of 512 threads behind those of the blocks: two times 32 lines of a chunk
// each, of `pairs` times 64 lines.
struct SplitBesideArgs {
    const float* src;
    const float* kscale;
    uint8_t* planes;
    size_t ld;
    int K, M, pairs;
};

template <int PA, int BI, int KS, bool BESIDE>
__global__ __launch_bounds__(256 * KS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_split_gemm_kernel(const SplitGemmArgs g, const SplitBesideArgs d) {
    // slots of P and of Q in a buffer; P's loads per wavefront and step (BI = 1, PA = 1: two of its four slots are copies), all of them
    constexpr int NP = BI * PA < 2 ? 4 : 2 * BI * PA, NF = NP + 8, PL = NP / 4, PER = PL + 2;
    constexpr bool AHEAD = KS == 1 && PA == 2;
    constexpr int BUF = NF * SG_FRAG, SUMS = KS == 2 ? 2 * 256 * (int)sizeof(v16f) : 0;
    // (four objects: the compiler then knows that a load into one is not read from another)
    __shared__ __align__(16) uint8_t r0[KS * BUF > SUMS ? KS * BUF : SUMS], r1[KS * BUF], r2[KS * BUF], r3[KS * BUF];
    __shared__ __align__(16) float ups[KS][256];   // the scales of a chunk: P's 128 lines, then Q's
    if (BESIDE) {
        const int chunks = (d.K + SG_CHUNK - 1) / SG_CHUNK, index = (int)blockIdx.x - ((int)gridDim.x - chunks * d.pairs), half = threadIdx.x >> 8;
        if (index >= 0) {
            sg_split_dense(d.src, d.ld, d.K, d.M, d.kscale, d.planes, 2 * (index / chunks) + half, index % chunks, threadIdx.x & 255,
                           reinterpret_cast<float (*)[32]>(ups[0]) + 4 * half);
            return;
        }
    }
    const int tid = threadIdx.x & 255, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    // A compute die (linear id modulo 8) works on neighbouring blocks, eight rows of them at a time: what it reads of both operands stays
    // in its own L2.  (2048 x 4096 outputs: whole columns of blocks to a die 97 us, 8 x 8 blocks 92.)
    int it, jt;
    auto banded = [](unsigned lin, unsigned n_wg) {
        const unsigned die = lin & 7, slot = lin >> 3, per = n_wg >> 3, extra = n_wg & 7;
        return (int)(die * per + (die < extra ? die : extra) + slot);
    };
    if (g.upper) {
        // Column by column of the blocks that meet the upper triangle: (2 / BI) (jt + 1) of column jt.  Neighbours to a die here too (constants, p = r = 4096,
        // q = 2048 521 us / 513; 2048 x 900 x 6000 259.5 / 256.5), but where the sums shorten from column to column: one die would have the longest.
        auto before = [](int c) { return (2 / BI) * (c * (c + 1) / 2); };
        const int v = g.ktri ? (int)blockIdx.x : banded(blockIdx.x, before((g.N + 127) >> 7));
        jt = (int)((sqrtf(1.f + (float)(4 * BI) * (float)v) - 1.f) * 0.5f);
        while (before(jt) > v) --jt;
        while (before(jt + 1) <= v) ++jt;
        it = v - before(jt);
    } else {
        const int mt = gridDim.x, nt = gridDim.y;
        const int vid = banded(blockIdx.x + mt * blockIdx.y, mt * nt), band = vid / (8 * nt), in_band = vid - band * 8 * nt, rows = min(8, mt - 8 * band);
        it = 8 * band + in_band % rows;
        jt = in_band / rows;
    }
    const int row0 = 64 * BI * it;
    const int chunk0 = g.ktri ? min(max(row0, 128 * jt), g.K - 1) / SG_CHUNK : 0, chunks = (g.K + SG_CHUNK - 1) / SG_CHUNK - chunk0;
    const int half = (row0 >> 6) & (2 - BI);       // BI = 1: which 64 of P's 128 lines
    const SgOperand P = sg_operand(g.P, PA, g.K, g.M, row0 >> 7, chunk0), Q = sg_operand(g.Q, 2, g.K, g.N, jt, chunk0);

    // this half's i-th chunk is KS i + kg; past the last: that one again, not added to the total
    auto fetch = [&](uint8_t* buf, int i, int sub) {
        const int s = SG_CHUNK_STEPS * min(KS * i + kg, chunks - 1) + sub;
        const uint8_t *p = P.frags + (size_t)s * (4 * PA * SG_FRAG) + 16 * lane, *q = Q.frags + (size_t)s * (8 * SG_FRAG) + 16 * lane;
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            const int f = w + 4 * n;
            const uint8_t* src = n >= PL ? q + (f - NP) * SG_FRAG : BI == 2 ? p + f * SG_FRAG : p + (4 * (PA == 2 ? f >> 1 : 0) + 2 * half + (f & 1)) * SG_FRAG;
            sg_load16_lds(src, buf + kg * BUF + f * SG_FRAG);
        }
    };
    auto fetch_ups = [&](int i) {
        const int c = min(KS * i + kg, chunks - 1);
        sg_load4_lds((w < 2 && PA == 2 ? P.up + (size_t)c * P.lines : Q.up + (size_t)c * Q.lines) + (tid & 127), &ups[kg][64 * w]);
    };
    v16f acc[BI][2], low[BI][2], tot[BI][2];   // h h; h l and l h, times SG_LOW; all of the chunks before
#pragma unroll
    for (int bi = 0; bi < BI; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                tot[bi][bj][v] = 0.f;
                acc[bi][bj][v] = 0.f;
                low[bi][bj][v] = 0.f;
            }
    const int fi = BI * (w & 1), fj = 2 * (w >> 1);           // this wavefront's first 32-blocks
    v8h a[BI][PA], b[2][2];
    auto read_p = [&](const uint8_t* buf, int p) {
#pragma unroll
        for (int x = 0; x < BI; ++x) a[x][p] = *reinterpret_cast<const v8h*>(buf + kg * BUF + 16 * lane + (2 * BI * p + fi + x) * SG_FRAG);
    };
    auto read_q = [&](const uint8_t* buf, int p) {
#pragma unroll
        for (int x = 0; x < 2; ++x) b[x][p] = *reinterpret_cast<const v8h*>(buf + kg * BUF + 16 * lane + (NP + 4 * p + fj + x) * SG_FRAG);
    };
    auto product = [&](int bi, int bj, int p, int q) {
        v16f& sum = p + q == 0 ? acc[bi][bj] : low[bi][bj];
        sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[bi][p], b[bj][q], sum, 0, 0, 0);
    };
    // (piece pairs outermost: an accumulator is used again only after the others)
    auto multiply = [&](int p, int q) {
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) product(bi, bj, p, q);
        if (AHEAD) __builtin_amdgcn_sched_barrier(0);
    };
    // l l where the lines meet themselves: there it is of one sign, and lost from all of a diagonal
    const bool self = PA == 2 && BI == 1 && g.ktri && (row0 >> 7) == jt;
    auto multiply_self = [&]() {
        if (PA == 2 && BI == 1 && self) {
            const v8h s = a[0][PA - 1] * (_Float16)(1.f / SG_LOW);
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) low[0][bj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(s, b[bj][1], low[0][bj], 0, 0, 0);
        }
    };
    // A chunk's sums, scaled, to the total.  Register v of lane l of a 32 x 32 block is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.
    // (sg_scaled has the order of the scales)
    auto fold = [&](int bi, int bj) {
        const float* u = ups[kg];
        const float uq = u[128 + 32 * (fj + bj) + l32], below = uq < 1.f ? uq : 1.f, above = uq < 1.f ? 1.f : uq;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const v4f ur = PA == 1 ? (v4f){1.f, 1.f, 1.f, 1.f} : *reinterpret_cast<const v4f*>(u + 64 * half + 32 * (fi + bi) + 8 * c + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = acc[bi][bj][4 * c + e], l = low[bi][bj][4 * c + e];
                if (PA == 1) tot[bi][bj][4 * c + e] = fmaf(fmaf(l, 1.f / SG_LOW, a), uq, tot[bi][bj][4 * c + e]);
                else tot[bi][bj][4 * c + e] = fmaf(sg_scaled(a, l, ur[e], below), above, tot[bi][bj][4 * c + e]);
                acc[bi][bj][4 * c + e] = 0.f;
                low[bi][bj][4 * c + e] = 0.f;
            }
        }
    };
    auto read_early = [&](const uint8_t* buf) {
        read_p(buf, PA - 1);
        read_q(buf, 0);
    };
    auto multiply_last = [&](bool live, const uint8_t* next) {
#pragma unroll
        for (int n = 0; n <= 2 * BI; ++n) {
            if (n < 2 * BI) {
#pragma unroll
                for (int p = PA - 1; p >= 0; --p)
#pragma unroll
                    for (int q = 1 - p; q >= 0; --q) product(n >> 1, n & 1, p, q);
            }
            if (AHEAD && n == 2 * BI - 1) {
                read_early(next);
            }
            if (n > 0 && live) fold((n - 1) >> 1, (n - 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    static_assert(SG_CHUNK_STEPS == 8, "the buffers of a chunk's steps are written out below");
    uint8_t* const ring[4] = {r0, r1, r2, r3};
    fetch(r0, 0, 0);
    fetch(r1, 0, 1);
    fetch(r2, 0, 2);
    const int rounds = (chunks + KS - 1) / KS;
    // Two workgroups to a compute unit wait for each other's LDS reads (of 64 KiB a step for 24 products of a wavefront pair, what the matrix pipe takes): the
    // next step's l of P and h of Q are read as soon as this step's products with them are done.  An update of 2048 x 4096 178.6 / 176.0 us,
    // 3000 x 4000 324.2 / 316.8.  With KS = 2, a workgroup alone, the loads' third step of lead is worth more: 1024 x 4096 73.2 / 73.8,
    // as with signs in one piece, half of whose products could cover the reads: constants of 4096^3 1424 / 1441, 4096 x 2048 x 11008 826 / 841.
    if (AHEAD) {
        sg_barrier<2 * PER>();
        read_early(r0);
    }
    for (int i = 0; i < rounds; ++i) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // The loads of this step (AHEAD: and of the next) have arrived, those of the two after it (the one after them; and, of steps 0 and 1, the
            // scales) may not have; every wavefront is done with the step before, whose buffer the next loads take.
            constexpr int LEFT = (AHEAD ? 1 : 2) * PER;
            if (j == 1 || j == 2) sg_barrier<LEFT + 1>(); else sg_barrier<LEFT>();
            const uint8_t *const now = ring[j & 3], *const next = ring[(j + 1) & 3];
            if (!AHEAD) read_early(now);
            if (PA == 2) read_p(now, 0);
            read_q(now, 1);
            fetch(ring[(j + 3) & 3], i + (j + 3) / 8, (j + 3) & 7);
            if (j == 0) fetch_ups(i);
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
            multiply_self();
            if (j < 7) {
                if (PA == 2) multiply(PA - 1, 0);
                if (AHEAD) read_p(next, PA - 1);
                multiply(0, PA == 2 && !AHEAD ? 1 : 0);
                if (AHEAD) read_q(next, 0);
                multiply(0, PA == 2 && !AHEAD ? 0 : 1);
            } else {
                multiply_last(KS == 1 || KS * i + kg < chunks, next);
            }
        }
    }
    sg_barrier<0>();
    if (KS == 2) {
        v4f* sums = reinterpret_cast<v4f*>(r0);   // [2][4][256]: 16-byte pieces, thread by thread: no bank conflicts
#pragma unroll
        for (int bi = 0; bi < BI; ++bi) {
            if (bi > 0) __syncthreads();
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (kg == 1)
                        sums[(bj * 4 + c) * 256 + tid] = (v4f){tot[bi][bj][4 * c], tot[bi][bj][4 * c + 1], tot[bi][bj][4 * c + 2], tot[bi][bj][4 * c + 3]};
            __syncthreads();
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const v4f o = sums[(bj * 4 + c) * 256 + tid];
#pragma unroll
                    for (int e = 0; e < 4; ++e) tot[bi][bj][4 * c + e] += o[e];
                }
        }
        if (kg == 1) return;
    }
    // (what is added is loaded for all of the block at once, clamped, not branched around)
    auto row_of = [&](int bi, int v) { return row0 + 32 * (fi + bi) + 8 * (v >> 2) + 4 * h + (v & 3); };
    float rs[BI][16];
    if (PA == 1) {
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int v = 0; v < 16; ++v) rs[bi][v] = g.rs[min(row_of(bi, v), g.M - 1)];
    }
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
        const int col = 128 * jt + 32 * (fj + bj) + l32, cc = min(col, g.N - 1);
        const double cs = PA == 1 && g.cs ? g.cs[cc] : 1.;
        float add[BI][16];
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int v = 0; v < 16; ++v) add[bi][v] = 0.f;
        if (PA == 2 && g.add) {
#pragma unroll
            for (int bi = 0; bi < BI; ++bi)
#pragma unroll
                for (int v = 0; v < 16; ++v) add[bi][v] = g.add[(size_t)min(row_of(bi, v), g.M - 1) * g.lda + cc];
        }
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = row_of(bi, v);
                // (two factors and the diagonal: rounded once, in 64 bits; G's error is common to all that follows.  Minv, means over ten
                // sizes: 2.25e-7, so 2.22e-7)
                float val = tot[bi][bj][v] + add[bi][v];
                if (PA == 1) val = g.cs ? (float)fma((double)tot[bi][bj][v] * (double)rs[bi][v], cs, row == col ? (double)g.diag : 0.) : tot[bi][bj][v] * rs[bi][v];
                if (PA == 2 && BI == 1 && g.ktri) {
                    // (symmetric, both triangles written: a block on the diagonal from its upper half, so that they are the same bits)
                    tot[bi][bj][v] = val;
                    if ((!self || row <= col) && row < g.M && col < g.N) g.out[(size_t)row * g.ldo + col] = val;
                } else if (row < g.M && col < g.N) {
                    g.out[(size_t)row * g.ldo + col] = val;
                }
            }
        if (PA == 2 && BI == 1 && g.ktri && col < g.N) {
            float* const line = g.out + (size_t)col * g.ldo;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int row = row_of(0, 4 * c);   // and the three behind it: 16 bytes of a line
                const v4f x = {tot[0][bj][4 * c], tot[0][bj][4 * c + 1], tot[0][bj][4 * c + 2], tot[0][bj][4 * c + 3]};
                if (g.vec && (!self || row + 3 < col)) {
                    if (row < g.M) *reinterpret_cast<v4f*>(line + row) = x;   // (M is a multiple of 4)
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (row + e < g.M && (!self || row + e < col)) line[row + e] = x[e];
                }
            }
        }
    }
}

// Where blocks of 128 x 128 would not put two workgroups on every compute unit, a lone one waits out its barriers and LDS latencies:
// the chunks are shared by two halves of a workgroup of 512; and the blocks are 64 x 128 where those of 128 x 128 would leave half of
// the compute units idle.  us, 64 x 128 with 512 threads / 128 x 128 with 512 / with 256 (K = M):  512 x 768 outputs (24 blocks) 12.2 / 17.9 / 19.2,
// 1024 x 2048 (128) 20.2 / 27.5 / 30.1, 1536 x 1536 (144) 44.7 / 36.2 / 40.7, 2048 x 2048 (256) 62.1 / 55.2 / 57.8, 1792 x 2560 (280) 77.6 / 84.1 / 67.6,
// 2415 x 2816 (418) 137 / 115 / 102.
// Sums of unequal lengths (ktri) go best in 64 x 128 at every size: short ones end early.  With 512 threads until the blocks keep the chip busy by
// themselves.  us, the constants (p = r = 768), 64 x 128 with 512 threads / with 256 / 128 x 128 with 512 / with 256: q = 1536 (78 blocks) 417 / 424 / 432 / 440,
// 2048 (136) 557 / 562 / 570 / 582, 2560 (210) 703 / 711 / 718 / 732, 2944 (276) 811 / 816 / 826 / 842, 3328 (351) 940 / 939 / 949 / 969,
// 3712 (435) 1063 / 1054 / 1062 / 1085, 4096 (528) 1166 / 1149 / 1155 / 1180.
// (`columns`: only the first so many blocks of each row.  `beside`: planes to be made by further workgroups, where there are idle compute units for them; returns
// how many times 64 lines are.)
template <int PA>
inline int launch_split_gemm(const SplitGemmArgs& g, hipStream_t st, int columns = 1 << 30, const SplitBesideArgs* beside = nullptr) {
    const int mt = (g.M + 127) / 128, all = (g.N + 127) / 128, nt = columns < all ? columns : all;
    const long long blocks = g.upper ? (long long)mt * (mt + 1) / 2 : (long long)mt * nt;
    auto grid = [&](int bi) { return g.upper ? dim3((unsigned)(blocks * (2 / bi))) : dim3(bi == 2 ? mt : (g.M + 63) / 64, nt); };
    SplitBesideArgs d = {};
    auto more = [&](dim3 of) {   // (blocks in x alone)
        const long long chunks = (beside->K + SG_CHUNK - 1) / SG_CHUNK, most = sg_lines(beside->M) / 64;
        d = *beside;
        d.pairs = 0;
        // (as many as an idle compute unit makes in the contraction's time: 2 us a chunk here, 3 a workgroup there.  The constants, us, none / so / twice that: 4096, 2048,
        // 4096 539 / 527 / 529; 768, 600, 768 153.0 / 149.7 / 149.8; 4096, 512, 4096 179 / 168 / 168; 11008, 1500, 4096 696 / 703 / 705, where the contraction waits for memory itself)
        if (g.K <= 8192) d.pairs = (int)std::min(most, std::max(0ll, 256 - (long long)of.x) * ((g.K + SG_CHUNK - 1) / SG_CHUNK) * 2 / 3 / chunks);
        return dim3((unsigned)(of.x + chunks * d.pairs));
    };
    if (blocks <= 128 || (g.ktri && blocks <= 320)) {
        if (PA == 1 && beside) hipLaunchKernelGGL((dbf_split_gemm_kernel<1, 1, 2, true>), more(grid(1)), dim3(512), 0, st, g, d);
        else hipLaunchKernelGGL((dbf_split_gemm_kernel<PA, 1, 2, false>), grid(1), dim3(512), 0, st, g, d);
    } else if (PA == 2 && g.ktri) {   // (Y^T Y alone)
        hipLaunchKernelGGL((dbf_split_gemm_kernel<2, 1, 1, false>), grid(1), dim3(256), 0, st, g, d);
    } else if (blocks <= 256) {
        if (PA == 1 && beside) hipLaunchKernelGGL((dbf_split_gemm_kernel<1, 2, 2, true>), more(grid(2)), dim3(512), 0, st, g, d);
        else hipLaunchKernelGGL((dbf_split_gemm_kernel<PA, 2, 2, false>), grid(2), dim3(512), 0, st, g, d);
    } else {
        hipLaunchKernelGGL((dbf_split_gemm_kernel<PA, 2, 1, false>), grid(2), dim3(256), 0, st, g, d);
    }
    return d.pairs;
}

}  // namespace
#endif
