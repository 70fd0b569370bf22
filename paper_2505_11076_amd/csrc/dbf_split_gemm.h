// fp32 contractions on the bf16 matrix cores, for the ADMM kernels (dbf_admm.hip): out = P^T Q in fp32 accuracy.
//
// An fp32 value is the sum of three bf16 values, x = h + m + l, each the rounded rest of the ones before it (8 + 8 + 8
// significant bits: the sum is exact unless l falls below the smallest bf16).  A product of two such sums is taken as the
// six partial products h h, h m, m h, m m, h l, l h; what is left out (m l, l m, l l) is below 2^-26 of the product, a
// quarter of fp32's own rounding.  Products of two bf16 are exact in the matrix cores, sums are kept in fp32.  An operand that
// is a matrix of signs is one bf16 plane of +-1, and three products suffice.
//
// Why: v_mfma_f32_32x32x16_bf16 does 16 k in 8 passes where v_mfma_f32_32x32x2_f32 does 2 k in 16: six of the former per
// 16 k are 2.7 times as fast, three 5.3 times.
#ifndef DBF_SPLIT_GEMM_H
#define DBF_SPLIT_GEMM_H

#include "dbf_kernels.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------------------------
// Operand planes.  The operand element (k, i) -- summation index k, output index i -- lives in a fragment of 16 k by 32 i, the
// operand of one matrix instruction: lane l of a wavefront holds i = l % 32, k = 8 (l / 32) .. + 7, 16 bytes, 1 KiB in all.
// Order in memory: [i / 128][k / 16][piece][(i / 32) % 4][lane][8], so that what a workgroup of 128 outputs stages per step is
// one contiguous run, every load and LDS access of it is 16 bytes per lane in lane order, and no operand is transposed
// anywhere but in the kernels below, which make the planes.  Zeros beyond K and beyond M.
// ---------------------------------------------------------------------------------------------
constexpr int SG_FRAG = 1024;                 // bytes of a fragment
inline size_t sg_plane_bytes(int pieces, size_t K, size_t M) {
    return ((M + 127) / 128) * ((K + 15) / 16) * (size_t)pieces * 4 * SG_FRAG;
}

// h, m, l of eight values
__device__ inline void sg_split8(const float (&x)[8], v8bf& h, v8bf& m, v8bf& l) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        h[e] = (__bf16)x[e];
        const float r1 = x[e] - (float)h[e];
        m[e] = (__bf16)r1;
        l[e] = (__bf16)(r1 - (float)m[e]);
    }
}

// Where a wavefront of the plane kernels works: fragment (ib, kb) of a grid of (ceil(K / 16) / 4) x 4 ceil(M / 128) workgroups.
struct SgSite {
    int i, k0;       // this lane's output index and first k
    bool live;       // the wavefront has a fragment
    size_t off;      // byte offset of the lane's 16 bytes in piece 0 (pieces are 4 fragments apart)
};
__device__ inline SgSite sg_site(int K, int pieces) {
    const int lane = threadIdx.x & 63, n_kb = (K + 15) / 16;
    const int kb = blockIdx.x * 4 + (threadIdx.x >> 6), ib = blockIdx.y;
    SgSite s;
    s.live = kb < n_kb;
    s.i = 32 * ib + (lane & 31);
    s.k0 = 16 * kb + 8 * (lane >> 5);
    s.off = (((size_t)(ib >> 2) * n_kb + kb) * (4 * pieces) + (ib & 3)) * SG_FRAG + lane * 16;
    return s;
}
inline dim3 sg_plane_grid(int K, int M) { return dim3(((K + 15) / 16 + 3) / 4, 4 * ((M + 127) / 128)); }

__device__ inline void sg_store3(uint8_t* planes, size_t off, const float (&x)[8]) {
    v8bf h, m, l;
    sg_split8(x, h, m, l);
    *reinterpret_cast<v8bf*>(planes + off) = h;
    *reinterpret_cast<v8bf*>(planes + off + 4 * SG_FRAG) = m;
    *reinterpret_cast<v8bf*>(planes + off + 8 * SG_FRAG) = l;
}

// Planes of a dense k-major matrix src [K][ld >= M], its rows scaled by kscale (or NULL).  A wavefront's load of one k is two
// runs of 128 bytes.  Bound by memory: 4 bytes read and 6 written per element.
__global__ __launch_bounds__(256) void dbf_split_dense_kernel(const float* __restrict__ src, size_t ld, int K, int M,
                                                             const float* __restrict__ kscale, uint8_t* __restrict__ planes) {
    const SgSite s = sg_site(K, 3);
    if (!s.live) return;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = min(s.k0 + e, K - 1), i = min(s.i, M - 1);   // (clamped, not branched around: eight loads in flight)
        const float v = src[(size_t)k * ld + i] * (kscale ? kscale[k] : 1.f);
        x[e] = (s.k0 + e < K && s.i < M) ? v : 0.f;
    }
    sg_store3(planes, s.off, x);
}

// Planes of a packed sign matrix S (rows = output index i, columns = k) in the 128 x 64 tile layout.  SCALED: three planes of
// +-kscale[k]^2; else one plane of +-1.  A lane's eight signs are bit (i % 128) / 16 of eight consecutive bytes.
template <bool SCALED>
__global__ __launch_bounds__(256) void dbf_split_signs_kernel(const uint8_t* __restrict__ bits, int n_ct, int K, int M,
                                                             const float* __restrict__ kscale, uint8_t* __restrict__ planes) {
    const SgSite s = sg_site(K, SCALED ? 3 : 1);
    if (!s.live) return;
    const int i = min(s.i, (M + 127) / 128 * 128 - 1), ir = i & 127;
    const uint2 b = *reinterpret_cast<const uint2*>(bits + ((size_t)(i >> 7) * n_ct + (s.k0 >> 6)) * DBF_TILE_BYTES +
                                                    256 * ((s.k0 >> 4) & 3) + 16 * (ir & 15) + (s.k0 & 15));
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned bit = ((e < 4 ? b.x : b.y) >> (8 * (e & 3) + (ir >> 4))) & 1u;
        float v = 1.f;
        if (SCALED) {
            const float c = kscale[min(s.k0 + e, K - 1)];
            v = c * c;
        }
        x[e] = (s.k0 + e < K && s.i < M) ? (bit ? v : -v) : 0.f;
    }
    if (SCALED) {
        sg_store3(planes, s.off, x);
    } else {
        v8bf h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (__bf16)x[e];
        *reinterpret_cast<v8bf*>(planes + s.off) = h;
    }
}

// ---------------------------------------------------------------------------------------------
// out[i][j] = rs[i] * cs[j] * sum_k P[k][i] Q[k][j] + add[i][j] + (i == j ? diag : 0)
// from the planes of P (PA = 3 pieces, or 1: signs) and Q (3 pieces).  Workgroup = 128 x 128 outputs, 4 wavefronts of 64 x 64
// (2 x 2 blocks of 32 x 32: 64 accumulator registers), 16 values of k per step: 24 matrix instructions of 32 cycles per wavefront
// (12 with PA = 1) against 12 (8) LDS reads of 1 KiB, a step's 24 (16) KiB double buffered in LDS and requested two steps ahead into
// registers, one barrier per step; two workgroups per compute unit cover each other's barriers.  Workgroups are renumbered so that a
// compute die (linear id modulo 8) works on neighbouring column blocks: the Q planes it needs stay in its own L2.
// ---------------------------------------------------------------------------------------------
struct SplitGemmArgs {
    const uint8_t* P;
    const uint8_t* Q;
    const float* add;      // [M][N] with leading dimension lda, or NULL
    const float* rs;       // [M] or NULL
    const float* cs;       // [N] or NULL
    float* out;            // [M][N], leading dimension ldo
    size_t lda, ldo;
    float diag;
    int M, N, K;
    int upper;             // symmetric output: workgroups whose block lies wholly below the diagonal do nothing
    int ktri;              // both operands are zero for k < output index: sums start at the first k that can contribute
};

// The products of a workgroup's 128 x 128 block: acc (2 x 2 blocks of 32 x 32 per wavefront, rows from 64 (w % 2), columns from
// 64 (w / 2)) = sum over `steps` fragments of 16 k from pp (P's planes) and qp (Q's).  `meanwhile` runs once the first loads
// are on their way.  Ends with a barrier behind the last read of `lds`.
template <int PA, class F>
__device__ inline void split_gemm_tile(uint8_t (*lds)[(4 * PA + 12) * SG_FRAG], const uint8_t* pp, const uint8_t* qp, int steps, v16f (&acc)[2][2],
                                       F meanwhile) {
    constexpr int PB = 4 * PA * SG_FRAG, QB = 12 * SG_FRAG;   // bytes per step
    constexpr int NF = (PB + QB) / 4096;                      // 16-byte pieces a thread stages per step
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    pp += 16 * tid;
    qp += 16 * tid;
    v4f st[NF];
    auto fetch = [&](int s) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
            st[f] = f < PA ? *reinterpret_cast<const v4f*>(pp + (size_t)s * PB + 4096 * f)
                           : *reinterpret_cast<const v4f*>(qp + (size_t)s * QB + 4096 * (f - PA));
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int f = 0; f < NF; ++f) *reinterpret_cast<v4f*>(&lds[buf][4096 * f + 16 * tid]) = st[f];
    };
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bi][bj][v] = 0.f;
    const int fi = 2 * (w & 1), fj = 2 * (w >> 1);            // this wavefront's first 32-blocks
    auto multiply = [&](int buf) {
        const uint8_t* base = &lds[buf][16 * lane];
        v8bf a[2][PA], b[2][3];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int p = 0; p < PA; ++p) a[x][p] = *reinterpret_cast<const v8bf*>(base + (4 * p + fi + x) * SG_FRAG);
#pragma unroll
            for (int p = 0; p < 3; ++p) b[x][p] = *reinterpret_cast<const v8bf*>(base + PB + (4 * p + fj + x) * SG_FRAG);
        }
        // (piece pairs outermost: an accumulator is used again only after the three others)
#pragma unroll
        for (int p = PA - 1; p >= 0; --p)
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                if (p + q > 2) continue;
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int bj = 0; bj < 2; ++bj)
                        acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[bi][p], b[bj][q], acc[bi][bj], 0, 0, 0);
            }
    };
    if (steps <= 0) return;
    fetch(0);
    stage(0);
    if (steps > 1) fetch(1);
    meanwhile();
    __syncthreads();
    for (int s = 0; s < steps; ++s) {
        if (s + 1 < steps) stage((s & 1) ^ 1);
        if (s + 2 < steps) fetch(s + 2);
        multiply(s & 1);
        __syncthreads();
    }
}

template <int PA>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_split_gemm_kernel(const SplitGemmArgs g) {
    constexpr int PB = 4 * PA * SG_FRAG, QB = 12 * SG_FRAG;   // bytes per step
    __shared__ __align__(16) uint8_t lds[2][PB + QB];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned n_wg = gridDim.x * gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
    const unsigned die = lin & 7, slot = lin >> 3, per = n_wg >> 3, extra = n_wg & 7;
    const unsigned vid = die * per + (die < extra ? die : extra) + slot;
    const int it = (int)(vid % gridDim.x), jt = (int)(vid / gridDim.x);
    if (g.upper && it > jt) return;
    const int n_kb = (g.K + 15) / 16;
    const int kb0 = g.ktri ? min(8 * max(it, jt), n_kb) : 0;
    const int fi = 2 * (w & 1), fj = 2 * (w >> 1);
    v16f acc[2][2];
    split_gemm_tile<PA>(lds, g.P + ((size_t)it * n_kb + kb0) * PB, g.Q + ((size_t)jt * n_kb + kb0) * QB, n_kb - kb0, acc, []() {});
    // register v of lane l of a 32 x 32 block is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
    const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            const int col = 128 * jt + 32 * (fj + bj) + l32;
            if (col >= g.N) continue;
            const float csj = g.cs ? g.cs[col] : 1.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 128 * it + 32 * (fi + bi) + 8 * (v >> 2) + 4 * h + (v & 3);
                if (row < g.M) {
                    float val = acc[bi][bj][v] * csj;
                    if (g.rs) val *= g.rs[row];
                    if (g.add) val += g.add[(size_t)row * g.lda + col];
                    if (row == col) val += g.diag;
                    g.out[(size_t)row * g.ldo + col] = val;
                }
            }
        }
}

template <int PA>
inline void launch_split_gemm(const SplitGemmArgs& g, hipStream_t st) {
    hipLaunchKernelGGL((dbf_split_gemm_kernel<PA>), dim3((g.M + 127) / 128, (g.N + 127) / 128), dim3(256), 0, st, g);
}

}  // namespace
#endif
