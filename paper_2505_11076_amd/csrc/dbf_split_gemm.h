// fp32 contractions on the bf16 matrix cores, for the ADMM kernels (dbf_admm.hip): out = P^T Q in fp32 accuracy.
//
// An fp32 value is the sum of three bf16 values, x = h + m + l, each the rounded rest of the ones before it (8 + 8 + 8
// significant bits: the sum is exact unless l falls below the smallest bf16, for |x| below about 1e-33).  A product of two such
// sums is taken as the six partial products h h, h m, m h, m m, h l, l h; what is left out (m l, l m, l l) is at most about 2^-24
// of the product, fp32's own unit roundoff (|m| reaches 2^-8 and |l| 2^-17 of x; 2^-28 on average), of either sign.  Products of two
// bf16 are exact in the matrix cores, sums are kept in fp32, 16 products entering a sum at once: measured against 64 bits the
// contractions are closer than on the fp32 matrix instructions (dbf_admm.hip).  An operand that is a matrix of signs is one bf16
// plane of +-1, and three products suffice.
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
    const unsigned* b = reinterpret_cast<const unsigned*>(bits + ((size_t)(i >> 7) * n_ct + (s.k0 >> 6)) * DBF_TILE_BYTES +
                                                          256 * ((s.k0 >> 4) & 3) + 16 * (ir & 15) + (s.k0 & 15));   // (a caller's: 4-byte aligned)
    const unsigned b0 = b[0], b1 = b[1];
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned bit = ((e < 4 ? b0 : b1) >> (8 * (e & 3) + (ir >> 4))) & 1u;
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
// from the planes of P (PA = 3 pieces, or 1: signs) and Q (3 pieces).  Workgroup = 128 x 128 outputs (BI = 2; BI = 1: 64 x 128), 4
// wavefronts of 64 x 64 (2 x 2 blocks of 32 x 32: 64 accumulator registers; BI = 1: 32 x 64), 16 values of k per step: 24 matrix
// instructions of 32 cycles per wavefront (12 with PA = 1) against 12 (8) LDS reads of 1 KiB, a step's 24 (16) KiB double buffered in
// LDS and requested two steps ahead into registers, one barrier per step; two workgroups per compute unit cover each other's barriers.
// KS = 2: eight wavefronts, two such halves that take every other step and add up through LDS at the end.  Workgroups are renumbered so that a
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

// The products of a workgroup's block of 64 BI x 128: acc (BI x 2 blocks of 32 x 32 per wavefront, rows from 32 BI (w % 2), columns from
// 64 (w / 2)) = sum over `steps` fragments of 16 k from pp (P's planes; BI = 1: of rows 64 `half` .. of the 128) and qp (Q's).
// KS = 2: a workgroup of 512 threads, wavefronts 4-7 take every second step with LDS buffers of their own (lds: [KS][2][..]); their sums
// are added at the end, and only threads 0-255 have the result.
// `meanwhile` runs once the first loads are on their way.  Ends with a barrier behind the last read of `lds`.
template <int PA, int BI, int KS, class F>
__device__ inline void split_gemm_tile(uint8_t (*lds)[(2 * BI * PA + 12) * SG_FRAG], const uint8_t* pp, const uint8_t* qp, int half, int all_steps,
                                       v16f (&acc)[BI][2], F meanwhile) {
    constexpr int PB = 4 * PA * SG_FRAG, QB = 12 * SG_FRAG;   // bytes per step in memory
    constexpr int NP = 2 * BI * PA, NF = NP + 12, PER = (NF + 3) / 4;   // fragments per step; of a wavefront's to stage
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    const int steps = (all_steps - kg + KS - 1) / KS, rounds = (all_steps + KS - 1) / KS;   // this half's steps; barriers are everybody's
    uint8_t(*const first_lds)[(2 * BI * PA + 12) * SG_FRAG] = lds;
    lds += 2 * kg;
    v4f st[PER];
    auto fetch = [&](int i) {
        const int s = KS * i + kg;
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            const int f = w + 4 * n;
            const uint8_t* src = f < NP ? pp + (size_t)s * PB + (4 * (f / (2 * BI)) + 2 * half + f % (2 * BI)) * SG_FRAG
                                        : qp + (size_t)s * QB + (min(f, NF - 1) - NP) * SG_FRAG;
            st[n] = *reinterpret_cast<const v4f*>(src + 16 * lane);
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int n = 0; n < PER; ++n)
            if (NF % 4 == 0 || w + 4 * n < NF) *reinterpret_cast<v4f*>(&lds[buf][(w + 4 * n) * SG_FRAG + 16 * lane]) = st[n];
    };
#pragma unroll
    for (int bi = 0; bi < BI; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bi][bj][v] = 0.f;
    const int fi = BI * (w & 1), fj = 2 * (w >> 1);           // this wavefront's first 32-blocks
    auto multiply = [&](int buf) {
        const uint8_t* base = &lds[buf][16 * lane];
        v8bf a[BI][PA], b[2][3];
#pragma unroll
        for (int p = 0; p < PA; ++p)
#pragma unroll
            for (int x = 0; x < BI; ++x) a[x][p] = *reinterpret_cast<const v8bf*>(base + (2 * BI * p + fi + x) * SG_FRAG);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int x = 0; x < 2; ++x) b[x][p] = *reinterpret_cast<const v8bf*>(base + (NP + 4 * p + fj + x) * SG_FRAG);
        // (piece pairs outermost: an accumulator is used again only after the others)
#pragma unroll
        for (int p = PA - 1; p >= 0; --p)
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                if (p + q > 2) continue;
#pragma unroll
                for (int bi = 0; bi < BI; ++bi)
#pragma unroll
                    for (int bj = 0; bj < 2; ++bj)
                        acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[bi][p], b[bj][q], acc[bi][bj], 0, 0, 0);
            }
    };
    if (all_steps <= 0) return;
    if (steps > 0) {
        fetch(0);
        stage(0);
    }
    if (steps > 1) fetch(1);
    meanwhile();
    __syncthreads();
    for (int s = 0; s < rounds; ++s) {
        if (s + 1 < steps) stage((s & 1) ^ 1);
        if (s + 2 < steps) fetch(s + 2);
        if (KS == 1 || s < steps) multiply(s & 1);
        __syncthreads();
    }
    if (KS == 2) {
        v16f* sums = reinterpret_cast<v16f*>(first_lds);      // [BI][2][256]
        static_assert(KS == 1 || BI * 2 * 256 * sizeof(v16f) <= 4 * (2 * BI * PA + 12) * SG_FRAG, "the sums fit the buffers");
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                for (int c = 0; c < 4; ++c) {                 // (16-byte pieces, thread by thread: no bank conflicts)
                    v4f* at = reinterpret_cast<v4f*>(sums) + ((bi * 2 + bj) * 4 + c) * 256 + tid;
                    if (kg == 1) *at = (v4f){acc[bi][bj][4 * c], acc[bi][bj][4 * c + 1], acc[bi][bj][4 * c + 2], acc[bi][bj][4 * c + 3]};
                }
        __syncthreads();
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const v4f o = reinterpret_cast<const v4f*>(sums)[((bi * 2 + bj) * 4 + c) * 256 + tid];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[bi][bj][4 * c + e] += o[e];
                }
    }
}

template <int PA, int BI, int KS>
__global__ __launch_bounds__(256 * KS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_split_gemm_kernel(const SplitGemmArgs g) {
    constexpr int PB = 4 * PA * SG_FRAG, QB = 12 * SG_FRAG;   // bytes per step
    __shared__ __align__(16) uint8_t lds[2 * KS][(2 * BI * PA + 12) * SG_FRAG];
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned n_wg = gridDim.x * gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
    const unsigned die = lin & 7, slot = lin >> 3, per = n_wg >> 3, extra = n_wg & 7;
    const unsigned vid = die * per + (die < extra ? die : extra) + slot;
    const int it = (int)(vid % gridDim.x), jt = (int)(vid / gridDim.x), row0 = 64 * BI * it;
    if (g.upper && row0 >= 128 * (jt + 1)) return;
    const int n_kb = (g.K + 15) / 16;
    const int kb0 = g.ktri ? min(max(row0, 128 * jt) / 16, n_kb) : 0;
    const int fi = BI * (w & 1), fj = 2 * (w >> 1);
    v16f acc[BI][2];
    split_gemm_tile<PA, BI, KS>(lds, g.P + ((size_t)(row0 >> 7) * n_kb + kb0) * PB, g.Q + ((size_t)jt * n_kb + kb0) * QB, (row0 >> 6) & (2 - BI),
                                n_kb - kb0, acc, []() {});
    if (KS == 2 && threadIdx.x >= 256) return;
    // register v of lane l of a 32 x 32 block is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
    const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int bi = 0; bi < BI; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            const int col = 128 * jt + 32 * (fj + bj) + l32;
            if (col >= g.N) continue;
            const float csj = g.cs ? g.cs[col] : 1.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = row0 + 32 * (fi + bi) + 8 * (v >> 2) + 4 * h + (v & 3);
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

// Where blocks of 128 x 128 would not put two workgroups on every compute unit, a lone one waits out its barriers and LDS latencies:
// the steps are shared by two halves of a workgroup of 512; and the blocks are 64 x 128 where those of 128 x 128 would leave half of
// the compute units idle.  Whole calls, us, 128 x 128 with 256 threads / with 512 / 64 x 128 with 512: an update of q = 512, r = 768 (24 blocks)
// 87.6 / 88.4 / 68.4, 1024 x 1024 (64) 112.9 / 111.4 / 84.9, 1408 x 1269 (110) 147.3 / 144.0 / 112.1, 1536 x 2048 (192) 143.5 / 139.5 / 157.5,
// 2048 x 4096 (512) 272 / 312 / 357; the constants at p = 4096, q = 700, r = 1000 531 / 488 / 424.
template <int PA>
inline void launch_split_gemm(const SplitGemmArgs& g, hipStream_t st) {
    const int mt = (g.M + 127) / 128, nt = (g.N + 127) / 128;
    const long long blocks = g.upper ? (long long)mt * (mt + 1) / 2 : (long long)mt * nt;
    if (blocks <= 128)
        hipLaunchKernelGGL((dbf_split_gemm_kernel<PA, 1, 2>), dim3((g.M + 63) / 64, nt), dim3(512), 0, st, g);
    else if (blocks <= 256)
        hipLaunchKernelGGL((dbf_split_gemm_kernel<PA, 2, 2>), dim3(mt, nt), dim3(512), 0, st, g);
    else
        hipLaunchKernelGGL((dbf_split_gemm_kernel<PA, 2, 1>), dim3(mt, nt), dim3(256), 0, st, g);
}

}  // namespace
#endif
