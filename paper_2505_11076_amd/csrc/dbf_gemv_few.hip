// Decode launches of few workgroups: a layer alone or a handful of them at a batch of 2 and more, rows long enough to be
// cut into column pieces, prompts of a few dozen tokens, and layers so small that one workgroup does both stages.
//
// The arithmetic is that of dbf_gemv_mfma.hip (16-bit fixed-point stage inputs as two int8 planes, masked sign bytes as the
// other operand of v_mfma_i32_16x16x64_i8, exact integer sums), and so are the bits.  The split is another one, because such
// a launch is not bound by memory or by the matrix cores but by its chain of latencies:
//   * every workgroup rounds the rows of the stage input it needs itself.  A launch of its own for that costs 3.4-4.3 us,
//     as much as half of the stage; here it is 5 vector instructions per value beside the sign tiles' way from memory;
//   * a workgroup has eight wavefronts, each with eight tiles in flight from its first instructions on (64 KiB per workgroup;
//     four wavefronts with four tiles each held a compute unit that has one workgroup to 11 GB/s);
//   * where compute units would idle, the tokens of a call and the bit planes of a row tile are dealt to several workgroups (less
//     rounding and fewer matrix instructions in each, the sign bytes come from L2), and long rows are cut into column pieces.
// Measured figures are at the rules that cut and choose such launches (few_cut, few_split, dbf_few_takes, dbf_small_layer_kernel).
#include <type_traits>

#include "dbf_kernels.h"
#include "dbf_wave.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int FEW_WAVES = 8;
constexpr int FEW_THREADS = 64 * FEW_WAVES;
constexpr int FEW_PF = 8;            // tiles in flight per wavefront
constexpr int FEW_HELD = 12;         // vectors of eight input values a lane can hold (four rows of 12288; 10: 11008 -> 4096, k = 4477, batch 8 / 16 14.64 / 18.71 us, so 14.21 / 16.85)
constexpr int FEW_RB = DBF_TILE_ROWS + 1;  // LDS row of a reduction buffer (see RB_STRIDE in dbf_gemv_mfma.hip)
constexpr float QMAX = 32512.f;
constexpr unsigned OOB = 0x80000000u;

struct FewMisc {
    float scale[DBF_MAX_BATCH];
    int sigma[DBF_MAX_BATCH];
    float wmax[DBF_MAX_BATCH][FEW_WAVES];
    int last, pad_[3];
};
static_assert(sizeof(FewMisc) % 16 == 0, "the planes behind it are read in 16-byte pieces");

// LDS: FewMisc, the quantised planes tile by tile -- per column tile 64 bytes of plane 0 (row 0's high bytes), of plane 1
// (its low bytes), ..., 64 bytes of padding that spread the writes over the banks --, then the sums.
__host__ __device__ inline int few_tile_block(int ncols) { return (ncols + 1) * DBF_TILE_COLS; }

// How the eight wavefronts share the input rows: P rows at a time (a power of two), 8 / P wavefronts each.
struct FewShare {
    int P, parts, log_parts, row, part;
};
__host__ __device__ inline int few_log_parts(int nb) { return nb <= 1 ? 3 : nb <= 2 ? 2 : nb <= 4 ? 1 : 0; }
__host__ __device__ inline int few_parts(int nb) { return 1 << few_log_parts(nb); }
__device__ inline FewShare few_share(int nb, int w) {
    FewShare s;
    s.log_parts = few_log_parts(nb);
    s.parts = 1 << s.log_parts;
    s.P = FEW_WAVES >> s.log_parts;
    s.row = w & (s.P - 1);
    s.part = w >> (3 - s.log_parts);
    return s;
}
static_assert(FEW_WAVES == 8, "the shift by 3");

// The rows of a stage's input: fp16 x times b (B stage), or the fp32 middle activations, which are padded with zeros.  load()
// requests the eight values of vector v of a row, get() turns what has arrived into numbers.
// ANY: rows start at any even address and have any number of columns (in a kernel of its own: the code for it cost calls that do not
// need it 3 %).  1024 x 1024, k = 512, batch 1, x two bytes off: 10.4 us read value by value and twice, 8.4 so; 4095 -> 4097 14.2 / 10.6.
struct FewRaw {
    v4u a, b;
};
template <bool ANY>
struct InputX {
    const uint16_t* x;   // first row of the group
    const uint16_t* b;   // zero padded to whole column tiles
    int cols;
    __device__ __forceinline__ void load(int bi, int v, FewRaw& r) const {
        const uint16_t* row = x + (size_t)bi * cols;
        r.b = *reinterpret_cast<const v4u*>(b + 8 * v);
        if (!ANY) {
            r.a = *reinterpret_cast<const v4u*>(row + (8 * v < cols ? 8 * v : 0));
        } else if (cols >= 8) {
            r.a = dbf_half8_load(row, v, cols);
        } else {   // (the row's end in the vector's end, as dbf_half8_load has it)
            unsigned h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = row[max(e + cols - 8, 0)];
#pragma unroll
            for (int e = 0; e < 4; ++e) r.a[e] = h[2 * e] | h[2 * e + 1] << 16;
        }
    }
    __device__ __forceinline__ void get(int v, const FewRaw& r, float (&u)[8]) const {
        const h8 xv = __builtin_bit_cast(h8, ANY ? dbf_half8_place(r.a, v, cols) : r.a), bv = __builtin_bit_cast(h8, r.b);
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = fmaf((float)xv[e], (float)bv[e], 0.f);  // (exact; past the row b is zero; one instruction with its conversions, v_fma_mix_f32)
    }
};
struct InputT {
    const float* t;
    int stride;
    __device__ __forceinline__ void load(int bi, int v, FewRaw& r) const {
        const v4u* p = reinterpret_cast<const v4u*>(t + (size_t)bi * stride + 8 * v);
        r.a = p[0];
        r.b = p[1];
    }
    __device__ __forceinline__ void get(int, const FewRaw& r, float (&u)[8]) const {
        const v4f a = __builtin_bit_cast(v4f, r.a), b = __builtin_bit_cast(v4f, r.b);
        u[0] = a.x;  u[1] = a.y;  u[2] = a.z;  u[3] = a.w;
        u[4] = b.x;  u[5] = b.y;  u[6] = b.z;  u[7] = b.w;
    }
};

// Largest |u| of a wavefront's part of a row, to every entry e of wmax[row] with e % parts == part: the eight of a row are read at once.
__device__ __forceinline__ void few_put_max(FewMisc* m, int bi, const FewShare s, float mx, int lane) {
    if (lane < FEW_WAVES && (lane & (s.parts - 1)) == s.part) m->wmax[bi][lane] = mx;
}
__device__ __forceinline__ float few_row_max(const FewMisc* m, int bi) {
    const v4f* p = reinterpret_cast<const v4f*>(m->wmax[bi]);
    const v4f a = p[0], b = p[1];
    return fmaxf(fmaxf(fmaxf(a.x, a.y), fmaxf(a.z, a.w)), fmaxf(fmaxf(b.x, b.y), fmaxf(b.z, b.w)));
}

// Largest |u| of every row (few_put_max).  held: every wavefront has one row and at most H vectors per lane, which have been
// requested into raw and stay there.
template <class IN, int H>
__device__ __forceinline__ void few_max(const IN& in, const FewShare s, int nb, int nvec, bool held, const FewRaw (&raw)[H],
                                        float (&u)[H][8], FewMisc* m, int lane) {
    if (held) {
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            in.get(min(lane + 64 * (s.part + s.parts * i), nvec - 1), raw[i], u[i]);   // (a vector past the row repeats its last)
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(u[i][e]));
        }
        mx = dbf_wave_max(mx);
        if (s.row < nb) few_put_max(m, s.row, s, mx, lane);
        return;
    }
    for (int bi = s.row; bi < nb; bi += s.P) {
        float mx = 0.f;
        for (int v0 = lane + 64 * s.part; v0 < nvec; v0 += 64 * s.parts * 4) {
            FewRaw r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) in.load(bi, min(v0 + 64 * s.parts * i, nvec - 1), r[i]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float u[8];
                in.get(min(v0 + 64 * s.parts * i, nvec - 1), r[i], u);
#pragma unroll
                for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(u[e]));
            }
        }
        mx = dbf_wave_max(mx);
        few_put_max(m, bi, s, mx, lane);
    }
}

// q = rint(u * inv) of eight values as high and low bytes; returns the sum of the q.  Adding 1.5 * 2^23 + 128 rounds to the
// integer q + 128 (ties to even: 128 is even) and leaves it in the low bits of the word, where byte 1 is the high byte of
// q and byte 0 the low one with its top bit flipped.
__device__ __forceinline__ int few_round8(const float (&u)[8], float inv, uint2& hi, uint2& lo) {
#pragma clang fp contract(off)
    unsigned p[4], h[2], l[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float t0 = u[2 * e] * inv, t1 = u[2 * e + 1] * inv;
        const unsigned b0 = __builtin_bit_cast(unsigned, t0 + 12583040.f), b1 = __builtin_bit_cast(unsigned, t1 + 12583040.f);
        p[e] = __builtin_amdgcn_perm(b1, b0, 0x05010400u);  // (b0.0, b1.0, b0.1, b1.1)
    }
    int sh = 0, sl = 0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        l[e] = __builtin_amdgcn_perm(p[2 * e + 1], p[2 * e], 0x05040100u) ^ 0x80808080u;
        h[e] = __builtin_amdgcn_perm(p[2 * e + 1], p[2 * e], 0x07060302u);
        sh = __builtin_amdgcn_sdot4((int)h[e], 0x01010101, sh, false);
        sl = __builtin_amdgcn_sdot4((int)l[e], 0x01010101, sl, false);
    }
    hi = make_uint2(h[0], h[1]);
    lo = make_uint2(l[0], l[1]);
    return 256 * sh + sl;
}

// Rounds the vectors [v0, v1) of every row into the planes (whose first column tile is v0's) and adds up the sums of the q; of held rows
// the lane's sum is returned, for few_sigma once the barrier behind the planes has been passed.
template <class IN, int H>
__device__ __forceinline__ int few_round(const IN& in, const FewShare s, int nb, int nvec, int v0, int v1, bool held,
                                          const float (&held_u)[H][8], FewMisc* m, unsigned char* planes, int tile_block, int lane) {
    auto inv_of = [&](int bi) {
        const float mx = few_row_max(m, bi);
        return mx > 0.f ? QMAX / mx : 0.f;
    };
    auto place = [&](int bi, int v) { return planes + ((v - v0) >> 3) * tile_block + 2 * bi * DBF_TILE_COLS + 8 * (v & 7); };
    auto put = [&](unsigned char* d, const float (&u)[8], float inv) {
        uint2 hi, lo;
        const int sum = few_round8(u, inv, hi, lo);
        *reinterpret_cast<uint2*>(d) = hi;
        *reinterpret_cast<uint2*>(d + DBF_TILE_COLS) = lo;
        return sum;
    };
    if (held) {
        if (s.row >= nb) return 0;
        const float inv = inv_of(s.row);
        int sum = 0;
        const int va = lane + 64 * s.part;
        unsigned char* d = place(s.row, va);
#pragma unroll
        for (int i = 0; i < H; ++i) {   // vector va + 64 parts i
            const int v = va + 64 * s.parts * i;
            if (v >= v0 && v < v1) sum += put(d, held_u[i], inv);
            d += 8 * s.parts * tile_block;
        }
        return sum;
    }
    for (int bi = s.row; bi < nb; bi += s.P) {
        const float inv = inv_of(bi);
        int sum = 0;
        for (int b = v0 + lane + 64 * s.part; b < v1; b += 64 * s.parts * 4) {
            FewRaw r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) in.load(bi, min(b + 64 * s.parts * i, nvec - 1), r[i]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b + 64 * s.parts * i < v1) {
                    float u[8];
                    in.get(b + 64 * s.parts * i, r[i], u);
                    sum += put(place(bi, b + 64 * s.parts * i), u, inv);
                }
        }
        sum = dbf_wave_sum(sum);
        if (lane == 0) atomicAdd(&m->sigma[bi], sum);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // (vectors past the row were requested and not used: nothing may be left for the loop over the tiles to wait for)
    return 0;
}
// What nobody needs before the sums are taken: the held rows' sums of the q, and the scales.
__device__ __forceinline__ void few_sigma(FewMisc* m, const FewShare s, int nb, bool held, int sum, int tid) {
    if (held && s.row < nb) {
        sum = dbf_wave_sum(sum);
        if ((tid & 63) == 0) atomicAdd(&m->sigma[s.row], sum);
    }
    if (tid < nb) m->scale[tid] = few_row_max(m, tid) / QMAX;
}

// One wavefront's tiles [lo, hi) of a span of tiles of one row tile.
struct FewStream {
    __amdgpu_buffer_rsrc_t rsrc;
    v4u tl[FEW_PF];
    int lo, hi, lane;

    __device__ __forceinline__ void fetch(int j, int unit) {
        const unsigned off = (unit < hi ? (unsigned)unit * DBF_TILE_BYTES : OOB) + 16u * lane;
        tl[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
    }
    __device__ __forceinline__ void start(const uint8_t* bits, int n_units, int lo_, int hi_, int lane_) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits), 0, n_units * DBF_TILE_BYTES, 0x00020000);
        lo = lo_;  hi = hi_;  lane = lane_;
#pragma unroll
        for (int j = 0; j < FEW_PF; ++j) {
            fetch(j, lo + j);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // planes: LDS planes whose tile 0 is the span's first tile.  The sign tiles' bit planes s0 .. s0 + NP - 1 are multiplied.
    template <int NP>
    __device__ __forceinline__ void run(const unsigned char* planes, int tile_block, int ncols, int s0, v4i (&acc)[NP]) {
        const int g = lane >> 4, c = lane & 15;
        // (unused operand columns read the last valid one)
        const unsigned char* xp = planes + min(c, ncols - 1) * DBF_TILE_COLS + 16 * g + lo * tile_block;
        // A tile's operand is read while the one before is multiplied (the last read, of a tile behind the span, lands in the LDS that the
        // launch keeps behind the planes and is not used).
        v4i next = *reinterpret_cast<const v4i*>(xp);
        auto multiply = [&](int j) {
            const v4i xv = next;
            xp += tile_block;
            next = *reinterpret_cast<const v4i*>(xp);
#pragma unroll
            for (int s = 0; s < NP; ++s) {
                const unsigned msk = 0x01010101u << (NP == 8 ? s : s0 + s);
                const v4i a = {(int)(tl[j].x & msk), (int)(tl[j].y & msk), (int)(tl[j].z & msk), (int)(tl[j].w & msk)};
                acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, xv, acc[s], 0, 0, 0);
            }
        };
        // (whole rounds of the ring, then the rest without new requests: with a way out in the middle of a round the compiler
        //  cannot tell which loads are still under way at its start, and waits for all of them)
        int i0 = lo;
        for (; i0 + FEW_PF <= hi; i0 += FEW_PF) {
#pragma unroll
            for (int j = 0; j < FEW_PF; ++j) {
                multiply(j);
                fetch(j, i0 + j + FEW_PF);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int j = 0; j < FEW_PF - 1; ++j) {
            if (i0 + j >= hi) break;
            multiply(j);
        }
    }
};

// The signed sum of a row of bit plane s from its sums over the high and the low bytes of the q: 2 * (sum over the set bits) - sigma, exact
// (modulo 2^32 on the way).
__device__ inline int few_total(int high, int low, int s, int sigma) {
    int vh = high >> s, vl = low >> s;
    if (s == 7) {  // the mask 0x80 is -128 as an int8
        vh = -vh;
        vl = -vl;
    }
    return (int)(2u * (unsigned)(vh * 256 + vl) - (unsigned)sigma);
}
// ... of row rho of a row tile and batch row bi of the small-layer kernel
__device__ inline int small_total(const int* red, int bi, int rho, int sigma) {
    return few_total(red[2 * bi * FEW_RB + rho], red[(2 * bi + 1) * FEW_RB + rho], rho >> 4, sigma);
}

// Rounded to fp32, then to fp16, as in every other kernel (left to itself the compiler rounds the last product to fp16 at once:
// one output in ten thousand in its last bit).
__device__ __forceinline__ uint16_t few_half(float v) {
    asm("" : "+v"(v));
    return __builtin_bit_cast(uint16_t, (_Float16)v);
}

// Operand columns of `nb` tokens, rounded up to a power of two (its logarithm): 1 .. 4.
__host__ __device__ inline int few_log_cols(int nb) { return nb <= 1 ? 1 : nb <= 2 ? 2 : nb <= 4 ? 3 : 4; }
__host__ __device__ inline int few_slot_bytes(int nb, int np) { return FEW_WAVES * 4 * np * 16 << few_log_cols(nb); }

// One stage, workgroup (row tile, group of tokens and of bit planes, column piece).  `first`: LIST: the items (one row tile each); else the layer's
// sign tiles, behind which its vectors lie in_off and row_off times 16 bytes.  All arguments fit the 14 scalar registers that are loaded before
// the wavefronts start (a layer alone: no memory round trip before its loads).
// NP: bit planes of a workgroup (blockIdx.y: group of tokens, then of bit planes), 8 where rows are cut.  tokens: T | group << 16 | aliased << 20; cut: tiles of an LDS chunk | pieces << 10 | (ceil(2^16 / pieces) - 1) << 16.
// io: x or y.  acc: zeroed integers, [row tile][DBF_MAX_BATCH][128], then an arrival counter per (row tile, token group).
// Where the time of a workgroup goes (three layers of 4096 x 4096, k = 3072, batch 8: 64 tiles, four tokens; cycles of 13000 on the compute
// unit): arguments, item and requests 2400, the input's arrival and maximum 1900, rounding 2900, tiles 3800, sums 1400, outputs 700.  The
// matrix instructions with their ANDs take 29 cycles each for 16 of work; nothing overlaps the rounding but the tiles' way from memory.
// The wavefronts' sums: every wavefront leaves its own in LDS in 16-byte pieces, a thread adds up the eight of two rows.  They lie behind the
// planes, or where the planes were (`aliased`), if both do not fit.
template <bool STAGE_A, bool LIST, int H, int NP, bool ANY>
__global__ __launch_bounds__(FEW_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_few_kernel(
    const void* __restrict__ first, float* __restrict__ t_base, uint16_t* __restrict__ io, int* __restrict__ acc_base, int in_off, int row_off,
    int cols_, int rows_, unsigned tokens, unsigned cut) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = tokens & 0xFFFF, group = (tokens >> 16) & 15, aliased = tokens >> 20;
    const int s0 = NP * (blockIdx.y % (8 / NP)), piece = blockIdx.z;
    const int chunk_tiles = cut & 1023, pieces = (cut >> 10) & 63;
    const int t0 = blockIdx.y / (8 / NP) * group, nb = min(group, T - t0), ncols = 2 * nb;
    const int tile_block = few_tile_block(ncols);
    const uint8_t* bits;
    const uint16_t *in_scale, *row_scale;
    int cols, rows, row0, stride, n_items;
    if (LIST) {
        const DbfItem& it = static_cast<const DbfItem*>(first)[blockIdx.x];
        bits = it.bits;
        cols = it.cols;  rows = it.rows;  row0 = it.row0;  stride = it.t_stride;
        in_scale = it.in_scale;  row_scale = it.row_scale;
        if (!t_base) t_base = it.t;
        io += it.io_off * T;
        n_items = rows_;
    } else {
        cols = cols_;  rows = rows_;  row0 = blockIdx.x * DBF_TILE_ROWS;
        stride = ((STAGE_A ? cols : rows) + DBF_TILE_ROWS - 1) & ~(DBF_TILE_ROWS - 1);
        const uint8_t* tiles = static_cast<const uint8_t*>(first);
        bits = tiles + (size_t)blockIdx.x * ((cols + DBF_TILE_COLS - 1) / DBF_TILE_COLS) * DBF_TILE_BYTES;
        in_scale = reinterpret_cast<const uint16_t*>(tiles + 16ll * in_off);
        row_scale = reinterpret_cast<const uint16_t*>(tiles + 16ll * row_off) + row0;
        n_items = (rows + DBF_TILE_ROWS - 1) / DBF_TILE_ROWS;
    }
    const int n_ct = (cols + DBF_TILE_COLS - 1) / DBF_TILE_COLS, nvec = 8 * n_ct;
    // (pieces of ceil(n_ct / pieces) tiles, or one more; the last takes what is left)
    const int piece_tiles = (int)(((unsigned)n_ct * (cut >> 16) + n_ct + 65535u) >> 16);
    const int ct0 = min(n_ct, piece * piece_tiles), ct1 = min(n_ct, ct0 + piece_tiles);
    FewMisc* m = reinterpret_cast<FewMisc*>(smem);
    unsigned char* planes = smem + sizeof(FewMisc);
    v4i* slots = reinterpret_cast<v4i*>(planes + (aliased ? 0 : chunk_tiles * tile_block));   // [wavefront][plane][g][column]
    float* t = t_base + (size_t)t0 * stride;
    const FewShare sh = few_share(nb, w);

    InputX<ANY> inx;
    inx.x = io + (size_t)t0 * cols;  inx.b = in_scale;  inx.cols = cols;
    const InputT inp = {t, stride};
    const int mine = (nvec + 64 * sh.parts - 1) >> (6 + sh.log_parts);
    const bool held = mine <= H && ct1 - ct0 <= chunk_tiles;
    // The input is requested before the first tiles: loads complete in order, and the tiles come from farther away.
    FewRaw raw[H];
    FewStream st;
    int c0 = ct0, c1 = min(ct1, c0 + chunk_tiles);
    auto start = [&]() {
        const int n = c1 - c0;
        st.start(bits + (size_t)c0 * DBF_TILE_BYTES, n, n * w / FEW_WAVES, n * (w + 1) / FEW_WAVES, lane);
    };
    if (held) {
        const int bi = min(sh.row, nb - 1);
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int v = min(lane + 64 * (sh.part + sh.parts * i), nvec - 1);
            if (STAGE_A) inp.load(bi, v, raw[i]); else inx.load(bi, v, raw[i]);
        }
    }
    // this thread's outputs: of token bi the rows rho and rho + 1 of the row tile, from the sums of columns c (high bytes even, low odd)
    const int lc = few_log_cols(nb), c = tid & ((1 << lc) - 1), plane = s0 + (tid >> (lc + 2)), bi = c >> 1, odd = c & 1;
    const int rho = 16 * plane + 4 * ((tid >> lc) & 3) + 2 * odd, row = row0 + rho;
    const bool mine_out = tid < (4 * NP << lc) && c < ncols;
    const unsigned rscale2 = *reinterpret_cast<const unsigned*>(row_scale + (rho & 127));
    __builtin_amdgcn_sched_barrier(0);
    start();
    __builtin_amdgcn_sched_barrier(0);
    if (tid < DBF_MAX_BATCH) m->sigma[tid] = 0;
    float u[H][8];
    if (STAGE_A) few_max(inp, sh, nb, nvec, held, raw, u, m, lane); else few_max(inx, sh, nb, nvec, held, raw, u, m, lane);
    __syncthreads();
    v4i acc[NP];
#pragma unroll
    for (int s = 0; s < NP; ++s) acc[s] = (v4i){0, 0, 0, 0};
    for (;;) {
        const int sum = STAGE_A ? few_round(inp, sh, nb, nvec, 8 * c0, 8 * c1, held, u, m, planes, tile_block, lane)
                                : few_round(inx, sh, nb, nvec, 8 * c0, 8 * c1, held, u, m, planes, tile_block, lane);
        __syncthreads();
        if (NP < 8 || c0 == ct0) few_sigma(m, sh, nb, held, sum, tid);
        st.run<NP>(planes, tile_block, ncols, s0, acc);
        if (NP < 8 || c1 >= ct1) break;   // (a part of the bit planes: of pieces that are one chunk)
        __syncthreads();   // every wavefront is done with the chunk's planes
        c0 = c1;
        c1 = min(ct1, c0 + chunk_tiles);
        start();
    }
    // register i of acc[s] of lane (g, c) is row 16 (s0 + s) + 4 g + i, operand column c
    if (aliased) __syncthreads();
    if ((lane & 15) < ncols) {
#pragma unroll
        for (int s = 0; s < NP; ++s) slots[((4 * (w * NP + s) + (lane >> 4)) << lc) + (lane & 15)] = acc[s];
    }
    __syncthreads();

    int total[2];
    if (mine_out) {
        v4i sum = slots[tid];
#pragma unroll
        for (int q = 1; q < FEW_WAVES; ++q) sum += slots[((4 * q * NP) << lc) + tid];
        // (rows 0 and 1 are finished by the even column's lane, 2 and 3 by the odd one's: each hands the other what it lacks)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int own = odd ? sum[2 + i] : sum[i], other = dbf_dpp_move<0xB1>(odd ? sum[i] : sum[2 + i]);   // quad_perm [1,0,3,2]
            total[i] = few_total(odd ? other : own, odd ? own : other, plane, m->sigma[bi]);
        }
    }
    auto store = [&]() {
        const float scale = m->scale[bi];
        const float v0 = (float)total[0] * scale * (float)__builtin_bit_cast(_Float16, (uint16_t)rscale2);
        const float v1 = (float)total[1] * scale * (float)__builtin_bit_cast(_Float16, (uint16_t)(rscale2 >> 16));
        if (STAGE_A) {
            uint16_t* out = io + (size_t)(t0 + bi) * rows + row;
            if (row < rows) out[0] = few_half(v0);
            if (row + 1 < rows) out[1] = few_half(v1);
        } else {
            *reinterpret_cast<float2*>(t + (size_t)bi * stride + row) = make_float2(v0, v1);   // (padded rows have scale 0)
        }
    };
    if (pieces == 1) {
        if (mine_out) store();
        return;
    }
    // A column piece: exact integer sums are added up in memory; the last piece of the row tile to arrive takes them out
    // (leaving zeros), scales and stores.
    int* a = acc_base + ((size_t)blockIdx.x * DBF_MAX_BATCH + t0 + bi) * DBF_TILE_ROWS + rho;
    if (mine_out) {
#pragma unroll
        for (int i = 0; i < 2; ++i) __hip_atomic_fetch_add(a + i, total[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's adds have been performed ...
    __syncthreads();                                  // ... and so have the workgroup's
    if (tid == 0) {
        int* cnt = acc_base + (size_t)n_items * DBF_MAX_BATCH * DBF_TILE_ROWS + (size_t)blockIdx.x * DBF_PIECE_CNT_STRIDE + blockIdx.y;
        m->last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pieces - 1;
        if (m->last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!m->last || !mine_out) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) total[i] = __hip_atomic_exchange(a + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    store();
}

// ---------------------------------------------------------------------------------------------
// A small layer in one launch: a workgroup per layer and pair of tokens runs both stages, the middle activations stay in LDS.  For layers
// of at most SMALL_TILES tiles a stage, i.e. four per wavefront: the signs of BOTH stages are requested at the start and have
// arrived when they are needed.  Such a call is bound by its launches -- the host takes 3.2 us for each, the device 2 --,
// not by the one compute unit that does the work.  Device, us per call at batch 1 / 8, two launches / one: 512 x 512, k = 256 (16 tiles)
// 7.6, 8.1 / 6.4, 7.2;  k = 512 (32) 7.8, 8.3 / 7.3, 8.2;  768 x 768, k = 384 (36) 8.1, 8.6 / 8.8, 9.0;  1024 x 1024, k = 512 (64) 8.3, 8.8 /
// 9.2, 10.4: hence the limit.  From Python, where a launch costs more, 512 x 512 went from 10.0 to 6.7.
// ---------------------------------------------------------------------------------------------
constexpr int SMALL_PER_WAVE = 4, SMALL_TILES = FEW_WAVES * SMALL_PER_WAVE;

// The sums of a wavefront's tiles (tiles[0 .. hi - lo) of the span, row tile major) into red[row tile].
__device__ __forceinline__ void small_stage(const FewStream& st, const unsigned char* planes, int tile_block, int ncols, int n_ct, int* red) {
    const int g = st.lane >> 4, c = st.lane & 15;
    const unsigned char* xp = planes + min(c, ncols - 1) * DBF_TILE_COLS + 16 * g;
    int rt = st.lo / n_ct, ct = st.lo - rt * n_ct;
    v4i acc[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) acc[s] = (v4i){0, 0, 0, 0};
    auto flush = [&]() {
        if (c < ncols) {
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i) atomicAdd(&red[(rt * ncols + c) * FEW_RB + 4 * g + 16 * s + i], acc[s][i]);
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) acc[s] = (v4i){0, 0, 0, 0};
    };
#pragma unroll
    for (int j = 0; j < SMALL_PER_WAVE; ++j) {
        if (st.lo + j >= st.hi) break;
        const v4i xv = *reinterpret_cast<const v4i*>(xp + ct * tile_block);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const unsigned msk = 0x01010101u << s;
            const v4i a = {(int)(st.tl[j].x & msk), (int)(st.tl[j].y & msk), (int)(st.tl[j].z & msk), (int)(st.tl[j].w & msk)};
            acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, xv, acc[s], 0, 0, 0);
        }
        if (++ct == n_ct) {
            flush();
            ct = 0;
            ++rt;
        }
    }
    if (ct != 0 && st.hi > st.lo) flush();
}

template <bool ANY>
__global__ __launch_bounds__(FEW_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbf_small_layer_kernel(
    const DbfStage* __restrict__ stages_b, const DbfStage* __restrict__ stages_a, const uint16_t* __restrict__ x_base,
    uint16_t* __restrict__ y_base, int T, int group, int planes_bytes, int red_ints) {
    extern __shared__ __align__(16) unsigned char smem[];
    const DbfStage sb = stages_b[blockIdx.x], sa = stages_a[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.y * group, nb = min(group, T - t0), ncols = 2 * nb;
    const int tile_block = few_tile_block(ncols);
    FewMisc* m = reinterpret_cast<FewMisc*>(smem);                 // one per stage
    unsigned char* planes = smem + 2 * sizeof(FewMisc);
    int* red_b = reinterpret_cast<int*>(planes + planes_bytes);    // [row tiles of both stages][ncols][FEW_RB]
    int* red_a = red_b + sb.n_rt * ncols * FEW_RB;
    float* t = reinterpret_cast<float*>(red_b + red_ints);         // [nb][rows of B, whole row tiles]
    const int t_len = sb.n_rt * DBF_TILE_ROWS;
    const FewShare sh = few_share(nb, w);
    constexpr int H = 2;

    InputX<ANY> inx;
    inx.x = x_base + sb.x_off * T + (size_t)t0 * sb.cols;  inx.b = sb.in_scale;  inx.cols = sb.cols;
    FewRaw raw[H];
    const int nvec_b = 8 * sb.n_ct, nvec_a = 8 * sa.n_ct;
    {
        const int bi = min(sh.row, nb - 1);
#pragma unroll
        for (int i = 0; i < H; ++i) inx.load(bi, min(lane + 64 * (sh.part + sh.parts * i), nvec_b - 1), raw[i]);
    }
    FewStream st, st2;
    const int n = sb.n_rt * sb.n_ct, n2 = sa.n_rt * sa.n_ct;
    __builtin_amdgcn_sched_barrier(0);
    st.start(sb.bits, n, n * w / FEW_WAVES, n * (w + 1) / FEW_WAVES, lane);
    st2.start(sa.bits, n2, n2 * w / FEW_WAVES, n2 * (w + 1) / FEW_WAVES, lane);
    __builtin_amdgcn_sched_barrier(0);
    for (int i = tid; i < red_ints; i += FEW_THREADS) red_b[i] = 0;
    if (tid < 2 * DBF_MAX_BATCH) m[tid / DBF_MAX_BATCH].sigma[tid % DBF_MAX_BATCH] = 0;
    float u[H][8];
    few_max(inx, sh, nb, nvec_b, true, raw, u, m, lane);
    __syncthreads();
    const int sum_b = few_round(inx, sh, nb, nvec_b, 0, nvec_b, true, u, m, planes, tile_block, lane);
    __syncthreads();
    few_sigma(m, sh, nb, true, sum_b, tid);
    small_stage(st, planes, tile_block, ncols, sb.n_ct, red_b);
    __syncthreads();
    for (int e = tid; e < nb * t_len; e += FEW_THREADS) {
        const int bi = e / t_len, row = e - bi * t_len;
        t[e] = (float)small_total(red_b + (row >> 7) * ncols * FEW_RB, bi, row & 127, m->sigma[bi]) * m->scale[bi] *
               (float)__builtin_bit_cast(_Float16, sb.row_scale[row]);
    }
    __syncthreads();
    const InputT inp = {t, t_len};
    {
        const int bi = min(sh.row, nb - 1);
#pragma unroll
        for (int i = 0; i < H; ++i) inp.load(bi, min(lane + 64 * (sh.part + sh.parts * i), nvec_a - 1), raw[i]);
    }
    ++m;
    few_max(inp, sh, nb, nvec_a, true, raw, u, m, lane);
    __syncthreads();
    const int sum_a = few_round(inp, sh, nb, nvec_a, 0, nvec_a, true, u, m, planes, tile_block, lane);
    __syncthreads();
    few_sigma(m, sh, nb, true, sum_a, tid);
    small_stage(st2, planes, tile_block, ncols, sa.n_ct, red_a);
    __syncthreads();
    const int rows = sa.rows, all = sa.n_rt * DBF_TILE_ROWS;
    uint16_t* y = y_base + sa.y_off * T + (size_t)t0 * rows;
    for (int e = tid; e < nb * all; e += FEW_THREADS) {
        const int bi = e / all, row = e - bi * all;
        if (row >= rows) continue;
        const float val = (float)small_total(red_a + (row >> 7) * ncols * FEW_RB, bi, row & 127, m->sigma[bi]) * m->scale[bi] *
                          (float)__builtin_bit_cast(_Float16, sa.row_scale[row]);
        y[(size_t)bi * rows + row] = few_half(val);
    }
}

constexpr int FEW_MAX_WGS = 256;     // compute units
constexpr int FEW_LDS = 156 * 1024;  // (its registers give a workgroup the compute unit to itself)

hipError_t raise_lds(const void* kernel) { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, FEW_LDS); }
template <int H, int NP>
hipError_t raise_lds_few() {
    hipError_t e = raise_lds(reinterpret_cast<const void*>(&dbf_few_kernel<false, false, H, NP, false>));
    if (e == hipSuccess) e = raise_lds(reinterpret_cast<const void*>(&dbf_few_kernel<false, true, H, NP, false>));
    if (e == hipSuccess) e = raise_lds(reinterpret_cast<const void*>(&dbf_few_kernel<false, false, H, NP, true>));
    if (e == hipSuccess) e = raise_lds(reinterpret_cast<const void*>(&dbf_few_kernel<false, true, H, NP, true>));
    if (e == hipSuccess) e = raise_lds(reinterpret_cast<const void*>(&dbf_few_kernel<true, false, H, NP, false>));
    if (e == hipSuccess) e = raise_lds(reinterpret_cast<const void*>(&dbf_few_kernel<true, true, H, NP, false>));
    return e;
}
template <int NP>
hipError_t raise_lds_planes() {
    for (hipError_t e : {raise_lds_few<2, NP>(), raise_lds_few<4, NP>(), raise_lds_few<6, NP>(), raise_lds_few<8, NP>(), raise_lds_few<10, NP>(),
                         raise_lds_few<FEW_HELD, NP>()})
        if (e != hipSuccess) return e;
    return hipSuccess;
}
// Whether every x row of a call can be read in 16-byte pieces.
bool rows_aligned(const DbfPlan& p, const void* x) { return p.x_vec_ok && (reinterpret_cast<uintptr_t>(x) & 15) == 0; }

// Tokens per workgroup and column pieces of a stage of n_items row tiles.  As many workgroups as there are compute units, and no
// more: a second one on a compute unit costs a whole round (its registers allow one).  Fewer tokens per workgroup first -- less
// rounding in each, no combination --, then, for rows of 80 column tiles and more, pieces of at least 24 tiles.  Microseconds per call:
//   4096 x 4096, k = 3072, batch 8, tokens per workgroup 8 / 4 / 2                 14.6 / 13.7 / 13.4 (96 workgroups a stage at most)
//   three of them, batch 8, 8 / 4 / 2                                              15.0 / 14.1 / 24.8 (288 workgroups)
//   28672 -> 8192, k = 12743, batch 1, pieces of the two stages 1, 1 / 2, 4 / 3, 4 27.1 / 22.5 / 29.6 (100 row tiles: 300 workgroups)
//   11008 -> 4096, k = 4477, batch 1, pieces 1 / 2 / 4 / 7                         16.7 / 15.7 / 14.5 / 14.1
//   4096 -> 11008, k = 4477 (70 column tiles), batch 1, pieces 1 / 2               13.5 / 13.8
struct FewCut {
    int group, pieces;
    long long wgs;
};
FewCut few_cut(int n_items, int n_ct, int T, bool pieces_ok) {
    FewCut c = {2, 1, 0};
    auto groups = [&]() { return (T + c.group - 1) / c.group; };
    while (c.group < 8 && (long long)n_items * groups() > FEW_MAX_WGS) c.group *= 2;
    c.wgs = (long long)n_items * groups();
    if (pieces_ok && n_ct >= 80 && 2 * c.wgs <= FEW_MAX_WGS) {
        c.pieces = (int)(FEW_MAX_WGS / c.wgs);
        if (c.pieces > n_ct / 24) c.pieces = n_ct / 24;
    }
    return c;
}
// How a stage that is not cut into column pieces is shared out: `group` tokens and `planes` bit planes of the row tile (16 rows each) to a
// workgroup, at most one workgroup per compute unit as in few_cut.  Per column tile a workgroup takes about 10 cycles to round a token (18 where
// it reads the row twice) and 8 to multiply a bit plane; the sign tiles come from L2 for all but one of those that read them.  The least of
// that sum.  us per call of both stages, (tokens, planes) the same for both:
//   4096 x 4096, k = 2048 (16 and 32 row tiles), batch 1       2, 8: 9.84   2, 4: 8.57   2, 2: 7.91   (2, 1: 8.1)
//   three of 4096 x 4096, k = 3072 (72 and 96), batch 1        2, 8: 10.83  2, 4: 9.37
//   one of those (24 and 32), batch 4                          2, 8: 10.66  2, 4: 9.22   2, 2: 8.61   4, 8: 11.74  4, 2: 9.39
//   batch 8                                                    2, 8: 10.77  2, 4: 9.41   4, 4: 10.31  4, 2: 9.62   8, 8: 13.81  8, 2: 11.08
//   batch 16                                                   2, 8: 11.08  4, 8: 12.04  4, 4: 10.62  8, 8: 13.89  8, 2: 11.37
// Column pieces stay as they are: 28672 -> 8192, k = 12743, batch 1, pieces 20.4, whole rows by planes 23.0.
struct FewSplit {
    int group, pieces, planes;
};
FewSplit few_split(const FewCut& base, int n_items, int n_ct, int T) {
    FewSplit best = {base.group, base.pieces, 8};
    if (base.pieces > 1) return best;
    int least = 1 << 30;
    for (int group = 2; group <= 8; group *= 2) {
        const int nb = group < T ? group : T;
        if (group > 2 && 2 * nb <= group) continue;   // (the smaller group is the same)
        if (nb * n_ct > 2560 && group > base.group) continue;
        const bool fits = (n_ct + 1) * few_tile_block(2 * nb) + (int)sizeof(FewMisc) <= FEW_LDS;   // (rows in one LDS chunk)
        const bool held = fits && (8 * n_ct + 64 * few_parts(nb) - 1) / (64 * few_parts(nb)) <= FEW_HELD;
        for (int planes : {8, 4, 2}) {
            if (planes < 8 && !fits) continue;
            if ((long long)n_items * ((T + group - 1) / group) * (8 / planes) > FEW_MAX_WGS) continue;
            const int cost = nb * (held ? 10 : 18) + 8 * planes;
            if (cost < least) {
                least = cost;
                best.group = group;
                best.planes = planes;
            }
        }
    }
    return best;
}
inline int few_cols(const DbfPlan& p, bool stage_a) { return dbf_col_tiles(stage_a ? p.max_cols_A : p.max_cols_B); }

}  // namespace

// More than 64 KiB of LDS per workgroup has to be asked for, once per process (see dbf_mfma_prepare).
hipError_t dbf_few_prepare() {
    static const hipError_t raised = [] {
        const hipError_t e[] = {raise_lds(reinterpret_cast<const void*>(&dbf_small_layer_kernel<false>)),
                                raise_lds(reinterpret_cast<const void*>(&dbf_small_layer_kernel<true>)), raise_lds_planes<8>(),
                                raise_lds_planes<4>(), raise_lds_planes<2>()};
        for (hipError_t x : e)
            if (x != hipSuccess) {
                (void)hipGetLastError();
                return x;
            }
        return hipSuccess;
    }();
    return raised;
}

// A stage is taken if it makes at most one workgroup per compute unit, and a workgroup has no more than 2560 column tiles to round
// (tokens x column tiles).  Against the launches it stands in for, microseconds per call of both stages:
//   4096 x 4096, k = 3072         batch 1 / 2 / 8 / 16   11.1 / 15.2 / 16.8 / 21.0 -> 10.9 / 11.5 / 11.6 / 11.9
//   three of them                                        11.3 / 15.3 / 17.0 / 21.4 -> 11.0 / 11.6 / 13.0 / 16.1
//   11008 -> 4096, k = 4477                              16.3 / 24.7 / 24.9 / 30.5 -> 12.0 / 13.8 / 17.1 / 21.9
//   28672 -> 8192, k = 12743                             36.5 / 58.0 / 60.3 / 68.9 -> 21.0 / 26.8 / 47.3 / (71.0: 8 x 448 column tiles)
//   512 x 512, k = 256                                    8.3 / 12.3 / 13.4 / 16.4 ->  7.6 /  8.0 /  8.1 /  8.3
//   two of 4096 -> 11008, k = 4477 at batch 16           23.1 -> (29.0: 344 workgroups)
// Nor is a group of layers taken whose workgroups would have more than four tokens of whole rows that are longer than the registers hold
// (80 column tiles; 128 where two groups of tokens share a call): every workgroup reads them twice by one wavefront a row, which
// the launches that round each layer's input once for all of its row tiles do in less.  Means over groups of 3-6 layers, against those
// launches: up to 8 tokens  80 column tiles 0.85 (26 calls)   96: 1.02 (12)   128: 1.07 (6)   172: 1.12 (6);   9-16 tokens  128: 0.91 (14)
// 144: 1.00 (17)   172: 1.02 (10)   224: 1.07 (4)   313: 1.12 (4).  Layers alone win throughout (0.67-0.92: few rows to round in those launches).
bool dbf_few_takes(const DbfPlan& p, bool stage_a, int T) {
    const int longest = p.max_cols_B > p.max_cols_A ? p.max_cols_B : p.max_cols_A;
    if (longest > DBF_INT_PATH_MAX_COLS) return false;
    const int n_items = stage_a ? p.nA1 : p.nB1, n_ct = few_cols(p, stage_a);
    const FewCut c = few_cut(n_items, n_ct, T, p.d_few_acc && T <= DBF_MAX_BATCH);
    const int nb = c.group < T ? c.group : T;
    if (c.wgs > FEW_MAX_WGS || nb * n_ct > 2560) return false;
    return !(p.n_layers > 1 && nb > 4 && c.pieces == 1 && n_ct > (T > 8 ? 128 : 80));
}

size_t dbf_few_acc_bytes(int n_items, int max_cols) {
    // (one token makes the fewest workgroups, so the rule cuts there if it cuts at all)
    const bool cut = max_cols <= DBF_INT_PATH_MAX_COLS && few_cut(n_items, dbf_col_tiles(max_cols), 1, true).pieces > 1;
    return cut ? sizeof(int) * (size_t)n_items * (DBF_MAX_BATCH * DBF_TILE_ROWS + DBF_PIECE_CNT_STRIDE) : 0;
}

hipError_t dbf_launch_few(const DbfPlan& p, bool stage_a, const void* x, void* y, float* t_over, int T, hipStream_t stream) {
    const hipError_t raised = dbf_few_prepare();
    if (raised != hipSuccess) return raised;
    // (a prompt, which brings its own middle activations, is never cut: its calls may overlap on one layer and share nothing of it)
    const FewSplit split = few_split(few_cut(stage_a ? p.nA1 : p.nB1, few_cols(p, stage_a), T, !t_over && p.d_few_acc && T <= DBF_MAX_BATCH),
                                     stage_a ? p.nA1 : p.nB1, few_cols(p, stage_a), T);
    const int group = split.group, pieces = split.pieces, np = split.planes;
    const int nb = group < T ? group : T, tile_block = few_tile_block(2 * nb), slots = few_slot_bytes(nb, np);
    const int n_ct = few_cols(p, stage_a), reciprocal = (65536 + pieces - 1) / pieces - 1;
    const int want = (int)(((unsigned)n_ct * reciprocal + n_ct + 65535u) >> 16);   // tiles of a piece
    // The wavefronts' sums behind the planes of a whole piece, or in their place where that does not fit (an idle tile behind the planes: see
    // FewStream::run).
    const bool aliased = (size_t)want * tile_block + slots + sizeof(FewMisc) > (size_t)FEW_LDS;
    const int fit = (FEW_LDS - (int)sizeof(FewMisc)) / tile_block - 1, chunk = aliased && want > fit ? fit : want;
    const int behind = aliased ? (slots > (chunk + 1) * tile_block ? slots : (chunk + 1) * tile_block) : chunk * tile_block + slots;
    const size_t lds = sizeof(FewMisc) + (size_t)behind;
    const int n_items = stage_a ? p.nA1 : p.nB1;
    const dim3 grid(n_items, (T + group - 1) / group * (8 / np), pieces);
    uint16_t* io = static_cast<uint16_t*>(stage_a ? y : const_cast<void*>(x));
    const unsigned tokens = (unsigned)T | (unsigned)group << 16 | (unsigned)aliased << 20;
    const unsigned cut = (unsigned)chunk | (unsigned)pieces << 10 | (unsigned)reciprocal << 16;
    const DbfStage& s = stage_a ? p.h_stage_A : p.h_stage_B;   // (a layer alone)
    const bool list = p.n_layers > 1;
    const void* first = list ? static_cast<const void*>(p.d_items_1 + (stage_a ? p.nB1 : 0)) : s.bits;
    float* t = t_over ? t_over : list ? nullptr : s.t;
    // (a layer's tiles and vectors lie in one block, every section on a multiple of 256 bytes)
    auto from_tiles = [&](const uint16_t* v) { return list || !v ? 0 : (int)((reinterpret_cast<const uint8_t*>(v) - s.bits) / 16); };
    const int in_off = from_tiles(s.in_scale), row_off = from_tiles(s.row_scale);
    const int held = (8 * n_ct + 64 * few_parts(nb) - 1) / (64 * few_parts(nb));   // vectors of eight values per lane
    auto launch = [&](auto h, auto planes) {
        constexpr int H = decltype(h)::value, NP = decltype(planes)::value;
        void (*kernel)(const void*, float*, uint16_t*, int*, int, int, int, int, unsigned, unsigned) =
            stage_a ? (list ? dbf_few_kernel<true, true, H, NP, false> : dbf_few_kernel<true, false, H, NP, false>)
            : rows_aligned(p, x) ? (list ? dbf_few_kernel<false, true, H, NP, false> : dbf_few_kernel<false, false, H, NP, false>)
                                 : (list ? dbf_few_kernel<false, true, H, NP, true> : dbf_few_kernel<false, false, H, NP, true>);
        hipLaunchKernelGGL(kernel, grid, dim3(FEW_THREADS), lds, stream, first, t, io, p.d_few_acc, in_off, row_off, s.cols,
                           list ? n_items : s.rows, tokens, cut);
    };
    // (In steps of two: values held beyond the row's cost requests and rounding of nothing.  us per call with as many as a row needs / 2 / 4 / 12 more: 8192 x 8192,
    // k = 4096, batch 8 12.80 / 13.25 / 13.78 / 15.00; 11008 -> 4096, k = 4477, batch 1 10.36 / 10.96 / 11.40 / 12.92; 4096 -> 11008, batch 8 11.96 / 12.42 / 13.08 / 14.01;
    // 2048 x 2048, batch 8 9.9 / 10.1 / 10.1 / 10.6.  Up to twelve in all.)
    auto launch_planes = [&](auto planes) {
        if (held <= 2) launch(std::integral_constant<int, 2>{}, planes);
        else if (held <= 4) launch(std::integral_constant<int, 4>{}, planes);
        else if (held <= 6) launch(std::integral_constant<int, 6>{}, planes);
        else if (held <= 8) launch(std::integral_constant<int, 8>{}, planes);
        else if (held <= 10) launch(std::integral_constant<int, 10>{}, planes);
        else launch(std::integral_constant<int, FEW_HELD>{}, planes);
    };
    if (np == 2) launch_planes(std::integral_constant<int, 2>{});
    else if (np == 4) launch_planes(std::integral_constant<int, 4>{});
    else launch_planes(std::integral_constant<int, 8>{});
    return hipGetLastError();
}

// LDS of a workgroup of the small-layer kernel for nb tokens.
static size_t small_lds(const DbfPlan& p, int nb, int* planes, int* red_ints) {
    const int ct_b = dbf_col_tiles(p.max_cols_B), ct_a = dbf_col_tiles(p.max_cols_A), rt_b = dbf_row_tiles(p.max_cols_A);  // (rows of B: columns of A)
    *planes = (ct_b > ct_a ? ct_b : ct_a) * few_tile_block(2 * nb);
    *red_ints = ((rt_b + p.max_rt_A) * 2 * nb * FEW_RB + 3) & ~3;   // (the activations behind them are read in 16-byte pieces)
    return 2 * sizeof(FewMisc) + (size_t)*planes + 4 * (size_t)*red_ints + 4 * (size_t)nb * rt_b * DBF_TILE_ROWS;
}
static int small_group(int T) { return T < 2 ? 1 : 2; }

bool dbf_small_layer_takes(const DbfPlan& p, int T) {
    const int nb = small_group(T);
    if (p.max_stage_tiles > SMALL_TILES || (long long)p.n_layers * ((T + nb - 1) / nb) > FEW_MAX_WGS) return false;
    int planes, red;
    const int longest = p.max_cols_B > p.max_cols_A ? p.max_cols_B : p.max_cols_A;
    return dbf_col_tiles(longest) * 8 <= 2 * 64 * few_parts(nb) && small_lds(p, nb, &planes, &red) <= (size_t)FEW_LDS;
}

hipError_t dbf_launch_small_layers(const DbfPlan& p, const void* x, void* y, int T, hipStream_t stream) {
    const hipError_t raised = dbf_few_prepare();
    if (raised != hipSuccess) return raised;
    const int group = small_group(T);
    int planes, red;
    const size_t lds = small_lds(p, group, &planes, &red);
    hipLaunchKernelGGL(rows_aligned(p, x) ? dbf_small_layer_kernel<false> : dbf_small_layer_kernel<true>,
                       dim3(p.n_layers, (T + group - 1) / group), dim3(FEW_THREADS), lds, stream, p.d_stagesB, p.d_stagesA,
                       static_cast<const uint16_t*>(x), static_cast<uint16_t*>(y), T, group, planes, red);
    return hipGetLastError();
}
