// Middle-channel pruning in the tiled layout (paper, section 3.5: the middle dimension is treated as
// channels and only some are kept; choosing them needs gradients and is the caller's business).
// Given the kept middle indices keep[0..k') (increasing), the new layer has
//     A'[:, j'] = A[:, keep[j']],   B'[j', :] = B[keep[j'], :],   m'[j'] = m[keep[j']],
// a and b unchanged.  Both sign matrices stay in the device tile layout (tile = 128 rows x 64
// columns = 1 KiB, byte 256 g + 16 r + j, bit s = sign(row 16 s + r, column 16 g + j)):
//   * a COLUMN of a tile is one byte position in each of its 16 r-rows, all eight bit planes at
//     once, so the column gather of A is a byte gather;
//   * a ROW of a tile is one bit plane of one r-row, so the row gather of B takes bit s_o of the
//     64 bytes of the old row and deposits it as bit s of the new row's bytes; the eight rows that
//     share an output byte are combined by OR in LDS.
// Every output tile is written whole (padding rows / columns as zero bits), coalesced 4-byte stores.  All of a new layer's device work is one launch: A's tiles
// (four of a column of tiles to a workgroup, their reads in flight together), B's (four of a row), the vectors, and the zeros of its scratch.
// Bound by a few trips to memory, one after the other -- index, signs, store -- in a block that has just been allocated.  4096 -> 11008, k = 5970 of which
// 4477 are kept: as three launches with a tile to a workgroup 11.7 + 5.7 + 3.1 us and a memset, now 11.9; the whole call and the first token, whose rest is host calls,
// 118 to 125 us, now 107 to 111.
#include <algorithm>

#include "dbf_kernels.h"

namespace {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int COLS_TILES = 4;                       // row tiles of A' to a workgroup
constexpr int COLS_SPAN = 4;
constexpr int ROWS_TILES = 4;                       // column tiles of B' to a workgroup
constexpr int CLEAR_BYTES = 256 * 16 * 4;           // of the scratch to a workgroup

struct PruneArgs {
    const uint8_t *old_A, *old_B;
    uint8_t *new_A, *new_B, *clear;
    const uint16_t *old_a, *old_m, *old_b;
    uint16_t *new_a, *new_m, *new_b;
    const int* keep;
    size_t clear_bytes;                             // a multiple of 16
    int n_keep, rt_A, ct_A_old, ct_A, rt_B, ct_B;   // tiles of A (old and new columns), of B
    int wg_A, wg_B, wg_vectors;                     // workgroups for each in this order, then the zeros
};

// A': out tiles (rt, ct') <- bytes of old tiles (rt, keep[.] / 64), four rt.  Thread -> new column
// ci = tid / 4 of the tile and four of its sixteen r-rows.
// The columns of a tile are kept from a few old tiles next to each other: up to COLS_SPAN of them come whole, a line at a time, and their bytes are picked in LDS
// (one by one from memory, 64 addresses an instruction: 13.1 us); a sparser choice is read byte by byte.
__device__ __forceinline__ void prune_cols(const PruneArgs& p, int index, uint8_t* tile, unsigned (*old)[COLS_TILES][256]) {
    const int ctn = index % p.ct_A, rt0 = index / p.ct_A * COLS_TILES, tid = threadIdx.x;
    const int ci = tid >> 2, q = tid & 3;
    const int cn = ctn * DBF_TILE_COLS + ci;                 // new column
    const int at = 256 * (ci >> 4) + 64 * q + (ci & 15);
    const bool live = cn < p.n_keep;
    const int o = live ? p.keep[cn] : 0;
    const int first = p.keep[ctn * DBF_TILE_COLS] >> 6, span = (p.keep[min(ctn * DBF_TILE_COLS + 63, p.n_keep - 1)] >> 6) - first + 1;
    const int in_tile = 256 * ((o & 63) >> 4) + 64 * q + (o & 15);   // four bytes, 16 apart
    auto row = [&](int n) { return p.old_A + (size_t)min(rt0 + n, p.rt_A - 1) * p.ct_A_old * DBF_TILE_BYTES; };
    uint8_t b[COLS_TILES][4];
    if (span <= COLS_SPAN) {
        unsigned w[COLS_SPAN][COLS_TILES];
#pragma unroll
        for (int t = 0; t < COLS_SPAN; ++t)
#pragma unroll
            for (int n = 0; n < COLS_TILES; ++n)
                w[t][n] = reinterpret_cast<const unsigned*>(row(n) + (size_t)(first + min(t, span - 1)) * DBF_TILE_BYTES)[tid];   // (no branch around a load)
#pragma unroll
        for (int t = 0; t < COLS_SPAN; ++t)
#pragma unroll
            for (int n = 0; n < COLS_TILES; ++n)
                old[t][n][tid] = w[t][n];
        __syncthreads();
        const int t = live ? (o >> 6) - first : 0;
#pragma unroll
        for (int n = 0; n < COLS_TILES; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) b[n][i] = reinterpret_cast<const uint8_t*>(old[t][n])[in_tile + 16 * i];
    } else {
#pragma unroll
        for (int n = 0; n < COLS_TILES; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) b[n][i] = row(n)[(size_t)(o >> 6) * DBF_TILE_BYTES + in_tile + 16 * i];
    }
#pragma unroll
    for (int n = 0; n < COLS_TILES; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[n * DBF_TILE_BYTES + at + 16 * i] = live ? b[n][i] : 0;
    __syncthreads();
#pragma unroll
    for (int n = 0; n < COLS_TILES; ++n)
        if (rt0 + n < p.rt_A)
            reinterpret_cast<unsigned*>(p.new_A + ((size_t)(rt0 + n) * p.ct_A + ctn) * DBF_TILE_BYTES)[tid] = reinterpret_cast<const unsigned*>(tile)[n * 256 + tid];
}

// B': out tiles (rt', ct) <- bit planes of old tiles (keep[.] / 128, ct), four ct.  Thread -> new row
// rho = tid / 2 of the tile (bit s = rho / 16 of r-row rho % 16) and two of the four column groups.
__device__ __forceinline__ void prune_rows(const PruneArgs& p, int index, unsigned* tile) {
    const int groups = (p.ct_B + ROWS_TILES - 1) / ROWS_TILES, ct0 = index % groups * ROWS_TILES, rtn = index / groups, tid = threadIdx.x;
#pragma unroll
    for (int n = 0; n < ROWS_TILES; ++n) tile[256 * n + tid] = 0;
    const int rho = tid >> 1, hf = tid & 1;
    const int s = rho >> 4, r = rho & 15;
    const int rn = rtn * DBF_TILE_ROWS + rho;                // new row
    const int o = p.keep[min(rn, p.n_keep - 1)], so = (o & 127) >> 4;
    const uint8_t* src = p.old_B + (size_t)(o >> 7) * p.ct_B * DBF_TILE_BYTES + 16 * (o & 15) + 512 * hf;
    v4u w[ROWS_TILES][2];
#pragma unroll
    for (int n = 0; n < ROWS_TILES; ++n)
#pragma unroll
        for (int g = 0; g < 2; ++g) w[n][g] = *reinterpret_cast<const v4u*>(src + (size_t)min(ct0 + n, p.ct_B - 1) * DBF_TILE_BYTES + 256 * g);
    __syncthreads();
    if (rn < p.n_keep) {
#pragma unroll
        for (int n = 0; n < ROWS_TILES; ++n)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                unsigned* dst = tile + 256 * n + (256 * (2 * hf + g) + 16 * r) / 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) atomicOr(dst + e, ((w[n][g][e] >> so) & 0x01010101u) << s);
            }
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < ROWS_TILES; ++n)
        if (ct0 + n < p.ct_B) reinterpret_cast<unsigned*>(p.new_B + ((size_t)rtn * p.ct_B + ct0 + n) * DBF_TILE_BYTES)[tid] = tile[256 * n + tid];
}

__global__ __launch_bounds__(256) void dbf_prune_kernel(const PruneArgs p) {
    __shared__ __align__(16) unsigned tiles[4 * DBF_TILE_BYTES / 4], old[COLS_SPAN][COLS_TILES][256];
    int index = blockIdx.x;
    static_assert(COLS_TILES <= 4 && ROWS_TILES <= 4, "their tiles");
    if (index < p.wg_A) return prune_cols(p, index, reinterpret_cast<uint8_t*>(tiles), old);
    index -= p.wg_A;
    if (index < p.wg_B) return prune_rows(p, index, tiles);
    index -= p.wg_B;
    if (index < p.wg_vectors) {   // m'[i] = m[keep[i]], zero beyond the kept channels (padded to whole row tiles); a and b as they are
        const int i = index * 256 + threadIdx.x;
        if (i < p.rt_B * DBF_TILE_ROWS) p.new_m[i] = i < p.n_keep ? p.old_m[p.keep[i]] : (uint16_t)0;
        if (i < p.rt_A * DBF_TILE_ROWS) p.new_a[i] = p.old_a[i];
        if (i < p.ct_B * DBF_TILE_COLS) p.new_b[i] = p.old_b[i];
        return;
    }
    index -= p.wg_vectors;
#pragma unroll
    for (int n = 0; n < CLEAR_BYTES / (256 * 16); ++n) {
        const size_t at = (size_t)index * CLEAR_BYTES + 256 * 16 * n + 16 * threadIdx.x;
        if (at < p.clear_bytes) *reinterpret_cast<v4u*>(p.clear + at) = (v4u){0, 0, 0, 0};
    }
}

}  // namespace

// src: the layer to prune; dst: a freshly created layer with k = n_keep (its buffers allocated, of its scratch `clear_bytes` from `clear` on still to be
// zeroed); keep_dev: device copy of the kept indices.  Queued on `stream`.
hipError_t dbf_prune_launch(const dbf_layer* src, dbf_layer* dst, const int* keep_dev, int n_keep, void* clear, size_t clear_bytes, hipStream_t stream) {
    PruneArgs p = {};
    p.old_A = src->dA;  p.old_B = src->dB;  p.new_A = dst->dA;  p.new_B = dst->dB;
    p.old_a = src->da;  p.old_m = src->dm;  p.old_b = src->db;  p.new_a = dst->da;  p.new_m = dst->dm;  p.new_b = dst->db;
    p.clear = static_cast<uint8_t*>(clear);  p.clear_bytes = clear_bytes;
    p.keep = keep_dev;  p.n_keep = n_keep;
    p.rt_A = dbf_row_tiles(src->n_out);  p.ct_A_old = dbf_col_tiles(src->k);  p.ct_A = dbf_col_tiles(n_keep);
    p.rt_B = dbf_row_tiles(n_keep);  p.ct_B = dbf_col_tiles(src->n_in);
    const long long wg_A = (long long)p.ct_A * ((p.rt_A + COLS_TILES - 1) / COLS_TILES), wg_B = (long long)p.rt_B * ((p.ct_B + ROWS_TILES - 1) / ROWS_TILES);
    const int most = std::max({p.rt_B * DBF_TILE_ROWS, p.rt_A * DBF_TILE_ROWS, p.ct_B * DBF_TILE_COLS});
    const long long all = wg_A + wg_B + (most + 255) / 256 + (long long)((clear_bytes + CLEAR_BYTES - 1) / CLEAR_BYTES);
    if (all > 0x7fffffff) return hipErrorInvalidValue;   // (2^31 tiles are more than the memory)
    p.wg_A = (int)wg_A;  p.wg_B = (int)wg_B;  p.wg_vectors = (most + 255) / 256;
    hipLaunchKernelGGL(dbf_prune_kernel, dim3((unsigned)all), dim3(256), 0, stream, p);
    return hipGetLastError();
}
