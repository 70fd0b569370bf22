// Wavefront-wide reductions shared by the HIP kernels of libdbf (device code only).
#ifndef DBF_WAVE_H
#define DBF_WAVE_H

#include <hip/hip_runtime.h>

// Reductions with data-parallel-primitive moves (register to register, a few cycles each) instead of
// LDS-crossbar shuffles (~100 cycles each, six in a chain): butterflies inside every row of 16 lanes, then
// the four row results through scalar registers.
template <int CTRL>
__device__ inline int dbf_dpp_move(int v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
__device__ inline float dbf_row16_max(float v) {  // of the row's 16 lanes, in every one of them
    v = fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0xB1>(__builtin_bit_cast(int, v))));   // quad_perm [1,0,3,2]
    v = fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0x4E>(__builtin_bit_cast(int, v))));   // quad_perm [2,3,0,1]
    v = fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0x124>(__builtin_bit_cast(int, v))));  // row_ror:4
    return fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0x128>(__builtin_bit_cast(int, v))));  // row_ror:8
}
__device__ inline int dbf_row16_sum(int v) {
    v += dbf_dpp_move<0xB1>(v);
    v += dbf_dpp_move<0x4E>(v);
    v += dbf_dpp_move<0x124>(v);
    return v + dbf_dpp_move<0x128>(v);
}
// ... and of eight neighbouring lanes
__device__ inline float dbf_row8_max(float v) {
    v = fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0xB1>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0x4E>(__builtin_bit_cast(int, v))));
    return fmaxf(v, __builtin_bit_cast(float, dbf_dpp_move<0x141>(__builtin_bit_cast(int, v))));  // row_half_mirror
}
__device__ inline int dbf_row8_sum(int v) {
    v += dbf_dpp_move<0xB1>(v);
    v += dbf_dpp_move<0x4E>(v);
    return v + dbf_dpp_move<0x141>(v);
}
__device__ inline float dbf_wave_max(float v) {
    v = dbf_row16_max(v);
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}
__device__ inline int dbf_wave_sum(int v) {
    v = dbf_row16_sum(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}

// Sum of a float over the wavefront, the same value in every lane: each row of 16 lanes is summed by its
// lane 0 in a fixed tree, the four row sums are added as (r0 + r1) + (r2 + r3).
__device__ inline float dbf_row16_sum_f(float v) {
    v += __builtin_bit_cast(float, dbf_dpp_move<0xB1>(__builtin_bit_cast(int, v)));
    v += __builtin_bit_cast(float, dbf_dpp_move<0x4E>(__builtin_bit_cast(int, v)));
    v += __builtin_bit_cast(float, dbf_dpp_move<0x124>(__builtin_bit_cast(int, v)));
    return v + __builtin_bit_cast(float, dbf_dpp_move<0x128>(__builtin_bit_cast(int, v)));
}
__device__ inline float dbf_row8_sum_f(float v) {   // of eight neighbouring lanes
    v += __builtin_bit_cast(float, dbf_dpp_move<0xB1>(__builtin_bit_cast(int, v)));
    v += __builtin_bit_cast(float, dbf_dpp_move<0x4E>(__builtin_bit_cast(int, v)));
    return v + __builtin_bit_cast(float, dbf_dpp_move<0x141>(__builtin_bit_cast(int, v)));  // row_half_mirror
}
__device__ inline float dbf_wave_sum_f(float v) {
    v = dbf_row16_sum_f(v);
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return (r0 + r1) + (r2 + r3);
}

// Eight fp16 values, columns 8 v .. + 7 of a row of `cols` values (8 at least) that starts at any even address, in one load: a vector
// that reaches past the row's end is read as the row's last eight values.  dbf_half8_place moves what has arrived where it belongs
// (apart, so that a load has no use of its data right behind it); from column `cols` on it leaves zeros or values of the row:
// callers multiply by a vector that is zero there.
typedef unsigned int dbf_v4u __attribute__((ext_vector_type(4)));
typedef unsigned int dbf_v4u_any __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ dbf_v4u dbf_half8_load(const uint16_t* row, int v, int cols) {
    return *reinterpret_cast<const dbf_v4u_any*>(row + min(8 * v, cols - 8));
}
__device__ __forceinline__ dbf_v4u dbf_half8_place(dbf_v4u r, int v, int cols) {
    if ((cols & 7) == 0) return r;   // (a row of whole vectors has no part of one)
    unsigned __int128 b = __builtin_bit_cast(unsigned __int128, r);
    b >>= 16 * min(max(8 * v + 8 - cols, 0), 7);
    return __builtin_bit_cast(dbf_v4u, b);
}

#endif  // DBF_WAVE_H
