// C out of the accumulators, without a stage in LDS: what the kernels share whose MFMAs take the B fragment first, so that lane l of a
// 32 x 32 block holds row l & 31 and in register i column 8 (i >> 2) + 4 (l >> 5) + (i & 3).
#pragma once
#include "abft_device.h"
#include "gemm_epilogue.h"

namespace abft {

// The sixteen values of a block, added up.
template <typename V, typename ACC> __device__ __forceinline__ V sum16(const ACC &v)
{
    V a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = add_t((V)v[i], (V)v[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = add_t(a[i], a[i + 4]);
    return add_t(add_t(a[0], a[2]), add_t(a[1], a[3]));
}

// 16-bit types: the block rounded, as words of two columns: word 2 q + j = columns 8 q + 4 (lane >> 5) + 2 j + {0, 1}
template <int DT, typename ACC> __device__ __forceinline__ void pack_block(const ACC &acc, uint32_t (&w)[8])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = pack2<DT>((float)acc[2 * j], (float)acc[2 * j + 1]);
}
template <int DT> __device__ __forceinline__ float unpack_lo(uint32_t w)
{
    return DT == DT_BF16 ? __uint_as_float(w << 16) : f16_bits_to_f32(w & 0xFFFFu);
}
template <int DT> __device__ __forceinline__ float unpack_hi(uint32_t w)
{
    return DT == DT_BF16 ? __uint_as_float(w & 0xFFFF0000u) : f16_bits_to_f32(w >> 16);
}

// A 32 x 32 block as row segments.  16-bit C: after the swaps a lane holds 16 bytes of row
// (lane & 15) + 16 pass, and the four lanes of a row its 64 bytes.  int32 C: one more exchange, between
// lane and lane ^ 8, makes it eight rows of 128 bytes (segments of 64 bytes, off their 64-byte boundaries
// as rows of C usually are, wrote 1024 x 577 x 577 in 584 us, unprotected).
template <int DT> constexpr int out_passes() { return Traits<DT>::OS == 4 ? 4 : 2; }
// QUADS, int32 C of unprotected tiles: four neighbouring lanes hold 64 bytes of a row, which a store takes as one piece; in the other order
// neighbours lie in different rows, and a store of 1 KB is 64 pieces.  Its exchanges between neighbours are 24 vector instructions more, which hide
// behind the stores where there are no sums to form.  us, graph replays, other order / so: int8 197 x 768 x 768 4.09 / 3.81, 1576 x 768 x 768
// 5.96 / 5.53, 64 x 64 x 64 3.09 / 2.86.  Protected tiles 0.98 to 1.03 and items 1.00 to 1.01 of their time, so they keep the other.
// a lane's row of pass 0, the rows from one pass to the next, and its first column
template <int DT, bool QUADS = false> __device__ __forceinline__ int out_row(int lane) { return lane & (QUADS ? 28 : Traits<DT>::OS == 4 ? 7 : 15); }
template <int DT, bool QUADS = false> constexpr int out_step() { return QUADS ? 1 : 32 / out_passes<DT>(); }
template <int DT, bool QUADS = false> __device__ __forceinline__ int out_col(int lane)
{
    if constexpr (QUADS) return 4 * (lane & 3) + 16 * (lane >> 5);
    else if constexpr (Traits<DT>::OS == 4) return 16 * ((lane >> 3) & 1) + 8 * ((lane >> 4) & 1) + 4 * (lane >> 5);
    else return 16 * ((lane >> 4) & 1) + 8 * (lane >> 5);
}
// lo: x in lanes with `up` clear, in the others the y of the lane that CTRL pairs with theirs; hi: what is left of both
template <int CTRL> __device__ __forceinline__ void swap_lanes(uint32_t x, uint32_t y, bool up, uint32_t *lo, uint32_t *hi)
{
    const uint32_t xs = (uint32_t)dpp_get<CTRL>((int)x), ys = (uint32_t)dpp_get<CTRL>((int)y);
    *lo = up ? ys : x;
    *hi = up ? y : xs;
}
// A lane's row is bits 0..4 of its number and its columns 16 q1 + 8 q0 + 4 (lane >> 5) + j (word 8 q1 + 4 q0 + j).  q1 changes place with bit 5, what was
// bit 5 with bit 0, q0 with bit 1: the low two bits of the row number the passes.
__device__ __forceinline__ void turn_quads(const uint32_t *w, i32x4 (&out)[4], int lane)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t t[2][2], even[2], odd[2], r[4];             // t: [what was bit 5][q0]
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            auto p = __builtin_amdgcn_permlane32_swap(w[4 * q + j], w[8 + 4 * q + j], false, false);
            t[0][q] = p[0];
            t[1][q] = p[1];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) swap_lanes<0xB1>(t[0][q], t[1][q], (lane & 1) != 0, &even[q], &odd[q]);
        swap_lanes<0x4E>(even[0], even[1], (lane & 2) != 0, &r[0], &r[2]);
        swap_lanes<0x4E>(odd[0], odd[1], (lane & 2) != 0, &r[1], &r[3]);
#pragma unroll
        for (int p = 0; p < 4; ++p) out[p][j] = (int)r[p];
    }
}
template <int DT> __device__ __forceinline__ void turn_block(const uint32_t *w, i32x4 (&out)[out_passes<DT>()])
{
    constexpr int OS = Traits<DT>::OS;
    if constexpr (OS == 4) {
        i32x4 s[2][2];                           // [half of the columns][rows 0..15, 16..31]
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                auto p = __builtin_amdgcn_permlane16_swap(w[8 * h + j], w[8 * h + 4 + j], false, false);
                s[h][0][j] = (int)p[0];
                s[h][1][j] = (int)p[1];
            }
        // lanes with bit 3 clear: the first half of row (lane & 7), of row (lane & 7) + 8; the others the second
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                out[2 * r][j] = __builtin_amdgcn_update_dpp(s[0][r][j], s[1][r][j], 0x128, 0xF, 0xC, false);
                out[2 * r + 1][j] = __builtin_amdgcn_update_dpp(s[1][r][j], s[0][r][j], 0x128, 0xF, 0x3, false);
            }
    } else {
        uint32_t u[4], v[4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            auto p = __builtin_amdgcn_permlane32_swap(w[j], w[2 + j], false, false);
            u[j] = p[0]; u[2 + j] = p[1];
            auto q = __builtin_amdgcn_permlane32_swap(w[4 + j], w[6 + j], false, false);
            v[j] = q[0]; v[2 + j] = q[1];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            auto p = __builtin_amdgcn_permlane16_swap(u[j], v[j], false, false);
            out[0][j] = (int)p[0];
            out[1][j] = (int)p[1];
        }
    }
}

}  // namespace abft
