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
// a lane's row of pass 0 (pass p: 32 / passes rows on) and its first column
template <int DT> __device__ __forceinline__ int out_row(int lane) { return lane & (Traits<DT>::OS == 4 ? 7 : 15); }
template <int DT> __device__ __forceinline__ int out_col(int lane)
{
    if constexpr (Traits<DT>::OS == 4) return 16 * ((lane >> 3) & 1) + 8 * ((lane >> 4) & 1) + 4 * (lane >> 5);
    else return 16 * ((lane >> 4) & 1) + 8 * (lane >> 5);
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
