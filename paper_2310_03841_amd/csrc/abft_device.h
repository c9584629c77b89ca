// Device-side helpers for gfx950 (64-wide wavefronts, MFMA, DPP).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "abft_internal.h"

namespace abft {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

// The thread's index inside its workgroup, as a value the optimiser cannot move or merge.  Code
// that runs once per tile inside a loop over tiles derives dozens of per-lane addresses from
// it; taken from the plain built-in they are all computed once before the loop and held in
// registers across it (40 more vector registers in the fast GEMM kernel).
__device__ __forceinline__ int tile_thread_index()
{
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// A kernel's arguments (its first parameter), read from where the launch put them: each phase of a tile or item takes its own.  Taken from
// the parameter, every argument and every offset, pitch and condition that follows from them is formed ahead of the loop over tiles
// or items and held across it: too many scalars, which go to lanes of vector registers and come back one by one.
template <typename ARGS> __device__ __forceinline__ const ARGS &kernel_args()
{
    const __attribute__((address_space(4))) ARGS *p = (const __attribute__((address_space(4))) ARGS *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const ARGS *)p;
}

// Asks for every 64-byte line of a kernel's arguments at once, first thing.  A launch's arguments lie in memory, and a line that is touched for
// the first time takes a compute unit some 500 clocks (0.22 us); left alone, the compiler loads each argument where it is used, and the
// kernels of a small call went through three to five such trips one behind the other.  BYTES: of which a kernel reads the first ones only.
template <typename ARGS, int BYTES = (int)sizeof(ARGS)> __device__ __forceinline__ void fetch_args()
{
    const __attribute__((address_space(4))) uint32_t *p = (const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LINES = (BYTES + 63) / 64;
    static_assert(LINES <= 16, "one wait for all");
    uint32_t v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = i < LINES ? p[16 * i] : 0u;
    if constexpr (LINES <= 4) asm volatile("" :: "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]));
    else if constexpr (LINES <= 8) asm volatile("" :: "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]));
    else asm volatile("" :: "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]), "s"(v[8]), "s"(v[9]), "s"(v[10]),
                            "s"(v[11]), "s"(v[12]), "s"(v[13]), "s"(v[14]), "s"(v[15]));
}

// ---------------------------------------------------------------- conversions
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// fp32 -> bf16, round to nearest even; NaN stays NaN (quiet).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if (f != f) return (u >> 16) | 0x0040u;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

__device__ __forceinline__ float f16_bits_to_f32(uint32_t h)
{
    _Float16 x = __builtin_bit_cast(_Float16, (uint16_t)h);
    return (float)x;
}

// fp32 -> fp16, round to nearest even (the conversion instruction's default mode).
__device__ __forceinline__ uint32_t f32_to_f16_bits(float f)
{
    _Float16 x = (_Float16)f;
    return (uint32_t)__builtin_bit_cast(uint16_t, x);
}

// ---------------------------------------------------------------- per-dtype traits
template <int DT> struct Traits;

template <> struct Traits<DT_I8> {
    typedef int acc_t;
    typedef i32x16 accv_t;
    static constexpr int ES = 1;       // bytes per operand element
    static constexpr int OS = 4;       // bytes per output element
    static constexpr bool IS_INT = true;
    // one 32x32 MFMA step consumes 32 bytes of K per row (16 per half-wave)
    __device__ static __forceinline__ accv_t mfma(i32x4 a, i32x4 b, accv_t c)
    {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ int elem(const i32x4 &v, int e)   // element e of a 16-byte chunk
    {
        return (int)(int8_t)((uint32_t)v[e >> 2] >> (8 * (e & 3)));
    }
    __device__ static __forceinline__ void store_c(void *C, long idx, acc_t v) { ((int *)C)[idx] = v; }
    __device__ static __forceinline__ acc_t load_c(const void *C, long idx) { return ((const int *)C)[idx]; }
    __device__ static __forceinline__ acc_t zero() { return 0; }
};

template <> struct Traits<DT_BF16> {
    typedef float acc_t;
    typedef f32x16 accv_t;
    static constexpr int ES = 2;
    static constexpr int OS = 2;
    static constexpr bool IS_INT = false;
    __device__ static __forceinline__ accv_t mfma(i32x4 a, i32x4 b, accv_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    __device__ static __forceinline__ float elem(const i32x4 &v, int e)
    {
        uint32_t w = (uint32_t)v[e >> 1];
        return __uint_as_float((e & 1) ? (w & 0xFFFF0000u) : (w << 16));
    }
    __device__ static __forceinline__ void store_c(void *C, long idx, acc_t v)
    {
        ((uint16_t *)C)[idx] = (uint16_t)f32_to_bf16_bits(v);
    }
    __device__ static __forceinline__ acc_t load_c(const void *C, long idx)
    {
        return bf16_bits_to_f32(((const uint16_t *)C)[idx]);
    }
    __device__ static __forceinline__ acc_t zero() { return 0.f; }
};

template <> struct Traits<DT_F16> {
    typedef float acc_t;
    typedef f32x16 accv_t;
    static constexpr int ES = 2;
    static constexpr int OS = 2;
    static constexpr bool IS_INT = false;
    __device__ static __forceinline__ accv_t mfma(i32x4 a, i32x4 b, accv_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
    __device__ static __forceinline__ float elem(const i32x4 &v, int e)
    {
        uint32_t w = (uint32_t)v[e >> 1];
        return f16_bits_to_f32((e & 1) ? (w >> 16) : (w & 0xFFFFu));
    }
    __device__ static __forceinline__ void store_c(void *C, long idx, acc_t v)
    {
        ((uint16_t *)C)[idx] = (uint16_t)f32_to_f16_bits(v);
    }
    __device__ static __forceinline__ acc_t load_c(const void *C, long idx)
    {
        return f16_bits_to_f32(((const uint16_t *)C)[idx]);
    }
    __device__ static __forceinline__ acc_t zero() { return 0.f; }
};

// ---------------------------------------------------------------- 16 x 16 MFMA: 64 bytes of K per row, four registers
// Lane l of an operand holds row l & 15 and the 16-byte piece l >> 4 along K; of the result, column l & 15
// (row of b) and rows 4 (l >> 4) + register.
template <int DT> struct Acc4 { typedef __attribute__((ext_vector_type(4))) float type; };
template <> struct Acc4<DT_I8> { typedef i32x4 type; };
template <int DT>
__device__ __forceinline__ typename Acc4<DT>::type mfma16(const i32x4 &a, const i32x4 &b, const typename Acc4<DT>::type &c)
{
    if constexpr (DT == DT_I8)
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
    else if constexpr (DT == DT_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <int DT> __device__ __forceinline__ typename Acc4<DT>::type acc4_zero()
{
    return typename Acc4<DT>::type{0, 0, 0, 0};
}
// ---------------------------------------------------------------- 32-bit word views of checksum values
__device__ __forceinline__ uint32_t as_word(int v) { return (uint32_t)v; }
__device__ __forceinline__ uint32_t as_word(float v) { return __float_as_uint(v); }
template <typename T> __device__ __forceinline__ T from_word(uint32_t w);
template <> __device__ __forceinline__ int from_word<int>(uint32_t w) { return (int)w; }
template <> __device__ __forceinline__ float from_word<float>(uint32_t w) { return __uint_as_float(w); }

// Device-scope atomic add on a 32-bit checksum word (integer: wraps modulo 2^32).
__device__ __forceinline__ void atomic_add_word(uint32_t *p, int v) { atomicAdd((int *)p, v); }
__device__ __forceinline__ void atomic_add_word(uint32_t *p, float v) { unsafeAtomicAdd((float *)p, v); }

// ---------------------------------------------------------------- wave-level reductions (DPP)
template <int CTRL> __device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
__device__ __forceinline__ int add_t(int a, int b) { return a + b; }
__device__ __forceinline__ float add_t(float a, float b) { return a + b; }
template <int CTRL> __device__ __forceinline__ int dpp_get(int v) { return dpp_mov<CTRL>(v); }
template <int CTRL> __device__ __forceinline__ float dpp_get(float v)
{
    return __int_as_float(dpp_mov<CTRL>(__float_as_int(v)));
}

// Exchange between the rows of 16 lanes and between the halves of a wave with the row-swap
// instructions of gfx950 (v_permlane16_swap, v_permlane32_swap: vector ALU, no trip through the
// LDS crossbar as a lane shuffle takes).  Called with the same value twice, the two results
// hold, lane by lane, the lane's own value and that of lane ^ 16 (lane ^ 32), in either order.
__device__ __forceinline__ int add_xor16(int v)
{
    auto p = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return (int)(p[0] + p[1]);
}
__device__ __forceinline__ int add_xor32(int v)
{
    auto p = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return (int)(p[0] + p[1]);
}
__device__ __forceinline__ float add_xor16(float v)
{
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float add_xor32(float v)
{
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float max_xor16(float v)
{
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float max_xor32(float v)
{
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}

// Sum over each aligned group of 16 lanes; every lane of the group ends with the total.
template <typename T> __device__ __forceinline__ T row16_sum(T v)
{
    v = add_t(v, dpp_get<0xB1>(v));    // quad_perm [1,0,3,2]: lane ^ 1
    v = add_t(v, dpp_get<0x4E>(v));    // quad_perm [2,3,0,1]: lane ^ 2
    v = add_t(v, dpp_get<0x141>(v));   // row_half_mirror: i <-> 7 - i inside 8 lanes
    v = add_t(v, dpp_get<0x140>(v));   // row_mirror: i <-> 15 - i inside 16 lanes
    return v;
}

// Sum over each half-wave (lanes 0..31 and 32..63); every lane of the half ends with the total.
template <typename T> __device__ __forceinline__ T half_wave_sum(T v)
{
    v = row16_sum(v);
    return add_xor16(v);
}

// Sum over the whole wave; every lane ends with the total.
template <typename T> __device__ __forceinline__ T wave_sum(T v)
{
    v = half_wave_sum(v);
    return add_xor32(v);
}

// Sum over aligned groups of `width` lanes (8, 16, 32 or 64); every lane of a group ends with
// the total.
template <typename V> __device__ __forceinline__ V seg_sum(V v, int width)
{
    v = add_t(v, dpp_get<0xB1>(v));    // lane ^ 1
    v = add_t(v, dpp_get<0x4E>(v));    // lane ^ 2
    v = add_t(v, dpp_get<0x141>(v));   // i <-> 7 - i inside 8 lanes
    if (width >= 16) v = add_t(v, dpp_get<0x140>(v));   // i <-> 15 - i inside 16 lanes
    if (width >= 32) v = add_xor16(v);
    if (width >= 64) v = add_xor32(v);
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_get<0xB1>(v));    // lane ^ 1
    v = fmaxf(v, dpp_get<0x4E>(v));    // lane ^ 2
    v = fmaxf(v, dpp_get<0x141>(v));   // i <-> 7 - i inside 8 lanes
    v = fmaxf(v, dpp_get<0x140>(v));   // i <-> 15 - i inside 16 lanes
    v = max_xor16(v);
    v = max_xor32(v);
    return v;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    auto up = [&](uint32_t w) __attribute__((always_inline)) { v = w > v ? w : v; };
    up((uint32_t)dpp_mov<0xB1>((int)v));       // lane ^ 1
    up((uint32_t)dpp_mov<0x4E>((int)v));       // lane ^ 2
    up((uint32_t)dpp_mov<0x141>((int)v));      // i <-> 7 - i inside 8 lanes
    up((uint32_t)dpp_mov<0x140>((int)v));      // i <-> 15 - i inside 16 lanes
    auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = p[0] > p[1] ? p[0] : p[1];
    auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return q[0] > q[1] ? q[0] : q[1];
}

// ---------------------------------------------------------------- sums over the 32 lanes of a half-wave
__device__ __forceinline__ uint32_t item_bits(int v) { return (uint32_t)v; }
__device__ __forceinline__ uint32_t item_bits(float v) { return __float_as_uint(v); }

// lanes with bit 4 clear get a, the others b, each summed over lane and lane ^ 16
template <typename V> __device__ __forceinline__ V fold_xor16(V a, V b)
{
    auto p = __builtin_amdgcn_permlane16_swap(item_bits(a), item_bits(b), false, false);
    return add_t(from_word<V>(p[0]), from_word<V>(p[1]));
}
// lanes with up set get b, the others a, each summed with the lane that CTRL names (its `up` is the other one)
template <int CTRL, typename V> __device__ __forceinline__ V fold_dpp(V a, V b, bool up)
{
    const V keep = up ? b : a, send = up ? a : b;
    return add_t(keep, dpp_get<CTRL>(send));
}
// The sixteen values of an accumulator block, each summed over the 32 lanes of a half of the wave; the lane
// gets the value of column fold16_column(lane)
template <typename V, typename ACC> __device__ __forceinline__ V fold16(const ACC &v, int lane)
{
    V w[8], x[4], y[2];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = fold_xor16<V>(v[2 * j], v[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = fold_dpp<0x128>(w[2 * j], w[2 * j + 1], (lane & 8) != 0);
#pragma unroll
    for (int j = 0; j < 2; ++j) y[j] = fold_dpp<0x141>(x[2 * j], x[2 * j + 1], (lane & 4) != 0);
    V z = fold_dpp<0x4E>(y[0], y[1], (lane & 2) != 0);
    return add_t(z, dpp_get<0xB1>(z));
}
// column inside a 32 x 32 block of the value fold16 leaves in this lane (register i of a block holds
// column 8 (i >> 2) + 4 (lane >> 5) + (i & 3); i = 8 b1 + 4 b2 + 2 b3 + b4 in bits of the lane)
__device__ __forceinline__ int fold16_column(int lane)
{
    const int i = ((lane & 2) << 2) + (lane & 4) + ((lane >> 2) & 2) + ((lane >> 4) & 1);
    return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
}

// Sum of the layer bias over its N entries, by the whole block (every thread gets the total).
template <typename acc_t>
__device__ __forceinline__ acc_t block_bias_sum(const uint32_t *bias, int N, acc_t *red4)
{
    acc_t v = acc_t(0);
    for (int n = threadIdx.x; n < N; n += 256) v = add_t(v, from_word<acc_t>(bias[n]));
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red4[threadIdx.x >> 6] = v;
    __syncthreads();
    return add_t(add_t(red4[0], red4[1]), add_t(red4[2], red4[3]));
}

// Products of checksum values (integer: in Z/2^32).
__device__ __forceinline__ int mul_t(int x, int y) { return (int)((uint32_t)x * (uint32_t)y); }
__device__ __forceinline__ float mul_t(float x, float y) { return x * y; }

// The check of Sec. III-B.1 item (2): equality for fixed point, tolerance for floating point.
template <bool IS_INT>
__device__ __forceinline__ bool mismatch(uint32_t obs, uint32_t pred, float tol)
{
    if (IS_INT) return obs != pred;                          // equality in Z/2^32
    float d = fabsf(__uint_as_float(obs) - __uint_as_float(pred));
    return !(d <= tol);                                      // NaN and Inf always flag
}

__device__ __forceinline__ uint32_t status_of(uint32_t nr, uint32_t nc)
{
    if (nr == 0 && nc == 0) return 0u;      // clean
    if (nr == 0 || nc == 0) return 2u;      // checksum suspect
    return 1u;                              // localised
}

// Keep the first nbytes (0..16) of a 16-byte chunk, zero the rest.
__device__ __forceinline__ i32x4 mask_chunk(i32x4 v, int nbytes)
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        int keep = nbytes - 4 * w;                 // bytes of this word to keep
        uint32_t m = keep >= 4 ? 0xFFFFFFFFu : (keep <= 0 ? 0u : ((1u << (8 * keep)) - 1u));
        v[w] = (int)((uint32_t)v[w] & m);
    }
    return v;
}

}  // namespace abft
