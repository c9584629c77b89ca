// Input-side checksums of A taken from the operand slabs the GEMM already holds in LDS.
//
// The checksum scheme (Sec. III-B.1 "Checksums") needs two reductions of A: the column sums
// a = e^T A (which give the column checksum prediction (e^T A) B) and the matrix-vector product
// A (B e) (the row checksum prediction).  Both read every element of A exactly once, and every
// element of A passes through LDS on its way to the matrix cores anyway: of the workgroups that
// share a tile row, the one in tile column (s mod tiles_n) reduces slab s while it is resident.
// So A is read from memory once, by the GEMM.  The fast kernel does it unless its tiles leave compute units
// idle (those then run a_beside below), the general one for large problems (small ones form the
// checksums beside their tiles: encode_pass.h).
//
// LDS slab layout (both GEMM kernels): row r is 128 bytes = eight 16-byte chunks, chunk c stored
// in slot c ^ ((r >> 1) & 7).  The general kernel reduces it element by element, thread t chunk c = t & 7 of rows
// (t >> 3) + 32 p (a_pass); the fast kernel by matrix instructions on the fragments (FastPass below).
#pragma once
#include <type_traits>

#include "abft_device.h"
#include "gemm_args.h"

namespace abft {

template <int I, int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

constexpr int FAST_WAVES = 8;                         // of a workgroup of the fast kernel

// Sum over each aligned group of 8 lanes; every lane of the group ends with the total.
template <typename T> __device__ __forceinline__ T row8_sum(T v)
{
    v = add_t(v, dpp_get<0xB1>(v));    // lane ^ 1
    v = add_t(v, dpp_get<0x4E>(v));    // lane ^ 2
    v = add_t(v, dpp_get<0x141>(v));   // i <-> 7 - i inside 8 lanes
    return v;
}

// LDS atomic add on a 32-bit checksum word, written as the instruction itself.  Through the
// compiler's atomicAdd every one of these is preceded by a wait for ALL outstanding memory
// operations of the wave: the operand loads of the next slab go straight into LDS
// (global_load_lds) and the compiler, which cannot tell their target from this word, orders the
// atomic behind them -- the pass then stalls for a full load latency in every slab it reduces.
// The words added to here are never a target of those loads.
__device__ __forceinline__ void lds_add_word(uint32_t *p, float v)
{
    const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)p;
    asm volatile("ds_add_f32 %0, %1" :: "v"(a), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_add_word(uint32_t *p, int v)
{
    const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)p;
    asm volatile("ds_add_u32 %0, %1" :: "v"(a), "v"(v) : "memory");
}

// Per-thread state of the A pass that lives across the slabs of one tile.
template <int DT> struct APassState {
    typename Traits<DT>::acc_t rdot;   // dot of row (t >> 3) + 32 (t & 7) with b, over the owned slabs
    float amax;                        // max |A| seen (floating point only)
};

// LDS the pass needs for a tile besides the operand buffers: for every owned slab KE words of
// column sums and KE words of b (staged once, at the start of the tile, zero beyond K).
__host__ __device__ inline int apass_owned_slabs(int nslab, int tiles_n) { return (nslab + tiles_n - 1) / tiles_n; }
__host__ __device__ inline size_t apass_lds_bytes(int dt, int nslab, int tiles_n)
{
    return (size_t)apass_owned_slabs(nslab, tiles_n) * (SLAB_BYTES / elem_size(dt)) * 8;
}
// Reduce one resident slab of A.  sA: the slab in LDS (BM rows).  b_lds: the KE values of b
// that belong to the slab (LDS).  rows_valid: rows of the tile inside M (rows beyond may hold
// anything, finite or not: they are ignored).  col_lds: KE words of this slab's column sums.
// keep: bytes of a row of the slab that are inside K.
// GIVEN: the caller supplied a = e^T A and max|A| (a checksum carried over from the kernel that
// produced A): only the row dots are formed.
// int8: |b| < 2^23 (the callers' N is below 65536).
template <int DT, int BM, bool GIVEN>
__device__ __forceinline__ void a_pass(const uint8_t *sA, const uint32_t *b_lds, int rows_valid,
                                       uint32_t *col_lds, APassState<DT> &st, int keep = SLAB_BYTES)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int CE = 16 / T::ES;
    constexpr int P = BM / 32;
    const int tid = tile_thread_index();
    const int c = tid & 7, rg = tid >> 3;
    const uint8_t *src = sA + rg * SLAB_BYTES + ((c ^ ((rg >> 1) & 7)) * 16);

    acc_t bv[CE], cs[CE];
#pragma unroll
    for (int q4 = 0; q4 < CE / 4; ++q4) {
        const i32x4 w = *reinterpret_cast<const i32x4 *>(b_lds + c * CE + 4 * q4);
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[4 * q4 + e] = from_word<acc_t>((uint32_t)w[e]);
    }
#pragma unroll
    for (int q = 0; q < CE; ++q) cs[q] = T::zero();
    i32x4 v[P];
#pragma unroll
    for (int p = 0; p < P; ++p) v[p] = *reinterpret_cast<const i32x4 *>(src + p * 32 * SLAB_BYTES);
    if (keep < SLAB_BYTES) {
#pragma unroll
        for (int p = 0; p < P; ++p) v[p] = mask_chunk(v[p], keep - c * 16);
    }
    acc_t mine = T::zero();
    if constexpr (T::IS_INT) {
        // |b| <= 128 N < 2^23: b = 256 hi + lo with 0 <= lo < 256 and |hi| < 2^15.  The bytes of a
        // word of A as two pairs of 16-bit integers (bytes 0, 2 and bytes 1, 3): the column sums
        // add pair-wise (at most 8 rows per thread), the row product takes two products per
        // instruction against the pairs of hi and of lo.
        typedef short s16x2 __attribute__((ext_vector_type(2)));
        s16x2 bhi[8], blo[8], csp[8];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int b0 = (int)bv[4 * d], b1 = (int)bv[4 * d + 1], b2 = (int)bv[4 * d + 2], b3 = (int)bv[4 * d + 3];
            bhi[2 * d] = s16x2{(short)(b0 >> 8), (short)(b2 >> 8)};
            bhi[2 * d + 1] = s16x2{(short)(b1 >> 8), (short)(b3 >> 8)};
            blo[2 * d] = s16x2{(short)(b0 & 255), (short)(b2 & 255)};
            blo[2 * d + 1] = s16x2{(short)(b1 & 255), (short)(b3 & 255)};
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) csp[j] = s16x2{0, 0};
#pragma unroll
        for (int p = 0; p < P; ++p) {
            i32x4 x4 = v[p];
            if (rg + 32 * p >= rows_valid) x4 = i32x4{0, 0, 0, 0};
            int dhi = 0, dlo = 0;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int wd = x4[d];
                const s16x2 w = s16x2{(short)(wd & 0xFFFF), (short)(wd >> 16)};
                const s16x2 ev = (w << 8) >> 8, od = w >> 8;       // bytes 0, 2 and 1, 3, sign-extended
                if (!GIVEN) {
                    csp[2 * d] += ev;
                    csp[2 * d + 1] += od;
                }
                dhi = __builtin_amdgcn_sdot2(ev, bhi[2 * d], dhi, false);
                dhi = __builtin_amdgcn_sdot2(od, bhi[2 * d + 1], dhi, false);
                dlo = __builtin_amdgcn_sdot2(ev, blo[2 * d], dlo, false);
                dlo = __builtin_amdgcn_sdot2(od, blo[2 * d + 1], dlo, false);
            }
            acc_t dot = (acc_t)(int)((uint32_t)dhi * 256u + (uint32_t)dlo);
            dot = row8_sum(dot);
            if (c == p) mine = dot;
        }
#pragma unroll
        for (int q = 0; q < CE; ++q) cs[q] = (acc_t)csp[2 * (q >> 2) + (q & 1)][(q >> 1) & 1];
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            i32x4 x4 = v[p];
            if (rg + 32 * p >= rows_valid) x4 = i32x4{0, 0, 0, 0};
            acc_t dot = T::zero();
#pragma unroll
            for (int q = 0; q < CE; ++q) {
                const acc_t x = T::elem(x4, q);
                if (!GIVEN) cs[q] = add_t(cs[q], x);
                dot = __builtin_fmaf((float)x, (float)bv[q], (float)dot);
                if (!GIVEN) st.amax = fmaxf(st.amax, fabsf((float)x));
            }
            dot = row8_sum(dot);
            if (c == p) mine = dot;
        }
    }
    st.rdot = add_t(st.rdot, mine);
    if constexpr (GIVEN) return;
    // Column sums: first over the eight row groups of the wave (lanes with equal c), then one
    // LDS atomic per column and wave.  (LDS atomics in which several lanes of one instruction
    // hit the same word are served one lane at a time.)
#pragma unroll
    for (int q = 0; q < CE; ++q) {
        acc_t t = cs[q];
        t = add_t(t, dpp_get<0x128>(t));      // row_ror:8 inside 16 lanes: lane ^ 8
        t = add_xor16(t);
        t = add_xor32(t);
        cs[q] = t;
    }
    if ((tid & 63) < 8) {
#pragma unroll
        for (int q = 0; q < CE; ++q) {
            lds_add_word(col_lds + c * CE + q, cs[q]);
        }
    }
}

// ---- The fast kernel's form of the pass: matrix instructions on the MFMA fragments of the slab.
// A 16 x 16 MFMA takes lane l of a 32-row fragment for row l & 15 and piece l >> 4 along its own K, so rows r and r + 16 meet
// in one sum.  Times the identity, positions along K come out in the lanes, to be added up over rows (four registers and two
// exchanges per slab); times b, split into terms that the operand type holds exactly, the dots of the fragment's 32 rows do, a
// term to a register.  (The item kernels do the same: gemm_item.h.)  The four waves that share rows of A take a step
// of the slab each.  Per owned slab of a 256-row tile that is eight MFMAs of 16 clocks (int8 twelve) and some seventy-five
// vector instructions of one wave in four, where element by element it was two hundred of every wave.  int8 36928 x 1024 x 4096
// (eight to a tile): the launch 171.9 -> 156 us.
// Products with one are exact, and so are those with b's terms before they are added.  But Inf and NaN reach through
// products with zeros what they have no part in, and a NaN hides the largest |element| of a lane: sums, dots and maxima that are not
// finite are formed again, element by element, from memory (dots_again, columns_again, amax_again).
//
// LDS: the column sums of every owned slab; b in three terms, of two slabs in turn; 128 bytes of zeros; words of b, of two slabs in turn.
__host__ __device__ inline size_t fast_aux_bytes(int dt, int nslab, int tiles_n)
{
    return (size_t)(apass_owned_slabs(nslab, tiles_n) + 2) * (SLAB_BYTES / elem_size(dt)) * 4 + (2 * 3 + 1) * SLAB_BYTES;
}

// The operand of ones that turns a fragment: of positions 0..15 of a step (16-bit types), of 16 u .. + 15 (int8).
template <int DT> __device__ __forceinline__ i32x4 turn_operand(int lane, int u)
{
    constexpr int ONE = DT == DT_BF16 ? 0x3F80 : 0x3C00;
    const int j = lane & 15, lh = lane >> 5, pos = j - 8 * lh;
    i32x4 f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (DT == DT_I8) f[w] = lh == u && (j >> 2) == w ? 1 << (8 * (j & 3)) : 0;
        else f[w] = pos == 2 * w ? ONE : pos == 2 * w + 1 ? (int)((unsigned)ONE << 16) : 0;
    }
    return f;
}

// Term d = 0, 1, 2 of b, as bits of the operand type; what is left of it in v.  int8: signed bytes, which hold up to 0x7F7F7F
// (N below 65536, see gemm_fast_eligible: b is 127 * 65535 = 0x7EFF81 at most, and -128 * 65535 at least).  bf16: three times
// eight bits, cut off and not rounded (a value near the largest must not become Inf).  fp16: of b times a power of two that
// brings N values of the type below 2^15, and each rest times 2^11, so that it does not sink below the type's range: the last
// bit of the last term is 2^-45 N (N as a power of two), below that of any sum of fp16 values.  (Rests as they are would leave off
// 2^-40 of the largest b: all of the b of a column whose elements are small.)
constexpr float F16_REST = 2048.f;
template <int DT> __device__ __forceinline__ uint32_t b_term(typename Traits<DT>::acc_t &v)
{
    if constexpr (DT == DT_I8) {
        const int lo = (int)(int8_t)(v & 0xFF);
        v = (v - lo) >> 8;
        return (uint32_t)lo & 0xFFu;
    } else if constexpr (DT == DT_BF16) {
        const uint32_t hi = __float_as_uint(v) & 0xFFFF0000u;
        v -= __uint_as_float(hi);
        return hi >> 16;
    } else {
        const uint32_t h = f32_to_f16_bits(v);
        v = (v - f16_bits_to_f32(h)) * F16_REST;
        return h;
    }
}
// fp16: that power of two, and what undoes it
__device__ __forceinline__ void b_scale(int N, float *scale, float *back)
{
    const int e = 16 + 32 - __builtin_clz((unsigned)N - 1);     // N values below 2^16: b below 2^e
    *scale = __uint_as_float((uint32_t)(127 + 15 - e) << 23);
    *back = __uint_as_float((uint32_t)(127 - 15 + e) << 23);
}

// d0 += b x[0], d1 += b x[1] and c = x[0], x[1] turned and added up; operands and results in vector registers.  As instructions: the
// built-in's results would be given accumulation registers in the kernels that keep their accumulators there, which the tile fills.  The waits cover what the compiler does not
// see in here: operands written by vector instructions just ahead, results read right behind.
template <int DT> struct TurnSums { typename Acc4<DT>::type c[2]; };
#define ABFT_M16(OP, D, A, B, C) OP " %" D ", %" A ", %" B ", " C "\n\t"
template <int DT>
__device__ __forceinline__ void pass_mfmas(typename Acc4<DT>::type &d0, typename Acc4<DT>::type &d1, TurnSums<DT> &ts, const i32x4 (&x)[2],
                                           const i32x4 &b, const i32x4 &id0, const i32x4 &id1)
{
    if constexpr (DT == DT_I8) {
        // c[0]: positions 0..15 of the step, c[1]: 16..31
        asm volatile("s_nop 4\n\t"
                     ABFT_M16("v_mfma_i32_16x16x64_i8", "0", "4", "7", "0") ABFT_M16("v_mfma_i32_16x16x64_i8", "1", "4", "8", "0")
                     ABFT_M16("v_mfma_i32_16x16x64_i8", "2", "6", "4", "%2") ABFT_M16("v_mfma_i32_16x16x64_i8", "3", "6", "5", "%3") "s_nop 7\n\t"
                     ABFT_M16("v_mfma_i32_16x16x64_i8", "0", "5", "7", "%0") ABFT_M16("v_mfma_i32_16x16x64_i8", "1", "5", "8", "%1")
                     "s_nop 15\n\ts_nop 3"
                     : "=&v"(ts.c[0]), "=&v"(ts.c[1]), "+v"(d0), "+v"(d1)
                     : "v"(x[0]), "v"(x[1]), "v"(b), "v"(id0), "v"(id1));
    } else {
        // c[0] of x[0], c[1] of x[1]; the caller adds them
#define ABFT_PASS16(OP)                                                                                                             \
        asm volatile("s_nop 4\n\t"                                                                                                  \
                     ABFT_M16(OP, "0", "4", "7", "0") ABFT_M16(OP, "1", "5", "7", "0")                                              \
                     ABFT_M16(OP, "2", "6", "4", "%2") ABFT_M16(OP, "3", "6", "5", "%3")                                            \
                     "s_nop 15\n\ts_nop 3"                                                                                          \
                     : "=&v"(ts.c[0]), "=&v"(ts.c[1]), "+v"(d0), "+v"(d1)                                                           \
                     : "v"(x[0]), "v"(x[1]), "v"(b), "v"(id0))
        if constexpr (DT == DT_BF16) ABFT_PASS16("v_mfma_f32_16x16x32_bf16");
        else ABFT_PASS16("v_mfma_f32_16x16x32_f16");
#undef ABFT_PASS16
    }
}
#undef ABFT_M16

// What the pass leaves of a tile.
template <int DT, int MI> struct FastPass {
    typedef typename Traits<DT>::acc_t acc_t;
    typename Acc4<DT>::type dot[MI];   // lane l < 32, registers 0, 1, 2: products of row l of block mi with the terms of b, over the owned slabs
    uint32_t amax;                     // 16-bit types: largest |element| as bits, in either half
    // the dot of row lane & 31 (lanes 0..31) of block mi over what this wave has taken
    __device__ __forceinline__ acc_t total(int mi) const
    {
        if constexpr (DT == DT_I8) return (int)((uint32_t)dot[mi][0] + ((uint32_t)dot[mi][1] << 8) + ((uint32_t)dot[mi][2] << 16));
        else {
            constexpr float REST = DT == DT_F16 ? 1.f / F16_REST : 1.f;
            return __builtin_fmaf(__builtin_fmaf((float)dot[mi][2], REST, (float)dot[mi][1]), REST, (float)dot[mi][0]);
        }
    }
};

// The same reductions by a workgroup of its own, for a launch whose tiles leave compute units idle: rows
// rb * rpb .. of A, a window of 2^cw_log2 16-byte chunks along K.  A thread keeps one chunk column (its values of b
// and its column sums stay in registers) and takes UN consecutive rows at a time, all UN loads in flight:
// 64 KB per compute unit, bound by the latency of memory and not by the 40-odd vector instructions per
// chunk.  smem: 64 FAST_WAVES * (16 / element size) words.  K is a whole number of slabs: no chunk is cut.
template <int DT>
__device__ __forceinline__ void a_beside(const GemmArgs &g, int blk, uint8_t *smem)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int CE = 16 / T::ES, UN = 8;
    const int per_item = g.beside.nwin * g.beside.nrb;
    const int bz = blk / per_item, in_item = blk - bz * per_item;
    const int rb = in_item / g.beside.nwin, win = in_item - rb * g.beside.nwin;
    const int tid = threadIdx.x;
    const int CW = 1 << g.beside.cw_log2, RL = 64 * FAST_WAVES >> g.beside.cw_log2;
    const int cx = tid & (CW - 1), ry = tid >> g.beside.cw_log2;
    const int col0 = (win * CW + cx) * CE;
    const bool colok = col0 < g.K;
    const uint8_t *src = g.A + ((long)bz * g.sA + (colok ? col0 : 0)) * T::ES;
    const int rbeg = rb * g.beside.rpb, rend = min(rbeg + g.beside.rpb, g.M);
    const long ldb = g.lda * T::ES;

    acc_t bv[CE], cs[CE];
#pragma unroll
    for (int e = 0; e < CE; ++e) {
        bv[e] = colok ? from_word<acc_t>(g.b_sum[(long)bz * g.K + col0 + e]) : T::zero();
        cs[e] = T::zero();
    }
    float amax = 0.f;
    for (int r0 = rbeg; r0 < rend; r0 += RL * UN) {
        const int rt = r0 + ry * UN;                            // this thread's rows: rt .. rt + UN
        i32x4 v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int r = min(rt + u, g.M - 1);                 // loads without a branch: rows past the end are cleared below
            v[u] = *reinterpret_cast<const i32x4 *>(src + (long)r * ldb);
        }
        acc_t part[CE], mine = T::zero();                       // the batch's column sums; the dot of row cx
#pragma unroll
        for (int e = 0; e < CE; ++e) part[e] = T::zero();
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            i32x4 x4 = v[u];
            if (!colok || rt + u >= rend) x4 = i32x4{0, 0, 0, 0};
            acc_t dot = T::zero();
#pragma unroll
            for (int e = 0; e < CE; ++e) {
                const acc_t x = T::elem(x4, e);
                part[e] = add_t(part[e], x);
                if constexpr (T::IS_INT) {
                    dot += __mul24((int)x, (int)bv[e]);         // |b| < 2^23 (gemm_fast_eligible)
                } else {
                    dot = __builtin_fmaf((float)x, (float)bv[e], (float)dot);
                    amax = fmaxf(amax, fabsf((float)x));
                }
            }
            dot = seg_sum(dot, CW);
            if (cx == u) mine = dot;
        }
#pragma unroll
        for (int e = 0; e < CE; ++e) cs[e] = add_t(cs[e], part[e]);
        if (cx < UN && rt + cx < rend) atomic_add_word(g.rc_pred + (long)bz * g.M + rt + cx, mine);
    }
    if (g.a_given) return;
    acc_t *red = reinterpret_cast<acc_t *>(smem);
#pragma unroll
    for (int e = 0; e < CE; ++e) red[(ry * CW + cx) * CE + e] = cs[e];
    __syncthreads();
    for (int c = tid; c < CW * CE; c += 64 * FAST_WAVES) {
        const int k = win * CW * CE + c;
        if (k < g.K) {
            acc_t t = red[c];
            for (int y = 1; y < RL; ++y) t = add_t(t, red[y * CW * CE + c]);
            atomic_add_word(g.a_sum + (long)bz * g.K + k, t);
        }
    }
    if constexpr (!T::IS_INT) {
        amax = wave_max(amax);
        if ((tid & 63) == 0 && amax > 0.f) atomicMax(g.a_max + bz, __float_as_uint(amax));
    }
}

}  // namespace abft
