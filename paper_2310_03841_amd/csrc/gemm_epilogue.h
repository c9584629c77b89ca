// Epilogue of the fast GEMM kernel: store C, take the observed row / column sums of the
// M x N block from the accumulators (before rounding) and add them to cc_obs / rc_obs, and
// hand over what the pass over A's slabs collected (gemm_apass.h).  Paper: output checksum
// fused with the GEMM epilogue (Sec. IV-C memory paragraph, Sec. V "Optimizations" (2)).
//
// The kernels issue their MFMAs with the B fragment as first operand, so one 32x32 block of
// accumulators is laid out "row per lane": lane l holds row (l & 31) of the block and, in
// register i, column 8*(i>>2) + 4*(l>>5) + (i&3) -- four consecutive columns per register
// quad.  Consequences:
//   * C goes out through LDS: each lane packs four converted values into one LDS write, the
//     wave reads the staged rows back 16 bytes per lane and stores whole 128/256-byte row
//     segments to global memory.
//   * row sums are in-lane adds plus one exchange between the half-waves;
//   * column sums need a reduction over the 32 lanes (rows): lanes and values are folded together (fold16), sixteen values in some 45
//     instructions.  (Transposed through LDS, bf16 12608 x 3072 x 768 73.3 us, 71.7 so; int8 8192 x 3072 x 512 35.9 / 35.5, f16 6304 x 768 x 3072 43.1 /
//     42.8; problems of many tiles that hang over the right edge 1.00 to 1.01.)
// Every loop over accumulator registers is expanded at compile time (static_for): the
// accumulators must be addressed with constant indices to stay in registers.
//
// Two paths per group of 32 rows of a wave tile.  The common one (every row and column of the
// group inside C, no flip armed) works from registers as described.  The other one (edges of
// the problem, armed flip) stages the raw 32-bit accumulators in LDS and walks them with an
// ordinary loop, so that it costs little code: straight-line code that is rarely executed still
// has to be fetched past.
//
// LDS use: each wave owns EPI_WAVE_BYTES at smem + wave * EPI_WAVE_BYTES, then the block-wide
// partial-sum arrays follow.  The caller must have passed a barrier after its last LDS read.
#pragma once
#include <type_traits>

#include "abft_device.h"
#include "gemm_args.h"
#include "gemm_apass.h"

namespace abft {

// Sums of the values as stored beside those of the accumulators: none; in a kernel of 128-row tiles only; of both tile heights.
enum { STO_NO, STO_128, STO_256 };

// bytes of wave-private LDS the epilogue needs for a wave tile that is TN columns wide
__host__ __device__ constexpr int epi_wave_bytes(int TN) { return 32 * (TN * 4 + 16); }
__host__ __device__ constexpr int epi_total_bytes(int BM, int BN)
{
    return FAST_WAVES * epi_wave_bytes(BN / 4) + (12 * BM + 5 * BN) * 4 + 8 * FAST_WAVES;      // (with stored sums: the most)
}

// One accumulator element, at the point of use.  A kernel of 512 threads has 256 registers a lane, and where nothing asks for
// accumulation registers the compiler takes all of them as vector registers: the MFMAs write there, and the epilogue's instructions
// read there.  AGPR: the kernels that have no register to spare (STO_256) keep the accumulators in 128 accumulation
// registers and read them one by one (left alone, the register allocator moves all of them at the top of the epilogue and
// spills).  us, all read one by one / so: bf16 12608 x 3072 x 768 69.1 / 68.4, 6304 x 768 x 768 unprotected 10.54 / 10.36, f16 6304 x 768 x
// 3072 42.9 / 42.6.
template <bool AGPR> __device__ __forceinline__ float acc_read(float v)
{
    if constexpr (!AGPR) return v;
    float r;
    asm("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(v));
    return r;
}
template <bool AGPR> __device__ __forceinline__ int acc_read(int v)
{
    if constexpr (!AGPR) return v;
    int r;
    asm("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(v));
    return r;
}

// pack converted outputs
// Two fp32 values -> two storage-type values in one word, round to nearest even (the packed
// conversion instructions of gfx950).
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
template <int DT> __device__ __forceinline__ uint32_t pack2(float a, float b);
template <> __device__ __forceinline__ uint32_t pack2<DT_BF16>(float a, float b)
{
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
template <> __device__ __forceinline__ uint32_t pack2<DT_F16>(float a, float b)
{
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}

// The value an accumulator becomes in memory, back as a float (round to nearest even).
template <int DT> __device__ __forceinline__ float stored_value(float v)
{
    const uint32_t w = pack2<DT>(v, 0.f) & 0xFFFFu;
    if constexpr (DT == DT_BF16) return __uint_as_float(w << 16);
    else return f16_bits_to_f32(w);
}

// What a protected tile hands to the epilogue besides its accumulators.
template <int DT, int MI> struct EpiProt {
    FastPass<DT, MI> pass;    // what the pass over the owned slabs left in registers
    const uint32_t *col_lds;  // column sums of the owned slabs (LDS)
    int owned;                // number of owned slabs: the j-th is slab slab0 + j * slab_step of K
    int slab0, slab_step;
    float back;               // fp16: what undoes the scale of b's terms
};

// Sums along K by matrix instructions that are not finite, formed again from memory.  A wave does it together, 16 bytes to a lane and
// several loads on their way: with an Inf or NaN in an operand these are some of a tile's sums (its own row or column, and what
// it reached through products with zeros) or, with one in B, the dots of all of a tile's rows.  A thread to a sum, a trip to memory for
// every element, took bf16 4096 x 4096 x 4096 with an Inf in A from 133 to 196 us, with a NaN to 171, 8200 x 512 x 640 with an
// Inf in B from 25 to 32; so 140, 140 and 28 (the element-wise pass over A in the tiles by four waves: 143, 143 and 28).

// The dots of rows row0 + r, r < 32, with b over the owned slabs, where bit r of `which` is set: to lane r, v of the others.
// Eight rows at a time, a chunk of the slab's eight to a lane.
template <int DT, int MI>
__device__ __forceinline__ float dots_again(const GemmArgs &g, const EpiProt<DT, MI> &ep, int bz, int row0, uint32_t which, float v)
{
    constexpr int KE = SLAB_BYTES / 2, UN = 4;
    const int lane = tile_thread_index() & 63;
#pragma unroll 1
    for (int r8 = 0; r8 < 32; r8 += 8) {
        if (!(which >> r8 & 0xFFu)) continue;
        const int row = row0 + r8 + (lane >> 3), at = (lane & 7) * 8;
        const uint8_t *src = g.A + ((long)bz * g.sA + (long)(row < g.M ? row : g.M - 1) * g.lda + at) * 2;
        const uint32_t *bsrc = g.b_sum + (long)bz * g.K + at;
        float dot = 0.f;
#pragma unroll 1
        for (int j0 = 0; j0 < ep.owned; j0 += UN) {
            i32x4 x[UN], b[UN][2];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int j = j0 + u < ep.owned ? j0 + u : ep.owned - 1, k = (ep.slab0 + j * ep.slab_step) * KE;
                x[u] = *reinterpret_cast<const i32x4 *>(src + 2 * k);
                b[u][0] = *reinterpret_cast<const i32x4 *>(bsrc + k);
                b[u][1] = *reinterpret_cast<const i32x4 *>(bsrc + k + 4);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u)
                if (j0 + u < ep.owned) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        dot = __builtin_fmaf((float)Traits<DT>::elem(x[u], e), __uint_as_float((uint32_t)b[u][e >> 2][e & 3]), dot);
                }
        }
        dot = __shfl(row8_sum(dot), (lane & 7) * 8);
        if ((lane >> 3) == (r8 >> 3) && (which >> lane & 1u)) v = dot;
    }
    return v;
}

// The sums of columns k0 + l of A, l < 64, over rows row0 .. + rows (at most 256), where bit l of `which` is set: to lane l, v of the
// others.  A row's chunk to a lane, all of a chunk's rows at a time.
template <int DT> __device__ __forceinline__ float columns_again(const GemmArgs &g, int bz, int row0, int rows, int k0, uint64_t which, float v)
{
    constexpr int UN = 4;
    const int lane = tile_thread_index() & 63;
#pragma unroll 1
    for (int c = 0; c < 8; ++c) {
        if (!(which >> (8 * c) & 0xFFu)) continue;
        const uint8_t *src = g.A + ((long)bz * g.sA + (long)row0 * g.lda + k0 + 8 * c) * 2;
        i32x4 x[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int r = lane + 64 * u;
            x[u] = *reinterpret_cast<const i32x4 *>(src + (long)(r < rows ? r : rows - 1) * g.lda * 2);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u)
            if (lane + 64 * u >= rows) x[u] = i32x4{0, 0, 0, 0};
        float mine = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float t = 0.f;
#pragma unroll
            for (int u = 0; u < UN; ++u) t += (float)Traits<DT>::elem(x[u], e);
            t = wave_sum(t);
            if ((lane & 7) == e) mine = t;
        }
        if ((lane >> 3) == c && (which >> lane & 1u)) v = mine;
    }
    return v;
}

// The largest |element| (bits) of those a lane saw in its pass over the owned slabs, where a NaN hides it: NaN left out.
template <int DT, int MI>
__device__ __forceinline__ uint32_t amax_again(const GemmArgs &g, const EpiProt<DT, MI> &ep, int bz, int m0, int wm, int wn)
{
    constexpr uint32_t INF_BITS = DT == DT_BF16 ? 0x7F80u : 0x7C00u;
    const int lane = tile_thread_index() & 63, row0 = m0 + wm * MI * 32 + (lane & 31);
    const uint8_t *src = g.A + (long)bz * g.sA * 2 + wn * 32 + (lane >> 5) * 16;
    uint32_t top = 0u;
#pragma unroll 1
    for (int j = 0; j < ep.owned; ++j) {
        i32x4 x[MI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int r = row0 + mi * 32;                       // (rows past the end: the last one's elements, as good as its own)
            x[mi] = *reinterpret_cast<const i32x4 *>(src + (long)(r < g.M ? r : g.M - 1) * g.lda * 2 + (long)(ep.slab0 + j * ep.slab_step) * SLAB_BYTES);
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t lo = (uint32_t)x[mi][e] & 0x7FFFu, hi = (uint32_t)x[mi][e] >> 16 & 0x7FFFu;
                if (lo <= INF_BITS && lo > top) top = lo;
                if (hi <= INF_BITS && hi > top) top = hi;
            }
    }
    return top;
}

// c += x times `elem`, r += x times `rows`, in vector registers and with waits as in pass_mfmas: the built-in's results would be
// given accumulation registers (STO_256: see acc_read), and a block of a 256-row tile's, which fills them, would go to scratch memory instead, in the main loop too.
template <int DT>
__device__ __forceinline__ void stored_mfmas(typename Acc4<DT>::type &c, typename Acc4<DT>::type &r, const i32x4 &x, const i32x4 &elem, const i32x4 &rows)
{
#define ABFT_STORED16(OP) \
    asm volatile("s_nop 4\n\t" OP " %0, %2, %3, %0\n\t" OP " %1, %2, %4, %1\n\ts_nop 15\n\ts_nop 3" : "+v"(c), "+v"(r) : "v"(x), "v"(elem), "v"(rows))
    if constexpr (DT == DT_BF16) ABFT_STORED16("v_mfma_f32_16x16x32_bf16");
    else ABFT_STORED16("v_mfma_f32_16x16x32_f16");
#undef ABFT_STORED16
}

template <int DT, int BM, bool PROT, int STO, bool BIAS>
__device__ __forceinline__ void gemm_epilogue_impl(const GemmArgs &tile, typename Traits<DT>::accv_t (&acc)[BM / 64][2],
                                              uint8_t *smem, int m0, int n0, int bz, const EpiProt<DT, BM / 64> &ep)
{
    const GemmArgs &g = PROT ? kernel_args<GemmArgs>() : tile;
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int BN = 256, THREADS = 64 * FAST_WAVES;
    constexpr int TM = BM / 2, TN = BN / 4;         // waves: two rows of four
    constexpr int MI = TM / 32, NI = TN / 32;
    constexpr int OS = T::OS;
    constexpr int KE = SLAB_BYTES / T::ES;
    static_assert(TN == 64, "a lane to a column where a wave walks a row");
    constexpr bool AGPR = STO == STO_256;
    constexpr int WAVE_BYTES = epi_wave_bytes(TN);
    constexpr int CROW = TN * OS + 16;              // staged C row (bytes), padded
    constexpr int SROW = TN * 4 + 16;               // staged 32-bit row (bytes), padded
    const int tid = tile_thread_index(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform by construction
    const int wm = wave >> 2, wn = wave & 3;
    const int l32 = lane & 31, lh = lane >> 5;
    const int M = g.M, N = g.N;

    uint8_t *wbuf = smem + wave * WAVE_BYTES;                              // wave-private staging
    acc_t *rs_part = reinterpret_cast<acc_t *>(smem + FAST_WAVES * WAVE_BYTES);      // [4][BM] by wave column
    acc_t *cs_part = rs_part + 4 * BM;                                     // [2][BN] by wave row: a place to a thread
    acc_t *rp_part = cs_part + 2 * BN;                                     // [4][BM] row dots of the A pass, by wave column
    uint32_t *amax_w = reinterpret_cast<uint32_t *>(rp_part + 4 * BM);     // largest |element| the pass saw (bits), by wave
    constexpr uint32_t DOTS_BAD = 1u << 31;                                // beside it: a dot of this wave's is not finite
    uint8_t *Cb = g.C + (long)bz * g.sC * OS;
    // layer bias of this tile's columns, staged once (zero beyond N); added to every accumulator
    // value on its way out, before the sums and before rounding
    constexpr bool has_bias = BIAS;
    acc_t *bias_lds = reinterpret_cast<acc_t *>(amax_w + FAST_WAVES);      // [BN]
    if (has_bias) {
        for (int t = tid; t < BN; t += THREADS) bias_lds[t] = n0 + t < N ? from_word<acc_t>(g.bias[n0 + t]) : T::zero();
        __syncthreads();
    }
    if (PROT && ep.owned > 0) {
        // what the pass over A's slabs left in registers (nothing in a tile that reduced no slab: where K has fewer slabs than the
        // tile row has tiles, that is most tiles)
        bool dots_bad = false;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            acc_t v = ep.pass.total(mi);
            if constexpr (DT == DT_F16) v *= ep.back;
            if (lane < 32) rp_part[wn * BM + wm * TM + mi * 32 + lane] = v;
            // (finite, and so is the sum of four)
            if constexpr (!T::IS_INT) dots_bad |= lane < 32 && !(fabsf(v) < 0x1p125f);
        }
        if constexpr (!T::IS_INT) {
            constexpr uint32_t INF_BITS = DT == DT_BF16 ? 0x7F80u : 0x7C00u;
            const uint32_t hi = ep.pass.amax >> 16, lo = ep.pass.amax & 0xFFFFu;
            uint32_t w = hi > lo ? hi : lo;
            if (__builtin_expect(__any(w > INF_BITS), 0)) {
                const uint32_t again = amax_again<DT>(g, ep, bz, m0, wm, wn);
                if (w > INF_BITS) w = again;
            }
            w = wave_max_u32(w);
            dots_bad = __any(dots_bad);
            if (lane == 0) amax_w[wave] = w | (dots_bad ? DOTS_BAD : 0u);
        }
    }
    const bool inj_here = g.inj_b == bz && g.inj_row >= m0 && g.inj_row < m0 + BM &&
                          g.inj_col >= n0 && g.inj_col < n0 + BN;
    const int wr0 = m0 + wm * TM, wc0 = n0 + wn * TN;                      // first row / column of the wave tile
    const bool cols_full = (wc0 + TN <= N) && !inj_here;

    auto wave_sync = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    // column partials: of the groups that went the register way (block column ni, register i:
    // this lane's rows) and of the groups that were walked row by row (column `lane`)
    acc_t cp[PROT ? NI : 1][16];
    acc_t colacc = T::zero();
    // STO: sums of the values as stored (after rounding), floating point only: edge groups
    // add to these while they walk their rows; register-path groups form them by MFMA from the row
    // pieces they store (stored_sums below).
    float colacc_s = 0.f;
    float cmax_s = 0.f;                 // max|value as stored| seen by this lane (with the stored-side sums)
    typename Acc4<DT>::type dcol = acc4_zero<DT>();      // stored-side column sums of the register-path groups
    // the sums of the wave's rows and columns, by wave column and by wave row: the tile adds each up before it hands it over
    float *rs_sto = reinterpret_cast<float *>(bias_lds + BN);
    float *cs_sto = rs_sto + 4 * BM, *cmax_w = cs_sto + 2 * BN;
    if constexpr (STO) cs_sto[tid] = 0.f;                // (a place to a thread)
    // A stored row piece of a group: lane l holds 16 bytes, chunk l & 7, of row 8 it + (l >> 3).  As an
    // operand of a 16 x 16 MFMA it has (chunk, parity of the row) for rows and (row / 2, element of the chunk) along K, so
    // times "element j" it gives the columns' sums over its rows of a parity, times "row pair j" each chunk's share of
    // the rows' sums: two MFMAs for what took some nine vector instructions per value.  Products with one are exact and the
    // values themselves are the stored ones.  Inf and NaN would reach their neighbours through the
    // zeros: a group that holds one is summed element by element.
    // FULL: a kernel of 256-row tiles, which has no register left: the pieces are read from LDS once more and the products stay out
    // of the accumulation registers, 1.5 to 2.5 % of a launch where all tiles have 128 rows (bf16 2048 x 2048 x 2048 45.1 -> 46.5 us).
    constexpr bool FULL = STO == STO_256;
    auto stored_sums = [&](int mi, const i32x4 *rowv) __attribute__((always_inline)) {
        if constexpr (STO) {
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            constexpr uint32_t INF_BITS = DT == DT_BF16 ? 0x7F80u : 0x7C00u;
            constexpr uint32_t ONE = DT == DT_BF16 ? 0x3F80u : 0x3C00u;
            static_assert(OS == 2, "eight lanes to a row");
            const int ln = tile_thread_index() & 63, j = ln & 15, k4 = ln >> 4;
            float *rsto = rs_sto + wn * BM + wm * TM + mi * 32;
            i32x4 elem;
#pragma unroll
            for (int w = 0; w < 4; ++w) elem[w] = j == 2 * w ? (int)ONE : j == 2 * w + 1 ? (int)(ONE << 16) : 0;
            u16x2 mx = {0, 0};
            auto sums = dcol, drow = acc4_zero<DT>();
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const i32x4 x = FULL ? *reinterpret_cast<const i32x4 *>(wbuf + (8 * it + (ln >> 3)) * CROW + (ln & 7) * 16) : rowv[it];
                const int w = j == 4 * it + k4 ? (int)(ONE | (ONE << 16)) : 0;
                if constexpr (FULL) {
                    stored_mfmas<DT>(sums, drow, x, elem, i32x4{w, w, w, w});
                } else {
                    sums = mfma16<DT>(x, elem, sums);
                    drow = mfma16<DT>(x, i32x4{w, w, w, w}, drow);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, x[e] & 0x7FFF7FFF));
            }
            // lane l: column j = 4 it + row / 2 of rows 4 (l >> 4) .. + 4 of the result: chunks of parity l >> 5
            const float row = add_xor16(((float)drow[0] + (float)drow[1]) + ((float)drow[2] + (float)drow[3]));
            const uint32_t m = mx[0] > mx[1] ? mx[0] : mx[1];
            if (!__any(m >= INF_BITS)) {
                cmax_s = fmaxf(cmax_s, DT == DT_BF16 ? __uint_as_float(m << 16) : f16_bits_to_f32(m));
                dcol = sums;
                if (!(k4 & 1)) rsto[2 * j + (k4 >> 1)] = row;
            } else {
                // column e of the lane's chunk over its rows, then its row; loops, to cost few registers and little code
                const uint16_t *piece = reinterpret_cast<const uint16_t *>(wbuf + (ln >> 3) * CROW + (ln & 7) * 16);
#pragma unroll 1
                for (int e = 0; e < 8; ++e) {
                    float c = 0.f;
                    for (int it = 0; it < 4; ++it) {
                        const float x = (float)T::load_c(piece, 4 * it * CROW + e);
                        c += x;
                        cmax_s = fmaxf(cmax_s, fabsf(x));
                    }
                    lds_add_word(reinterpret_cast<uint32_t *>(cs_sto) + wm * BN + wn * TN + 8 * (ln & 7) + e, c);
                }
#pragma unroll 1
                for (int it = 0; it < 4; ++it) {
                    float s = 0.f;
                    for (int e = 0; e < 8; ++e) s += (float)T::load_c(piece, 4 * it * CROW + e);
                    s = row8_sum(s);
                    if ((ln & 7) == 0) rsto[8 * it + (ln >> 3)] = s;
                }
            }
        }
    };
    if (PROT) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) cp[ni][i] = T::zero();
    }

    static_for<0, MI>([&](auto mi_c) {
        constexpr int mi = decltype(mi_c)::value;
        const int br = wr0 + mi * 32;                                      // first row of this 32-row group
        if (cols_full && br + 32 <= M) {
            // ---- register path: one read of every accumulator serves the sums and the store
            acc_t rowsum = T::zero();
            static_for<0, NI>([&](auto ni_c) {
                constexpr int ni = decltype(ni_c)::value;
                static_for<0, 4>([&](auto q_c) {
                    constexpr int q = decltype(q_c)::value;
                    acc_t v0 = acc_read<AGPR>(acc[mi][ni][4 * q]), v1 = acc_read<AGPR>(acc[mi][ni][4 * q + 1]),
                          v2 = acc_read<AGPR>(acc[mi][ni][4 * q + 2]), v3 = acc_read<AGPR>(acc[mi][ni][4 * q + 3]);
                    if (has_bias) {
                        const i32x4 bb = *reinterpret_cast<const i32x4 *>(bias_lds + wn * TN + ni * 32 + 8 * q + 4 * lh);
                        v0 = add_t(v0, from_word<acc_t>((uint32_t)bb[0])); v1 = add_t(v1, from_word<acc_t>((uint32_t)bb[1]));
                        v2 = add_t(v2, from_word<acc_t>((uint32_t)bb[2])); v3 = add_t(v3, from_word<acc_t>((uint32_t)bb[3]));
                    }
                    if (PROT) {
                        cp[PROT ? ni : 0][4 * q] = add_t(cp[PROT ? ni : 0][4 * q], v0);
                        cp[PROT ? ni : 0][4 * q + 1] = add_t(cp[PROT ? ni : 0][4 * q + 1], v1);
                        cp[PROT ? ni : 0][4 * q + 2] = add_t(cp[PROT ? ni : 0][4 * q + 2], v2);
                        cp[PROT ? ni : 0][4 * q + 3] = add_t(cp[PROT ? ni : 0][4 * q + 3], v3);
                        // (here and now: moved behind the branch, as the compiler would have them, the additions keep every value alive)
                        asm volatile("" : "+v"(cp[PROT ? ni : 0][4 * q]), "+v"(cp[PROT ? ni : 0][4 * q + 1]), "+v"(cp[PROT ? ni : 0][4 * q + 2]),
                                          "+v"(cp[PROT ? ni : 0][4 * q + 3]));
                        rowsum = add_t(rowsum, add_t(add_t(v0, v1), add_t(v2, v3)));
                    }
                    uint8_t *d = wbuf + l32 * CROW + (ni * 32 + 8 * q + 4 * lh) * OS;
                    if constexpr (DT == DT_I8) {
                        *reinterpret_cast<i32x4 *>(d) = i32x4{(int)v0, (int)v1, (int)v2, (int)v3};
                    } else {
                        uint2 w;
                        w.x = pack2<DT>((float)v0, (float)v1);
                        w.y = pack2<DT>((float)v2, (float)v3);
                        *reinterpret_cast<uint2 *>(d) = w;
                    }
                });
                __builtin_amdgcn_sched_barrier(0);      // keeps the accumulator reads from all moving to the top
            });
            if (PROT) {
                const acc_t t = add_xor32(rowsum);     // the half-waves hold different columns
                if (lh == 0) rs_part[wn * BM + wm * TM + mi * 32 + l32] = t;
            }
            wave_sync();
            // read rows back, 16 bytes per lane, and store whole row segments
            constexpr int LPR = TN * OS / 16;                              // lanes per row
            constexpr int RPI = 64 / LPR;                                  // rows per instruction
            constexpr int NIT = 32 / RPI;
            const int r0 = lane / LPR, cch = lane % LPR;
            uint8_t *crow = Cb + ((long)(br + r0) * g.ldc + wc0) * OS + cch * 16;
            const long cstep = (long)RPI * g.ldc * OS;
            i32x4 rowv[NIT];
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                rowv[it] = *reinterpret_cast<const i32x4 *>(wbuf + (it * RPI + r0) * CROW + cch * 16);
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                __builtin_nontemporal_store(rowv[it], reinterpret_cast<i32x4 *>(crow + it * cstep));
            if constexpr (STO) stored_sums(mi, rowv);
            wave_sync();
        } else if (br < M && wc0 < N) {
            // ---- edge path: raw accumulators to LDS, then a plain loop over rows
            static_for<0, NI>([&](auto ni_c) {
                constexpr int ni = decltype(ni_c)::value;
                static_for<0, 4>([&](auto q_c) {
                    constexpr int q = decltype(q_c)::value;
                    uint8_t *d = wbuf + l32 * SROW + (ni * 32 + 8 * q + 4 * lh) * 4;
                    *reinterpret_cast<i32x4 *>(d) =
                        i32x4{(int)as_word(acc_read<AGPR>(acc[mi][ni][4 * q])), (int)as_word(acc_read<AGPR>(acc[mi][ni][4 * q + 1])),
                              (int)as_word(acc_read<AGPR>(acc[mi][ni][4 * q + 2])), (int)as_word(acc_read<AGPR>(acc[mi][ni][4 * q + 3]))};
                });
            });
            wave_sync();
            if (inj_here && g.inj_row >= br && g.inj_row < br + 32 && g.inj_col >= wc0 && g.inj_col < wc0 + TN) {
                // the armed flip: one bit of one accumulator, before rounding and before the sums
                if (lane == 0)
                    *reinterpret_cast<uint32_t *>(wbuf + (g.inj_row - br) * SROW + (g.inj_col - wc0) * 4) ^= (1u << g.inj_bit);
                wave_sync();
            }
            const int nrow = M - br < 32 ? M - br : 32;
            // (1) lane <-> column, walking the rows: store C, column sums
            const int gc = wc0 + lane;
            for (int r = 0; r < nrow && gc < N; ++r) {
                acc_t v = from_word<acc_t>(*reinterpret_cast<const uint32_t *>(wbuf + r * SROW + lane * 4));
                if (has_bias) v = add_t(v, bias_lds[wn * TN + lane]);
                T::store_c(Cb, (long)(br + r) * g.ldc + gc, v);
                if (PROT) colacc = add_t(colacc, v);
                if constexpr (STO) {
                    const float sv = stored_value<DT>((float)v);
                    colacc_s += sv;
                    cmax_s = fmaxf(cmax_s, fabsf(sv));
                }
            }
            // (2) lane <-> row, the half-waves split the columns, walking the columns (each lane
            // starts at a different one: no bank conflicts): row sums without cross-lane traffic.
            // Rows of the group past M get a value too; nobody reads it.
            if (PROT) {
                constexpr int HC = TN / 2;
                const int ncol = N - wc0 < TN ? N - wc0 : TN;
                acc_t rs = T::zero();
                float rs_s = 0.f;
                for (int c = 0; c < HC; ++c) {
                    const int col = lh * HC + ((c + l32) & (HC - 1));
                    if (col < ncol) {
                        acc_t v = from_word<acc_t>(*reinterpret_cast<const uint32_t *>(wbuf + l32 * SROW + col * 4));
                        if (has_bias) v = add_t(v, bias_lds[wn * TN + col]);
                        rs = add_t(rs, v);
                        if constexpr (STO) rs_s += stored_value<DT>((float)v);
                    }
                }
                rs = add_xor32(rs);
                if (lane < 32) rs_part[wn * BM + wm * TM + mi * 32 + lane] = rs;
                if constexpr (STO) {
                    rs_s = add_xor32(rs_s);
                    if (lane < 32) rs_sto[wn * BM + wm * TM + mi * 32 + lane] = rs_s;
                }
            }
            wave_sync();
        } else if (PROT) {
            if (lane < 32) rs_part[wn * BM + wm * TM + mi * 32 + lane] = T::zero();
            if constexpr (STO) {
                if (lane < 32) rs_sto[wn * BM + wm * TM + mi * 32 + lane] = 0.f;
            }
        }
    });

    if (PROT) {
        // ---- column sums of the register-path groups: the lanes' partials folded, values and lanes together, without a trip through LDS
        static_for<0, NI>([&](auto ni_c) {
            constexpr int ni = decltype(ni_c)::value;
            const acc_t t = fold16<acc_t>(cp[PROT ? ni : 0], lane);
            if ((lane & 1) == 0) cs_part[wm * BN + wn * TN + ni * 32 + fold16_column(lane)] = t;
        });
        if (!(cols_full && wr0 + TM <= M)) {
            // groups that were walked row by row: column `lane`
            wave_sync();
            cs_part[tile_thread_index()] = add_t(colacc, cs_part[tile_thread_index()]);
        }
        if constexpr (STO) {
            const int ln = tile_thread_index() & 63, j16 = ln & 15;     // (addresses formed here, not kept across the tile)
            wave_sync();                                             // behind the additions of groups summed element by element
            // register-path groups: column j16 of a chunk; rows 4 (lane >> 4) + r of the product are chunk + 8 parity
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float c = add_xor32((float)dcol[r]);
                if (j16 < 8 && ln < 32) cs_sto[wm * BN + wn * TN + (4 * (ln >> 4) + r) * 8 + j16] += c;
            }
            wave_sync();
            cs_sto[tile_thread_index()] += colacc_s;                  // edge groups
            // the largest stored magnitude: what a consumer of this C needs as its max|A|
            cmax_s = wave_max(cmax_s);
            if (lane == 0) cmax_w[wave] = cmax_s;
        }
        // Barrier over LDS traffic only: the partial sums meet in LDS, and a full barrier would
        // also wait until every store of C issued above has been acknowledged.
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const GemmArgs &g = kernel_args<GemmArgs>();
        const int M = g.M, N = g.N;
        uint32_t amax = 0u;
        if (!T::IS_INT && ep.owned > 0) {
#pragma unroll
            for (int w = 0; w < FAST_WAVES; ++w) amax = amax_w[w] > amax ? amax_w[w] : amax;
        }
        const bool dots_bad = __builtin_amdgcn_readfirstlane(amax) >= DOTS_BAD;
        for (int t = tid; t < BM + BN; t += THREADS) {
            if (t < BM) {
                const int gr = m0 + t;
                if (gr < M) {
                    if constexpr (STO)
                        unsafeAtomicAdd(reinterpret_cast<float *>(g.rc_sto) + (long)bz * M + gr, (rs_sto[t] + rs_sto[BM + t]) + (rs_sto[2 * BM + t] + rs_sto[3 * BM + t]));
                    atomic_add_word(g.rc_obs + (long)bz * M + gr, add_t(add_t(rs_part[t], rs_part[BM + t]), add_t(rs_part[2 * BM + t], rs_part[3 * BM + t])));
                    if (ep.owned > 0 && __builtin_expect(!dots_bad, 1))
                        atomic_add_word(g.rc_pred + (long)bz * M + gr, add_t(add_t(rp_part[t], rp_part[BM + t]), add_t(rp_part[2 * BM + t], rp_part[3 * BM + t])));
                }
            } else {
                const int gc = n0 + (t - BM);
                if constexpr (STO) {
                    if (gc < N) unsafeAtomicAdd(reinterpret_cast<float *>(g.cc_sto) + (long)bz * N + gc, cs_sto[t - BM] + cs_sto[BN + t - BM]);
                }
                if (gc < N)
                    atomic_add_word(g.cc_obs + (long)bz * N + gc, add_t(cs_part[t - BM], cs_part[BN + t - BM]));
            }
        }
        if constexpr (STO) {
            // One atomic per tile: on one word they are served one after the other (bf16 6304 x 3072 x 768, 600 tiles: with the
            // verify behind it 110 us with one per wave, 74 so)
            if (tid == 64) {
                float m = 0.f;
                for (int w = 0; w < FAST_WAVES; ++w) m = fmaxf(m, cmax_w[w]);
                if (m > 0.f) atomicMax(g.c_max + bz, __float_as_uint(m));
            }
        }
        if (__builtin_expect(dots_bad, 0)) {
            // BM / 8 rows to a wave
            constexpr int RW = BM / FAST_WAVES;
            const int ln = tile_thread_index() & 63, t = wave * RW + (ln & (RW - 1));
            float v = (float)rp_part[t] + (float)rp_part[BM + t] + ((float)rp_part[2 * BM + t] + (float)rp_part[3 * BM + t]);
            const bool mine = ln < RW && m0 + t < M;
            const uint32_t which = (uint32_t)__ballot(mine && !(fabsf(v) < __builtin_inff()));
            if constexpr (!T::IS_INT) v = dots_again<DT>(g, ep, bz, m0 + wave * RW, which, v);
            if (mine) atomic_add_word(g.rc_pred + (long)bz * M + m0 + t, v);
        }
        // column sums of A over this tile's rows, for the slabs this workgroup reduced
        for (int t = tid; t < ep.owned * KE && !g.a_given; t += THREADS) {
            const int k = (ep.slab0 + (t / KE) * ep.slab_step) * KE + (t % KE);
            acc_t v = from_word<acc_t>(ep.col_lds[t]);
            if constexpr (!T::IS_INT) {
                // (a wave's 64 columns are one slab's)
                const uint64_t which = __ballot(!(fabsf(v) < __builtin_inff()));
                if (__builtin_expect(which != 0, 0)) v = columns_again<DT>(g, bz, m0, M - m0 < BM ? M - m0 : BM, k - (t % KE), which, v);
            }
            atomic_add_word(g.a_sum + (long)bz * g.K + k, v);
        }
        if (!T::IS_INT && !g.a_given && tid == 0) {
            uint32_t top = 0u;
            if (__builtin_expect(dots_bad, 0)) {
                for (int w = 0; w < FAST_WAVES; ++w) top = (amax_w[w] & ~DOTS_BAD) > top ? amax_w[w] & ~DOTS_BAD : top;
            } else {
                top = amax;
            }
            if (top > 0u) atomicMax(g.a_max + bz, __float_as_uint(DT == DT_BF16 ? bf16_bits_to_f32(top) : f16_bits_to_f32(top)));
        }
    }
}

// With and without a layer bias: two copies of the epilogue behind one uniform branch (a test per
// group of four values inside one copy costs a branch per group).
template <int DT, int BM, bool PROT, int STO>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &g,
                                              typename Traits<DT>::accv_t (&acc)[BM / 64][2],
                                              uint8_t *smem, int m0, int n0, int bz, const EpiProt<DT, BM / 64> &ep)
{
    if (g.bias != nullptr) gemm_epilogue_impl<DT, BM, PROT, STO, true>(g, acc, smem, m0, n0, bz, ep);
    else gemm_epilogue_impl<DT, BM, PROT, STO, false>(g, acc, smem, m0, n0, bz, ep);
}

}  // namespace abft
