// What the two kernels for batches of small problems share (gemm_item_rows.hip, gemm_item_cols.hip).
//
// One workgroup owns a batch item (the per-head attention products Q K^T and attn V), so every checksum
// of the scheme (Sec. III-B.1 "Checksums") is formed and checked inside that workgroup: no atomics on
// global memory but the final ticket, no pass over B, no check kernel.
//
// What bounds these products is memory traffic (about 39 flop per byte at 197 x 197 x 64) and, an
// item being small, the vector instructions per element and the chain of phases of an item.  So
//   * C leaves the accumulators directly: a 32 x 32 block is packed in registers and turned by the
//     row-swap instructions of gfx950 into stores of sixteen row segments of 64 bytes (no LDS stage);
//   * the checksums along K come from the operand fragments the MFMAs use, and mostly by MFMA themselves
//     (Turned, split_b_at); the column sums of C fold values and lanes together, n values over 32 lanes
//     in about 2.5 n instructions instead of 5 n.
// Operands in LDS keep their row orientation with a pitch of an odd number of 16-byte pieces (odd
// number of 32-byte pieces for a 16-bit B stored K x N), so that fragment reads meet no bank
// conflict; a B stored K x N is transposed on the way to the matrix cores (ds_read_b64_tr).
#pragma once
#include "abft_device.h"
#include "gemm_args.h"
#include "gemm_apass.h"
#include "gemm_epilogue.h"
#include "block_out.h"

namespace abft {

constexpr int ITEM_MAX_BLOCKS = 1024;      // workgroups; items beyond are taken in turn
constexpr int ITEM_GROUP = 16;             // workgroups per first-level ticket
constexpr int ITEM_LDS_LIMIT = 160 * 1024;

struct ItemArgs {
    const uint8_t *A, *B;
    uint8_t *C;
    int M, N, K, batch;
    long lda, ldb, ldc, sA, sB, sC;               // elements
    int nch;                                      // 16-byte chunks of a row along K that hold data
    int steps;                                    // MFMA steps over K (32 bytes per row each), rounded up to even
    int NB, MB;                                   // blocks of 32 columns / rows
    int pa, pb;                                   // LDS pitch of a row of A / of B as stored (bytes)
    int b_rows, b_chunks, b_lg;                   // B in LDS: rows, chunks per row, log2 of the threads that share a row
    int a_lg;                                     // the same for A
    int rch, nchunk;                              // blocks of rows of A resident at a time, and how many times
    int lds_a, lds_vec;                           // offsets in LDS
    int inj_b, inj_row, inj_col, inj_bit;         // armed accumulator flip (inj_b < 0: none)
    int cached_b;                                 // take b and max|B| from b_sum / b_max instead of forming them
    // protected launches: everything below is written with plain stores, item by item
    uint32_t *cc_obs, *rc_obs, *rc_pred, *a_sum, *a_max, *b_sum, *b_max, *cc_pred, *s_pred;
    uint32_t *cc_sto, *rc_sto;                    // sums of C as stored (after rounding), on request (floating point)
    float *maxabs, *tau;
    float tau_override, tau_override_cols;
    uint8_t *row_flag, *col_flag;
    uint32_t *counts;
    uint32_t *ticket;                             // [3]: ticket, flagged rows, flagged cols (self-cleaning)
    uint32_t *group_ticket;                       // [ITEM_MAX_BLOCKS / ITEM_GROUP] (self-cleaning)
    uint32_t *c_max;                              // max|C as stored| as float bits, with the stored-side sums
};

// (An item kernel with its arguments taken from the parameter had 200 to 290 scalars in vector registers and 500 of its 3400 instructions to move them.)
__device__ __forceinline__ const ItemArgs &item_args() { return kernel_args<ItemArgs>(); }

// Workgroup barrier over LDS traffic only: a full barrier would also wait until every store of C
// issued so far has been acknowledged.
__device__ __forceinline__ void item_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A lane number the optimiser cannot see through: what is derived from it is computed where it is
// used instead of being held in registers across the loop around it.
__device__ __forceinline__ int item_opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// ------------------------------------------------------------------ operands into LDS
// Rows [0, rows_total) of `chunks` 16-byte chunks each; what lies past `rows` or past rowbytes is zero.
// 1 << lg threads share a row.  A batch is ITEM_U independent loads per thread.
// Buffer loads: what lies outside comes as zeros without a branch, and a load costs one addition.  Offsets stay below 2^31 (item_offsets_fit).
constexpr int ITEM_U = 4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int ITEM_RSRC_FLAGS = 0x00027000;
struct ItemStage {
    __amdgpu_buffer_rsrc_t src;
    int ldbytes, rows_total, rowbytes, chunks, lg, pitch;
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stage_source(const uint8_t *base, int rows, int ldbytes, int rowbytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, rows > 0 ? (rows - 1) * ldbytes + ((rowbytes + 15) & ~15) : 0, ITEM_RSRC_FLAGS);
}
__device__ __forceinline__ void stage_load(const ItemStage &t, int row0, int nt, int tid, i32x4 (&v)[ITEM_U])
{
    const int c = tid & ((1 << t.lg) - 1), r0 = row0 + (tid >> t.lg), rp = nt >> t.lg;
    const unsigned at = c * 16 < t.rowbytes ? (unsigned)(r0 * t.ldbytes + c * 16) : 0x80000000u;
#pragma unroll
    for (int u = 0; u < ITEM_U; ++u) v[u] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(t.src, at + (unsigned)(u * rp * t.ldbytes), 0, 0));
}
__device__ __forceinline__ void stage_store(const ItemStage &t, int row0, int nt, int tid, uint8_t *dst, const i32x4 (&v)[ITEM_U])
{
    const int c = tid & ((1 << t.lg) - 1), r0 = row0 + (tid >> t.lg), rp = nt >> t.lg;
    const bool cut = (t.rowbytes & 15) != 0;                   // a chunk holds what does not belong to the row
    uint8_t *d = dst + r0 * t.pitch + c * 16;
#pragma unroll
    for (int u = 0; u < ITEM_U; ++u) {
        i32x4 x = v[u];
        if (cut) x = mask_chunk(x, t.rowbytes - c * 16);
        if (r0 + u * rp < t.rows_total && c < t.chunks) *reinterpret_cast<i32x4 *>(d + u * rp * t.pitch) = x;
    }
}
__device__ __forceinline__ int stage_batch_rows(const ItemStage &t, int nt) { return (nt >> t.lg) * ITEM_U; }
// the batches from row0 on
__device__ __forceinline__ void stage_rest(const ItemStage &t, int row0, int nt, int tid, uint8_t *dst)
{
    for (; row0 < t.rows_total; row0 += stage_batch_rows(t, nt)) {
        i32x4 v[ITEM_U];
        stage_load(t, row0, nt, tid, v);
        stage_store(t, row0, nt, tid, dst, v);
    }
}
template <int DT, bool TRANSB> __device__ __forceinline__ ItemStage b_stage(const ItemArgs &g, int bz)
{
    constexpr int ES = Traits<DT>::ES;
    ItemStage t;
    t.ldbytes = (int)g.ldb * ES;
    t.rowbytes = (TRANSB ? g.K : g.N) * ES;
    t.src = stage_source(g.B + (long)bz * g.sB * ES, TRANSB ? g.N : g.K, t.ldbytes, t.rowbytes);
    t.rows_total = g.b_rows; t.chunks = g.b_chunks; t.lg = g.b_lg; t.pitch = g.pb;
    return t;
}

// ------------------------------------------------------------------ fragments
// Lane l of a fragment holds row (column of B) l & 31 and the 16-byte chunk 2 s + (l >> 5) along K.
// KNPITCH: the pitch of a B stored K x N where it is known at compile time (0: it is not).
template <int DT, bool TRANSB, int KNPITCH> struct FragB {
    static constexpr int ES = Traits<DT>::ES;
    const uint8_t *base;                         // block 0, step 0
    int pitch_;
    __device__ __forceinline__ FragB(const uint8_t *sB, int pb, int lane) : pitch_(pb)
    {
        if (TRANSB) {
            base = sB + (lane & 31) * pb + (lane >> 5) * 16;
        } else {
            // sixteen lanes read 4 (8) rows of k of sixteen columns as 8-byte pieces; each gets a column
            const int lh = lane >> 5, i16 = lane & 15;
            const int kk = ES == 2 ? 8 * lh + (i16 >> 2) : 16 * lh + (i16 >> 1);
            base = sB + kk * pitch() + 16 * ((lane >> 4) & 1) * ES + (ES == 2 ? (i16 & 3) : (i16 & 1)) * 8;
        }
    }
    __device__ __forceinline__ int pitch() const { return !TRANSB && KNPITCH ? KNPITCH : pitch_; }
    __device__ __forceinline__ int off(int s) const { return TRANSB ? s * 32 : s * (ES == 2 ? 16 : 32) * pitch(); }
    // where step s lies; opaque, so that unrolled code does not keep a pointer per step
    __device__ __forceinline__ int at(int s) const
    {
        int o = off(s);
        asm volatile("" : "+s"(o));
        return o;
    }
    __device__ __forceinline__ i32x4 get(int nb, int at_s) const
    {
        if constexpr (TRANSB) {
            return *reinterpret_cast<const i32x4 *>(base + at_s + nb * 32 * pitch_);
        } else if constexpr (ES == 2) {
            typedef short v4 __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) v4 *p4;
            typedef int i32x2 __attribute__((ext_vector_type(2)));
            const uint8_t *p = base + at_s + nb * 64;
            const i32x2 lo = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((p4)(p)));
            const i32x2 hi = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((p4)(p + 4 * pitch())));
            return i32x4{lo[0], lo[1], hi[0], hi[1]};
        } else {
            typedef int i32x2 __attribute__((ext_vector_type(2)));
            typedef __attribute__((address_space(3))) i32x2 *p2;
            const uint8_t *p = base + at_s + nb * 32;
            const i32x2 lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((p2)(p));
            const i32x2 hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((p2)(p + 8 * pitch()));
            return i32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    }
};

// Largest magnitude of 16-bit values as pairs of 16-bit integers (the order of magnitudes is that of their
// bits); NaN, which a maximum ignores, compares above Inf and is seen at the end (item_max_out).
typedef unsigned short item_u16x2 __attribute__((ext_vector_type(2)));
template <int DT> __device__ __forceinline__ void mag_max(const i32x4 &x, uint32_t *mx)
{
    if constexpr (!Traits<DT>::IS_INT) {
        item_u16x2 m = __builtin_bit_cast(item_u16x2, *mx);
#pragma unroll
        for (int w = 0; w < 4; ++w) m = __builtin_elementwise_max(m, __builtin_bit_cast(item_u16x2, x[w] & 0x7FFF7FFF));
        *mx = __builtin_bit_cast(uint32_t, m);
    }
}
// What a wave saw, to its word in LDS.  With a NaN in it the wave looks through the whole operand again.
template <int DT>
__device__ __forceinline__ void item_max_out(uint32_t mx, const uint8_t *X, long ldbytes, int rows, int cols, int lane, uint32_t *word)
{
    using T = Traits<DT>;
    if constexpr (!T::IS_INT) {
        constexpr uint32_t INF_BITS = DT == DT_BF16 ? 0x7F80u : 0x7C00u;
        const uint32_t m = max(mx & 0xFFFFu, mx >> 16);
        float f = DT == DT_BF16 ? __uint_as_float(m << 16) : f16_bits_to_f32(m);
        if (__any(m > INF_BITS)) {
            f = 0.f;
            for (int r = 0; r < rows; ++r)
                for (int c = lane; c < cols; c += 64) {
                    const uint32_t h = *reinterpret_cast<const uint16_t *>(X + (long)r * ldbytes + c * 2);
                    f = fmaxf(f, fabsf(DT == DT_BF16 ? bf16_bits_to_f32(h) : f16_bits_to_f32(h)));
                }
        }
        f = wave_max(f);
        if (lane == 0) *word = __float_as_uint(f);
    }
}
// A sum along K that is not finite, formed again (see Turned).  stride: bytes from one of its elements to the next.
template <int DT>
__device__ __forceinline__ typename Traits<DT>::acc_t finite_or_again(typename Traits<DT>::acc_t v, const uint8_t *X, long stride, int n)
{
    if constexpr (Traits<DT>::IS_INT) {
        return v;
    } else {
        if (!(fabsf(v) < __builtin_inff())) {
            v = 0.f;
            for (int i = 0; i < n; ++i) {
                const uint32_t h = *reinterpret_cast<const uint16_t *>(X + (long)i * stride);
                v += DT == DT_BF16 ? bf16_bits_to_f32(h) : f16_bits_to_f32(h);
            }
        }
        return v;
    }
}

// ------------------------------------------------------------------ checksums along K
// The sum of an operand over its rows, a = e^T A or b = B e, runs over the lanes of its fragments, where
// an add takes an exchange; the dot of its rows with a vector costs a multiply-add per element.  The
// matrix cores do both with the fragment as it is.  A 16 x 16 MFMA takes lane l of a 32-row fragment for
// row l & 15 and piece l >> 4 along its own K, so rows r and r + 16 meet in one sum.
//   * Times the identity (the same for both pieces of a chunk position): a block of sixteen positions
//     along K in the lanes, row sums r + (r + 16) in four registers.  32 positions take two MFMAs, 8 adds
//     and 2 exchanges (folding lanes in vector instructions: 50).
//   * Times b, split into terms that the operand type holds exactly (int8: signed bytes; bf16: three
//     times eight bits, cut off and not rounded, since a value near the largest must not become Inf):
//     terms for rows 0..15 in columns 0..3, with zeros against the other sixteen rows, and for those in
//     columns 4..7.  Lane l then has in registers 0, 1, 2 the products of row l & 31 over all of K.
//     fp16 has no range for the split: its dot is formed in vector instructions (Dot).
// Products with one are exact, and an accumulator adds in 32 bits as the vector unit does.  But Inf and NaN
// reach through products with zeros what they have no part in: sums and dots that are not
// finite are formed again, element by element (finite_or_again, dot_or_again).
template <int DT> __device__ __forceinline__ typename Traits<DT>::accv_t item_zero()
{
    typename Traits<DT>::accv_t z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = Traits<DT>::zero();
    return z;
}
// 16-bit types: a step of K is the sixteen positions; int8: they are one of the step's two chunks
template <int DT> struct Ident {
    i32x4 f[Traits<DT>::IS_INT ? 2 : 1];
    __device__ __forceinline__ Ident(int lane)
    {
        const int j = lane & 15, lh = lane >> 5;
        if constexpr (Traits<DT>::IS_INT) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) f[u][w] = lh == u && (j >> 2) == w ? 1 << (8 * (j & 3)) : 0;
        } else {
            constexpr int ONE = DT == DT_BF16 ? 0x3F80 : 0x3C00;
            const int pos = j - 8 * lh;
#pragma unroll
            for (int w = 0; w < 4; ++w) f[0][w] = pos == 2 * w ? ONE : pos == 2 * w + 1 ? (int)((unsigned)ONE << 16) : 0;
        }
    }
};
// The sums of 32 positions along K, two blocks of sixteen.
template <int DT> struct Turned {
    typedef typename Acc4<DT>::type acc4;
    typedef typename Traits<DT>::acc_t acc_t;
    acc4 t[2];
    __device__ __forceinline__ Turned() : t{acc4_zero<DT>(), acc4_zero<DT>()} {}
    // 16-bit types: two steps; int8: one step (x0)
    __device__ __forceinline__ void add(const i32x4 &x0, const i32x4 &x1, const Ident<DT> &id)
    {
        if constexpr (Traits<DT>::IS_INT) {
            t[0] = mfma16<DT>(x0, id.f[0], t[0]);
            t[1] = mfma16<DT>(x0, id.f[1], t[1]);
        } else {
            t[0] = mfma16<DT>(x0, id.f[0], t[0]);
            t[1] = mfma16<DT>(x1, id.f[0], t[1]);
        }
    }
    // every lane ends with the total of position (lane & 31)
    __device__ __forceinline__ acc_t sum() const
    {
        const acc_t s0 = add_t(add_t((acc_t)t[0][0], (acc_t)t[0][1]), add_t((acc_t)t[0][2], (acc_t)t[0][3]));
        const acc_t s1 = add_t(add_t((acc_t)t[1][0], (acc_t)t[1][1]), add_t((acc_t)t[1][2], (acc_t)t[1][3]));
        return add_xor32(fold_xor16(s0, s1));
    }
};
// The share of a = e^T A of 32 positions from k0 on, added to the wave's copy.  (Read, add, write: the copy
// is the wave's own, and an LDS atomic would hold its next reads back.  Both halves of the wave hold
// the totals and write them.)  ATOMIC: a copy that several waves add to; integers only, so that their order does not show.
template <int DT, bool ATOMIC = false> __device__ __forceinline__ void a_sums(const Turned<DT> &t, uint32_t *copy, int k0, int lane)
{
    typedef typename Traits<DT>::acc_t acc_t;
    uint32_t *c = copy + k0 + (lane & 31);
    const acc_t v = t.sum();
    if constexpr (ATOMIC) {
        if (lane < 32) lds_add_word(c, v);
    } else {
        const acc_t old = from_word<acc_t>(*c);
        *c = as_word(add_t(old, v));
    }
}

template <int DT> __device__ __forceinline__ constexpr bool split_b() { return DT != DT_F16; }
// terms: [4][KP] elements, the last all zero
template <int DT> __device__ __forceinline__ void split_b_at(uint32_t b, uint8_t *terms, int KP, int k)
{
    (void)b; (void)terms; (void)KP; (void)k;
    if constexpr (DT == DT_I8) {
        int v = (int)b;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int lo = (int)(int8_t)(v & 0xFF);
            terms[d * KP + k] = (uint8_t)(d < 3 ? lo : 0);
            v = (v - lo) >> 8;
        }
    } else if constexpr (DT == DT_BF16) {
        float v = __uint_as_float(b);
        uint16_t *t = reinterpret_cast<uint16_t *>(terms);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t hi = __float_as_uint(v) & 0xFFFF0000u;
            t[d * KP + k] = (uint16_t)(d < 3 ? hi >> 16 : 0u);
            v -= __uint_as_float(hi);
        }
    }
}
// where this lane reads its terms: column c = lane & 15 belongs to the rows of half c >> 2
template <int DT> __device__ __forceinline__ const uint8_t *split_b_lane(const uint8_t *terms, int KP, int lane)
{
    const int c = lane & 15, d = (c >> 2) == ((lane >> 4) & 1) ? c & 3 : 3;
    return terms + d * KP * Traits<DT>::ES + (lane >> 5) * 16;
}
// the dot of row l & 31, in lanes 0..31
template <int DT> __device__ __forceinline__ typename Traits<DT>::acc_t split_b_dot(const typename Acc4<DT>::type &v)
{
    if constexpr (DT == DT_I8) return (int)((uint32_t)v[0] + ((uint32_t)v[1] << 8) + ((uint32_t)v[2] << 16));
    else return ((float)v[2] + (float)v[1]) + (float)v[0];
}
// Short chains of additions: flush() after some eight steps adds what there is to a total.  (In one chain the
// error of A b against 64 bits at K = 577 was 1.4e-7, where it had been 1.0e-7 with eight lanes to a row.)
template <int DT> struct SplitDot {
    typedef typename Traits<DT>::acc_t acc_t;
    typename Acc4<DT>::type v;
    acc_t total;
    __device__ __forceinline__ SplitDot() : v(acc4_zero<DT>()), total(Traits<DT>::zero()) {}
    __device__ __forceinline__ void add(const i32x4 &terms, const i32x4 &x) { v = mfma16<DT>(terms, x, v); }
    __device__ __forceinline__ void flush()
    {
        total = add_t(total, split_b_dot<DT>(v));
        v = acc4_zero<DT>();
    }
    __device__ __forceinline__ acc_t dot() const { return add_t(total, split_b_dot<DT>(v)); }
};
template <int DT>
__device__ __forceinline__ typename Traits<DT>::acc_t dot_or_again(typename Traits<DT>::acc_t v, const uint8_t *row, const uint32_t *b, int K)
{
    if constexpr (split_b<DT>() && !Traits<DT>::IS_INT) {
        if (!(fabsf(v) < __builtin_inff())) {
            v = 0.f;
            for (int k = 0; k < K; ++k)
                v = __builtin_fmaf(bf16_bits_to_f32(reinterpret_cast<const uint16_t *>(row)[k]), __uint_as_float(b[k]), v);
        }
    }
    return v;
}

// A fragment's dot with a vector of K words in LDS (its values at this lane's chunk: from v on), in four
// chains of additions, kept short like those of SplitDot.
template <int DT> struct Dot {
    typedef typename Traits<DT>::acc_t acc_t;
    acc_t d[4], total;
    __device__ __forceinline__ void clear() { d[0] = d[1] = d[2] = d[3] = Traits<DT>::zero(); }
    __device__ __forceinline__ Dot() : total(Traits<DT>::zero()) { clear(); }
    __device__ __forceinline__ acc_t chains() const { return add_t(add_t(d[0], d[1]), add_t(d[2], d[3])); }
    __device__ __forceinline__ void flush()
    {
        total = add_t(total, chains());
        clear();
    }
    __device__ __forceinline__ void add(const i32x4 &x, const uint32_t *v)
    {
        using T = Traits<DT>;
#pragma unroll
        for (int q4 = 0; q4 < 16 / T::ES / 4; ++q4) {
            const i32x4 w = *reinterpret_cast<const i32x4 *>(v + 4 * q4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // int8: the vector's values stay below 2^23 (N <= 640, M <= 1024): 24-bit multiplies are exact
                if constexpr (T::IS_INT) d[e] = __mul24((int)T::elem(x, 4 * q4 + e), w[e]) + d[e];
                else d[e] = __builtin_fmaf(T::elem(x, 4 * q4 + e), __int_as_float(w[e]), d[e]);
            }
        }
    }
    // both halves of the wave
    __device__ __forceinline__ acc_t sum() const { return add_xor32(add_t(total, chains())); }
};

// b = B e and max|B| from the resident B, b also as the terms of A b's operand.  X: B in memory, ks / ns: bytes from one k / one column to the next (finite_or_again).
template <int DT, typename FRAG>
__device__ __forceinline__ void b_pass(const ItemArgs &g, const FRAG &fb, const Ident<DT> &id, uint32_t *b_lds, uint8_t *terms, int KP,
                                       const uint8_t *X, long ks, long ns, int wave, int nw, int lane, uint32_t *bmax)
{
    using T = Traits<DT>;
    // one step of int8, two of a 16-bit type: 32 positions along K
    constexpr int SU = T::IS_INT ? 1 : 2;
    uint32_t mx = 0;
    for (int p = wave; p < g.steps / SU; p += nw) {
        const int at0 = fb.at(SU * p), at1 = fb.at(SU * p + SU - 1);
        Turned<DT> t;
        for (int nb = 0; nb < g.NB; ++nb) {
            const i32x4 x0 = fb.get(nb, at0), x1 = T::IS_INT ? x0 : fb.get(nb, at1);
            t.add(x0, x1, id);
            mag_max<DT>(x0, &mx);
            mag_max<DT>(x1, &mx);
        }
        const int k = p * 32 + (lane & 31);
        typename T::acc_t r = t.sum();
        if (k < g.K) r = finite_or_again<DT>(r, X + (long)k * ks, ns, g.N);
        b_lds[k] = as_word(r);
        split_b_at<DT>(as_word(r), terms, KP, k);
    }
    *bmax = mx;
}
// the same from an encoding formed before
template <int DT>
__device__ __forceinline__ void b_cached(const ItemArgs &g, int bz, uint32_t *b_lds, uint8_t *terms, int KP, int tid, int nt)
{
    for (int k = tid; k < KP; k += nt) {
        const uint32_t v = k < g.K ? g.b_sum[(long)bz * g.K + k] : 0u;
        b_lds[k] = v;
        split_b_at<DT>(v, terms, KP, k);
    }
}

// ------------------------------------------------------------------ C out of the accumulators
// The armed flip: one bit of one accumulator, before rounding and before the sums.
template <int DT, typename ACC>
__device__ __forceinline__ void item_flip(const ItemArgs &g, ACC &acc, int m0, int n0, int lane)
{
    if (m0 + (lane & 31) != g.inj_row) return;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (n0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3) == g.inj_col)
            acc[i] = from_word<typename Traits<DT>::acc_t>(as_word((typename Traits<DT>::acc_t)acc[i]) ^ (1u << g.inj_bit));
}

// Where an item's C goes: buffer stores, which leave out rows past M without a branch (they lie past the end: the descriptor ends
// with the last row), and a lane's place in a block as an offset, so that a store costs an addition.  Offsets stay below 2^31 (item_offsets_fit).
struct ItemOut {
    __amdgpu_buffer_rsrc_t dst;
    int N, ldbytes, lane;
};
template <int DT> __device__ __forceinline__ ItemOut item_out(const ItemArgs &g, int bz, int lane)
{
    constexpr int OS = Traits<DT>::OS;
    ItemOut o;
    o.N = g.N;
    o.ldbytes = (int)g.ldc * OS;
    o.dst = __builtin_amdgcn_make_buffer_rsrc(g.C + (long)bz * g.sC * OS, 0, (g.M - 1) * o.ldbytes + g.N * OS, ITEM_RSRC_FLAGS);
    o.lane = out_row<DT>(lane) * o.ldbytes + out_col<DT>(lane) * OS;
    return o;
}
// A block at (m0, n0), see turn_block.
template <int DT>
__device__ __forceinline__ void store_block(const ItemOut &o, const uint32_t *w, int m0, int n0, int lane)
{
    constexpr int OS = Traits<DT>::OS;
    constexpr int NP = out_passes<DT>(), RPP = 32 / NP;        // passes, rows per pass
    i32x4 out[NP];
    turn_block<DT>(w, out);
    const int at = o.lane + m0 * o.ldbytes + n0 * OS, step = RPP * o.ldbytes;
    if (n0 + 32 <= o.N) {
#pragma unroll
        for (int p = 0; p < NP; ++p) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[p]), o.dst, at + p * step, 0, 0);
    } else {
        // The right edge.  What is left of a lane's 16 bytes there is the same for every lane and leaves
        // in falling powers of two, all passes of a size together: few branches, they cost most here.
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const int left = (o.N * OS) & 15;
        const int col = n0 + out_col<DT>(lane);
        if (col + 16 / OS <= o.N) {
#pragma unroll
            for (int p = 0; p < NP; ++p) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out[p]), o.dst, at + p * step, 0, 0);
        } else if (col < o.N) {
            if (left & 8) {
#pragma unroll
                for (int p = 0; p < NP; ++p) __builtin_amdgcn_raw_buffer_store_b64(u32x2{(unsigned)out[p][0], (unsigned)out[p][1]}, o.dst, at + p * step, 0, 0);
            }
            if (left & 4) {
                const int from = left & 8;
#pragma unroll
                for (int p = 0; p < NP; ++p) __builtin_amdgcn_raw_buffer_store_b32((unsigned)(from ? out[p][2] : out[p][0]), o.dst, at + p * step + from, 0, 0);
            }
            if (left & 2) {
                const int from = left & 12;
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(from & 8 ? (from & 4 ? out[p][3] : out[p][2]) : (from & 4 ? out[p][1] : out[p][0])),
                                                          o.dst, at + p * step + from, 0, 0);
            }
        }
    }
}

// ------------------------------------------------------------------ the end of an item, the end of the launch
// The first n (at most 8) of eight values `stride` words apart, added up; all are requested at once.
template <typename acc_t> __device__ __forceinline__ acc_t sum_copies(const uint32_t *p, int stride, int n)
{
    acc_t v[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const uint32_t x = p[(w < n ? w : 0) * stride];
        v[w] = w < n ? from_word<acc_t>(x) : acc_t(0);
    }
    return add_t(add_t(add_t(v[0], v[1]), add_t(v[2], v[3])), add_t(add_t(v[4], v[5]), add_t(v[6], v[7])));
}
struct ItemTol { float ma, mb, tol; };
// misc: max|A| of eight waves, then max|B|
template <int DT> __device__ __forceinline__ ItemTol item_tolerance(const ItemArgs &g, const uint32_t *misc, int nw, int bz)
{
    ItemTol t = {0.f, 0.f, 0.f};
    if (Traits<DT>::IS_INT) return t;
    float v[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const i32x4 x = reinterpret_cast<const i32x4 *>(misc)[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * q + e] = (4 * q + e) % 8 < nw ? __int_as_float(x[e]) : 0.f;
    }
#pragma unroll
    for (int w = 0; w < 8; ++w) { t.ma = fmaxf(t.ma, v[w]); t.mb = fmaxf(t.mb, v[8 + w]); }
    if (g.cached_b) t.mb = __uint_as_float(g.b_max[bz]);
    t.tol = g.tau_override > 0.f ? g.tau_override : (1e-3f * (float)g.K) * t.ma * t.mb;
    return t;
}
// Row sums against A b, the vectors along K out, a.b.  rcsto null: no stored-side sums.
template <int DT>
__device__ __forceinline__ unsigned item_rows_out(const ItemArgs &g, int bz, int nt, int tid, const uint32_t *rcobs, const uint32_t *rcpred,
                                                  const uint32_t *rcsto, const uint32_t *a_lds, const uint32_t *b_lds, float tol,
                                                  uint32_t *dot_out)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    unsigned nr = 0;
    for (int r0 = 0; r0 < g.M; r0 += nt) {
        const int r = r0 + tid;
        bool fl = false;
        if (r < g.M) {
            const long o = (long)bz * g.M + r;
            const uint32_t obs = rcobs[r], pred = rcpred[r];
            g.rc_obs[o] = obs;
            g.rc_pred[o] = pred;
            if (rcsto) g.rc_sto[o] = rcsto[r];
            fl = mismatch<T::IS_INT>(obs, pred, tol);
            g.row_flag[o] = fl ? 1 : 0;
        }
        nr += __popcll(__ballot(fl));
    }
    acc_t sp = T::zero();
    for (int k = tid; k < g.K; k += nt) {
        const uint32_t aw = a_lds[k], bw = b_lds[k];
        g.a_sum[(long)bz * g.K + k] = aw;
        if (!g.cached_b) g.b_sum[(long)bz * g.K + k] = bw;
        sp = add_t(sp, mul_t(from_word<acc_t>(aw), from_word<acc_t>(bw)));
    }
    sp = wave_sum(sp);
    if ((tid & 63) == 0) *dot_out = as_word(sp);
    return nr;
}
// misc: from word 16 a.b of the waves, with STO from word 40 their max|C as stored|
template <int DT, bool STO>
__device__ __forceinline__ void item_scalars_out(const ItemArgs &g, int bz, const uint32_t *misc, int nw, const ItemTol &t)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    g.s_pred[bz] = as_word(sum_copies<acc_t>(misc + 16, 1, nw));
    if (STO) {
        float m = 0.f;
        for (int w = 0; w < nw; ++w) m = fmaxf(m, __uint_as_float(misc[40 + w]));
        g.c_max[bz] = __float_as_uint(m);
    }
    if (!T::IS_INT) {
        g.maxabs[(long)bz * 2] = t.ma;
        g.maxabs[(long)bz * 2 + 1] = t.mb;
        g.tau[bz] = t.tol;
        g.a_max[bz] = __float_as_uint(t.ma);
        if (!g.cached_b) g.b_max[bz] = __float_as_uint(t.mb);
    }
}
// The ticket of a workgroup, by one thread (in two levels: atomics on one word are served one after the other); the last workgroup writes
// counts and status.  cnt: the waves' flagged rows, then columns (2 nw words of LDS, put there ahead of a barrier).
__device__ __forceinline__ void item_ticket(const ItemArgs &g, const uint32_t *cnt, int nw)
{
    unsigned nr = 0, nc = 0;
    for (int w = 0; w < nw; ++w) { nr += cnt[w]; nc += cnt[nw + w]; }
    if (nr | nc) {
        // rare: the counts must have arrived before this workgroup's ticket does
        unsigned o1 = 0, o2 = 0;
        if (nr) o1 = atomicAdd(g.ticket + 1, nr);
        if (nc) o2 = atomicAdd(g.ticket + 2, nc);
        asm volatile("s_waitcnt vmcnt(0)" :: "v"(o1), "v"(o2) : "memory");
    }
    const unsigned grp = blockIdx.x / ITEM_GROUP, ngrp = (gridDim.x + ITEM_GROUP - 1) / ITEM_GROUP;
    const unsigned gsize = min((unsigned)ITEM_GROUP, gridDim.x - grp * ITEM_GROUP);
    bool last = false;
    if (atomicAdd(g.group_ticket + grp, 1u) == gsize - 1) {
        atomicExch(g.group_ticket + grp, 0u);
        last = atomicAdd(g.ticket, 1u) == ngrp - 1;
    }
    if (last) {
        const uint32_t r = atomicExch(g.ticket + 1, 0u), c = atomicExch(g.ticket + 2, 0u);
        atomicExch(g.ticket, 0u);
        g.counts[0] = r;
        g.counts[1] = c;
        g.counts[2] = status_of(r, c);
        g.counts[3] = 0u;
        g.counts[4] = status_of(r, c);
    }
}

inline int item_log2(int n)                      // rounded up
{
    int lg = 0;
    while ((1 << lg) < n) ++lg;
    return lg;
}

// The two kernels: a wave owns rows (N <= 128) or columns (wider) of its item.  0 bytes: does not fit.
size_t item_rows_lds(int dt, const Shape &s, bool protect, bool sto, ItemArgs *g);
size_t item_cols_lds(int dt, const Shape &s, bool protect, bool sto, ItemArgs *g);
hipError_t launch_item_rows(int dt, bool protect, bool transB, const ItemArgs &g, size_t smem, hipStream_t st);
hipError_t launch_item_cols(int dt, bool protect, bool transB, const ItemArgs &g, size_t smem, hipStream_t st);

}  // namespace abft
