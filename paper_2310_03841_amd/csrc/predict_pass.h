// Both predictions of a protected GEMM, cc_pred = (e^T A) B and rc_pred = A (B e), and the comparison with the
// observed sums, inside the launch of the GEMM itself: for problems of a few tiles, whose calls are chains of latencies.
//
// A matrix-vector product with a vector that sums over everything looks like two launches.  But along K it falls
// apart: a workgroup that holds a range of K of all rows of both operands has a and b of that range complete,
// and its shares of all predictions from the same bytes:
//   a[k] = sum_i A[i,k],   b[k] = sum_j B[j,k],   rc_pred[i] += sum_k A[i,k] b[k],   cc_pred[j] += sum_k a[k] B[j,k].
// It waits for nobody.  Where one operand has many rows they are split over nblk workgroups; each of them sums
// all rows of the other operand again (few, from the L2) and its share of its own operand, and as the products are
// linear in that share too, the shares add up.
//
// The workgroup's pieces of both operands go straight into LDS, all requested at once, and both passes read them
// there: one trip to memory.  What bounds it beyond that is instructions, of which a wave issues one per 8 to 13 clocks here, so
// the sums and the dots of an operand stored along K are MFMAs (16 x 16): a lane holds 16 bytes of k of one row, of
// 64 rows to a wave, as an operand of 16 rows whose depth is 4 rows and the k of a piece.
//   * Times S[j; p, e] = (e == j) that gives the sums over the 4 rows p for each k e of the piece: the sums along the rows
//     build up in the accumulators, one MFMA per 64 rows and piece.
//   * Times V[(q, t); p, e] = (p == q) v_t[e] it gives the products of each row with term t of the vector, split
//     exactly into bf16 terms, signed bytes or (scaled by a power of two) fp16 terms; pieces add up in the accumulator.
// (In vector instructions the two passes took 3.2 and 2.2 us of an int8 197 x 768 x 768, and, a wave to an
// operand, 1.3 and 0.7 so.)  Infinities and NaN
// would reach other rows and columns through the zeros: a workgroup that sees one forms everything element by element.
//
// The comparison: a tile row of C is a unit, and so is a tile column.  Every workgroup waits for its additions to arrive
// and then draws tickets: a tile those of its two units, the workgroups of the predictions one of their own, whose last
// holder tells every unit that they are complete.  A unit is compared by its last tile.  If the predictions are not complete by
// then it looks for them again for a while (POLLS); if they still are not, it leaves the unit to the last of their
// workgroups.  So nobody has to wait, and the order in which workgroups run does not matter.  (One last workgroup for
// everything reads what others have added at 7 KB per us: 7.7 us of a bf16 197 x 3072 x 768.  Tickets on one word are served
// one after the other: 256 workgroups, launch and end 6.6 us, with sixteen words in front 4.5; a second kernel instead
// 7.1.)  The tickets lie in the region that the call accumulates into and are cleared with it.
//
// What orders all this: everything others read here, shares, sums and maxima, moves through atomics of device scope, which are
// performed where all dies see them, and is read by atomic loads there.  A wave waits for its own with s_waitcnt vmcnt(0), which
// on gfx9 counts atomics without a result too and falls when they have been performed; the barrier collects the waves; then the
// ticket is drawn.  It is the sequence of the memory model for a release at device scope, without the write back of the L2 that
// comes first for plain stores: none of those is handed over.  Whoever draws the last ticket so finds what was added
// before the others were drawn, and asks for it behind the wait for the ticket and a barrier.
#pragma once
#include <type_traits>

#include "abft_device.h"

namespace abft {

struct PredArgs {
    int one_launch;                  // 0: none of this, a check kernel follows
    // ---- predictions
    const uint8_t *A, *B;
    long lda, ldb, sA, sB;           // elements
    int M, N, K;
    int nkr, nblk;                   // ranges of 64 bytes of K; blocks of the operand that is split
    int split_b;                     // which: 0 A, 1 B
    int blk_len;                     // rows of a block (B stored K x N and split: chunks of columns)
    int a_steps, b_steps;            // 4 KB of LDS each: 64 rows
    int waves_a;                     // B stored N x K: waves that work on A (the others on B)
    int w_log2;                      // B stored K x N: chunks of columns a step covers
    int a_given, b_given;            // a (a_vec) or b (b_sum) is there already
    const uint32_t *a_vec;
    uint32_t *a_sum, *b_sum;         // accumulated
    uint32_t *a_max, *b_max;
    double *cc_pacc, *rc_pacc;       // shares of the predictions; integers: 32-bit words in the same places
    double *s_pacc;
    // ---- the end of the call
    int wgs;                         // workgroups of a batch item
    int batch;
    int tiles_m, tiles_n, bm, bn;    // units: tile rows, then tile columns
    uint32_t *tickets;               // lines of TICKET_LINE words: [0] units done and what they flagged; [1 ..] of the
                                     // predictions: one for each batch item, of a single problem PRED_GROUPS + 1; then the units'
    const uint32_t *amax_in;         // max|A| (a_max, or the caller's)
    uint32_t *cc_obs, *rc_obs;
    const double *cc_acc, *rc_acc;   // floating point: observed sums as the tiles added them up
    const uint32_t *bias;
    uint32_t *cc_pred, *rc_pred, *s_pred;
    float *maxabs, *tau;
    float tau_override, tau_override_cols;
    uint8_t *row_flag, *col_flag;
    uint32_t *counts;
    uint32_t *zero_ptr, *zero2_ptr;  // what the previous call of this context accumulated into, and the b slot not in
    size_t zero_words, zero2_words;  // use: every workgroup clears a share
};

constexpr int PRED_GROUPS = 16;              // first-level tickets of a single problem
constexpr int PRED_TWO_LEVELS = 160;         // from this many of them on
constexpr int TICKET_LINE = 16;              // words
// a unit's ticket word: its tiles that have ended, and
constexpr uint32_t UNIT_TILES = 0xFFFFu, UNIT_PREDICTED = 0x10000u, UNIT_LEFT = 0x20000u;
constexpr uint32_t UNIT_NO_WAIT = 0x40000u;  // in the word before the call (tests put it there): the last tile does not look again
constexpr int POLLS = 64;                    // about half a microsecond each
__host__ __device__ constexpr int unit_line0(int batch) { return 1 + (batch > PRED_GROUPS + 1 ? batch : PRED_GROUPS + 1); }
constexpr int PRED_STEP_BYTES = 256 * 16;
constexpr int PRED_CHUNKS = 4;               // 16-byte pieces of a row in a range of K
// words: shares of a and b by wave (8 x 64), a, b (2 x 64), their terms (2 x 4 x 64 bytes), scales and maxima
constexpr int PRED_VEC_WORDS = 8 * 64 + 2 * 64 + 2 * 64 + 16;

template <int DT, typename V> __device__ __forceinline__ void add_share(double *base, long at, V v)
{
    if constexpr (Traits<DT>::IS_INT) atomicAdd(reinterpret_cast<int *>(base) + at, v);
    else unsafeAtomicAdd(base + at, (double)v);
}

// Rows of an operand stored along K, in LDS: a step holds 64 rows of four pieces, row r of a group of 16 with piece c in
// slot c ^ (r >> 2), so that 16 lanes that read one piece of 16 rows meet 16 different groups of banks.
__device__ __forceinline__ int pred_at(int row, int c)
{
    return (row >> 6) * PRED_STEP_BYTES + (row & 63) * 64 + ((c ^ ((row >> 2) & 3)) * 16);
}

// One operand of a workgroup, and the waves that work on it.
struct PredRows {
    uint8_t *lds;
    int steps, cnt;                  // steps, rows
    int left;                        // bytes of K from the range's start on
    int w0, nw;                      // wave w0 + i of nw takes steps i, i + nw, ...
};

// What lies past the operand (every row of every step from cnt on, and bytes of K) is cleared in LDS, by the wave that
// requested it: rare, and both passes then read pieces as they are.  The last block of a split operand can end steps
// before the others do (385 rows: 129, 129, 127, in three steps each).
__device__ __forceinline__ void pred_clear(const PredRows &x, int wave, int lane)
{
    const bool ragged = x.left < PRED_CHUNKS * 16;
    if (!ragged && x.steps * 64 == x.cnt) return;
    for (int t = wave - x.w0; t < x.steps; t += x.nw) {
        if (!ragged && (t + 1) * 64 <= x.cnt) continue;
        const int row = t * 64 + lane;
        for (int c = 0; c < PRED_CHUNKS; ++c) {
            i32x4 *at = reinterpret_cast<i32x4 *>(x.lds + pred_at(row, c));
            const int keep = row < x.cnt ? x.left - c * 16 : 0;
            if (keep < 16) *at = mask_chunk(*at, keep);
        }
    }
}

// the pieces of this lane's row of step t (the last one past the end)
__device__ __forceinline__ void pred_read(const PredRows &x, int t, int lane, i32x4 (&v)[PRED_CHUNKS])
{
    t = t < x.steps ? t : x.steps - 1;
#pragma unroll
    for (int c = 0; c < PRED_CHUNKS; ++c) v[c] = *reinterpret_cast<const i32x4 *>(x.lds + pred_at(t * 64 + lane, c));
}

template <int DT> __device__ __forceinline__ uint32_t pred_inf() { return DT == DT_BF16 ? 0x7F80u : 0x7C00u; }
template <int DT> __device__ __forceinline__ float pred_mag(uint32_t m)
{
    return DT == DT_BF16 ? __uint_as_float(m << 16) : f16_bits_to_f32(m);
}

// a + its neighbour in lane ^ 16 (^ 32) in the even quarters (lower half) of the wave, b likewise in the others
template <typename V> __device__ __forceinline__ V pred_fold16(V a, V b)
{
    auto p = __builtin_amdgcn_permlane16_swap(as_word(a), as_word(b), false, false);
    return add_t(from_word<V>(p[0]), from_word<V>(p[1]));
}
template <typename V> __device__ __forceinline__ V pred_fold32(V a, V b)
{
    auto p = __builtin_amdgcn_permlane32_swap(as_word(a), as_word(b), false, false);
    return add_t(from_word<V>(p[0]), from_word<V>(p[1]));
}

// This wave's share of the sums over the rows, into part[0 .. 4 CE); floating point: the largest magnitude's bits.
template <int DT> __device__ __forceinline__ void pred_sums(const PredRows &x, int wave, uint32_t *part, uint32_t *mag)
{
    using T = Traits<DT>;
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    constexpr int CE = 16 / T::ES;
    const int lane = threadIdx.x & 63, j = lane & 15;
    i32x4 sel;                                               // element j of a piece
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (T::IS_INT) sel[w] = (j >> 2) == w ? 1 << (8 * (j & 3)) : 0;
        else {
            constexpr int ONE = DT == DT_BF16 ? 0x3F80 : 0x3C00;
            sel[w] = j == 2 * w ? ONE : j == 2 * w + 1 ? ONE << 16 : 0;
        }
    }
    typename Acc4<DT>::type acc[PRED_CHUNKS];
    u16x2 mx = {0, 0};
#pragma unroll
    for (int c = 0; c < PRED_CHUNKS; ++c) acc[c] = acc4_zero<DT>();
    i32x4 next[PRED_CHUNKS];                                 // pieces of a step are read while the step before is multiplied
    pred_read(x, wave - x.w0, lane, next);
    for (int t = wave - x.w0; t < x.steps; t += x.nw) {
        i32x4 v[PRED_CHUNKS];
#pragma unroll
        for (int c = 0; c < PRED_CHUNKS; ++c) v[c] = next[c];
        pred_read(x, t + x.nw, lane, next);
#pragma unroll
        for (int c = 0; c < PRED_CHUNKS; ++c) {
            acc[c] = mfma16<DT>(v[c], sel, acc[c]);
            if constexpr (!T::IS_INT) {
#pragma unroll
                for (int e = 0; e < 4; ++e) mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, v[c][e] & 0x7FFF7FFF));
            }
        }
    }
    // over the four row groups of the accumulators and the four quarters of the wave; quarter c ends with piece c
    typename T::acc_t s[PRED_CHUNKS];
#pragma unroll
    for (int c = 0; c < PRED_CHUNKS; ++c) s[c] = add_t(add_t(acc[c][0], acc[c][1]), add_t(acc[c][2], acc[c][3]));
    const typename T::acc_t s01 = pred_fold16(s[0], s[1]), s23 = pred_fold16(s[2], s[3]);
    const typename T::acc_t all = pred_fold32(s01, s23);
    if (j < CE) part[(lane >> 4) * CE + j] = as_word(all);
    if constexpr (!T::IS_INT) {
        const uint32_t m = mx[0] > mx[1] ? mx[0] : mx[1];    // of 15 bits: exact as a float
        *mag = (uint32_t)wave_max((float)m);
    }
}

// The same of operands that hold infinities or NaN, by thread k < 4 CE of the workgroup's first wave; the largest
// magnitude (NaN aside, as everywhere) to *mag.
template <int DT> __device__ __forceinline__ void pred_sums_slow(const PredRows &x, uint32_t *part, uint32_t *mag)
{
    using T = Traits<DT>;
    constexpr int CE = 16 / T::ES, KR = PRED_CHUNKS * CE;
    const int k = threadIdx.x;
    if (k >= 64) return;
    float s = 0.f, mx = 0.f;
    if (k < KR && k * T::ES < x.left)
        for (int r = 0; r < x.cnt; ++r) {
            const int w = *reinterpret_cast<const int *>(x.lds + pred_at(r, k / CE) + (k % CE) / 2 * 4);
            const float v = (float)T::elem(i32x4{w, 0, 0, 0}, k % 2);
            s += v;
            mx = fmaxf(mx, fabsf(v));
        }
    mx = wave_max(mx);
    if (k == 0) *mag = __float_as_uint(mx);
    if (k < KR) {
        part[k] = __float_as_uint(s);
        for (int w = 1; w < x.nw; ++w) part[w * 64 + k] = 0u;
    }
}

// Term t of value v as bits of the operand type; what is left of it in v.
template <int DT> __device__ __forceinline__ uint32_t pred_term(typename Traits<DT>::acc_t &v)
{
    if constexpr (DT == DT_I8) {
        const int d = (int)(int8_t)v;
        v = (int)((uint32_t)v - (uint32_t)d) >> 8;
        return (uint32_t)d & 0xFFu;
    } else {
        // A finite value that the type would round to infinity starts with the type's largest; infinities and NaN are one
        // term (what is left of them would be NaN).
        uint32_t h = DT == DT_BF16 ? f32_to_bf16_bits(v) : f32_to_f16_bits(v);
        const bool finite = (__float_as_uint(v) & 0x7F800000u) != 0x7F800000u;
        if (finite && (h & pred_inf<DT>()) == pred_inf<DT>()) h = (h & 0x8000u) | (pred_inf<DT>() - 1u);
        const float left = v - (DT == DT_BF16 ? bf16_bits_to_f32(h) : f16_bits_to_f32(h));
        v = finite ? left : 0.f;
        return h;
    }
}

// Products of the rows with the vector whose terms lie at `terms` ([4][64 bytes]), added to out[row].
template <int DT>
__device__ __forceinline__ void pred_dots(const PredRows &x, int wave, const uint8_t *terms, float scale, double *out)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    const int lane = threadIdx.x & 63, t4 = lane & 3, l16 = lane >> 4;
    i32x4 vec[PRED_CHUNKS];
#pragma unroll
    for (int c = 0; c < PRED_CHUNKS; ++c) {
        vec[c] = i32x4{0, 0, 0, 0};
        if (l16 == ((lane >> 2) & 3)) vec[c] = *reinterpret_cast<const i32x4 *>(terms + t4 * 64 + c * 16);
    }
    i32x4 next[PRED_CHUNKS];
    pred_read(x, wave - x.w0, lane, next);
    for (int t = wave - x.w0; t < x.steps; t += x.nw) {
        i32x4 v[PRED_CHUNKS];
#pragma unroll
        for (int c = 0; c < PRED_CHUNKS; ++c) v[c] = next[c];
        pred_read(x, t + x.nw, lane, next);
        auto acc = acc4_zero<DT>();
#pragma unroll
        for (int c = 0; c < PRED_CHUNKS; ++c) acc = mfma16<DT>(v[c], vec[c], acc);
        // register m of lane l: row 16 ((l >> 2) & 3) + 4 (l >> 4) + m, term l & 3.  The lane takes row m = l & 3; the
        // terms' products are added in doubles, so that splitting the vector costs no rounding.
        typename std::conditional<T::IS_INT, int, double>::type d;
        if constexpr (T::IS_INT) {
            d = 0;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                int v = (int)((uint32_t)acc[m] << (8 * t4));
                v = add_t(v, dpp_get<0xB1>(v));              // lane ^ 1
                v = add_t(v, dpp_get<0x4E>(v));              // lane ^ 2
                d = t4 == m ? v : d;
            }
        } else {
            auto term = [&](auto ctrl) __attribute__((always_inline)) {       // of row l & 3, from the lane of that term
                constexpr int C = decltype(ctrl)::value;
                float v = dpp_get<C>(acc[0]);
#pragma unroll
                for (int m = 1; m < 4; ++m) {
                    const float w = dpp_get<C>(acc[m]);
                    v = t4 == m ? w : v;
                }
                return (double)v;
            };
            d = term(std::integral_constant<int, 0x00>{}) + term(std::integral_constant<int, 0x55>{}) +
                term(std::integral_constant<int, 0xAA>{});
            if constexpr (DT == DT_F16) d *= (double)scale;
        }
        const int row = t * 64 + 16 * ((lane >> 2) & 3) + 4 * l16 + t4;
        if (row < x.cnt) add_share<DT>(out, row, d);
    }
}
template <int DT> __device__ __forceinline__ void pred_dots_slow(const PredRows &x, int wave, const uint32_t *vec, double *out)
{
    using T = Traits<DT>;
    constexpr int CE = 16 / T::ES;
    for (int r = (wave - x.w0) * 64 + (threadIdx.x & 63); r < x.cnt; r += x.nw * 64) {
        typename T::acc_t d = T::zero();
        for (int c = 0; c < PRED_CHUNKS; ++c) {
            const i32x4 v = *reinterpret_cast<const i32x4 *>(x.lds + pred_at(r, c));
#pragma unroll
            for (int q = 0; q < CE; ++q) d = add_t(d, mul_t(T::elem(v, q), from_word<typename T::acc_t>(vec[c * CE + q])));
        }
        add_share<DT>(out, r, d);
    }
}

// Workgroup e of nkr * nblk of batch item bz; with a bias one more, which adds what it contributes: M bias[n] to the
// column predictions, its sum to the rows'.  smem: (a_steps + b_steps) steps, at least 256 * (16 / element size) words;
// PRED_VEC_WORDS behind them, at vec_off.
template <int DT, bool TRANSB>
__device__ __forceinline__ void predict_block(const PredArgs &p, int e, int bz, uint8_t *smem, int vec_off)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    typedef const __attribute__((address_space(1))) void *gas;
    typedef __attribute__((address_space(3))) void *las;
    constexpr int ES = T::ES, CE = 16 / ES, KR = PRED_CHUNKS * CE;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = p.M, N = p.N, K = p.K;
    double *rc = p.rc_pacc, *cc = p.cc_pacc;
    // (integers keep 32-bit words in these places)
    auto item = [&](double *base, long at) { return T::IS_INT ? reinterpret_cast<double *>(reinterpret_cast<int *>(base) + at) : base + at; };
    rc = item(rc, (long)bz * M);
    cc = item(cc, (long)bz * N);
    if (e == p.nkr * p.nblk) {
        constexpr int U = 8;
        acc_t sum = T::zero();
        for (int n0 = tid; n0 < N; n0 += 256 * U) {
            acc_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = n0 + 256 * u < N ? from_word<acc_t>(p.bias[n0 + 256 * u]) : T::zero();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                sum = add_t(sum, v[u]);
                if (n0 + 256 * u < N) add_share<DT>(cc, n0 + 256 * u, mul_t((acc_t)M, v[u]));
            }
        }
        sum = wave_sum(sum);
        acc_t *red = reinterpret_cast<acc_t *>(smem);
        if (lane == 0) red[wave] = sum;
        __syncthreads();
        sum = add_t(add_t(red[0], red[1]), add_t(red[2], red[3]));
        for (int r = tid; r < M; r += 256) add_share<DT>(rc, r, sum);
        if (tid == 0) add_share<DT>(p.s_pacc, bz, mul_t((acc_t)M, sum));
        return;
    }
    const int kr = e % p.nkr, blk = e / p.nkr;
    const int k0 = kr * KR, nch = (K + CE - 1) / CE;
    const bool split_a = !p.split_b;
    const uint8_t *Ab = p.A + (long)bz * p.sA * ES, *Bb = p.B + (long)bz * p.sB * ES;
    const int a_beg = split_a ? blk * p.blk_len : 0;
    const int a_cnt = split_a ? min(p.blk_len, M - a_beg) : M;
    // of B: rows (N x K), or pieces of columns (K x N)
    const int b_all = TRANSB ? N : (N + CE - 1) / CE;
    const int b_beg = split_a ? 0 : blk * p.blk_len;
    const int b_cnt = split_a ? b_all : min(p.blk_len, b_all - b_beg);
    const int W = 1 << p.w_log2, RB = 256 >> p.w_log2;                          // K x N: pieces and rows of k of a step
    const int bc = tid & (W - 1), bk = tid >> p.w_log2;
    uint8_t *b_smem = smem + p.a_steps * PRED_STEP_BYTES;
    const uint8_t *b_mine = b_smem + tid * 16;                                  // K x N: this thread's piece of step 0
    uint32_t *vec = reinterpret_cast<uint32_t *>(smem + vec_off);
    uint32_t *part_a = vec, *part_b = vec + 4 * 64, *a_lds = vec + 8 * 64, *b_lds = vec + 9 * 64, *misc = vec + 12 * 64;
    uint8_t *a_terms = reinterpret_cast<uint8_t *>(vec + 10 * 64), *b_terms = a_terms + 256;
    // a wave works on one operand: the passes are chains of latencies, whose length a second operand would double
    const int wa = TRANSB ? p.waves_a : 4;
    const PredRows a = {smem, p.a_steps, a_cnt, (K - k0) * ES, 0, wa}, b = {b_smem, p.b_steps, b_cnt, (K - k0) * ES, wa, 4 - wa};
    const bool on_b = TRANSB && wave >= wa;
    const PredRows x = on_b ? b : a;

    // a given vector's word, wanted behind the sums
    uint32_t given = 0u;
    if (tid < 2 * KR && k0 + (tid & (KR - 1)) < K) {
        if (tid < KR ? p.a_given : p.b_given) given = (tid < KR ? p.a_vec : p.b_sum)[(long)bz * K + k0 + (tid & (KR - 1))];
    }
    // a load instruction: 16 rows of four pieces
    {
        const uint8_t *X = on_b ? Bb : Ab;
        const long ld = on_b ? p.ldb : p.lda;
        const int beg = on_b ? b_beg : a_beg, r16 = lane >> 2;
        int ch = kr * PRED_CHUNKS + ((lane & 3) ^ (r16 >> 2));
        ch = ch < nch ? ch : nch - 1;
        for (int t = wave - x.w0; t < x.steps; t += x.nw)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r = beg + min(t * 64 + g * 16 + r16, x.cnt - 1);
                __builtin_amdgcn_global_load_lds((gas)(X + ((long)r * ld + ch * CE) * ES), (las)(x.lds + (t * 4 + g) * 1024), 16, 0, 0);
            }
    }
    if constexpr (!TRANSB) {
        for (int t = 0; t < p.b_steps; ++t) {
            const int k = min(k0 + min(t * RB + bk, KR - 1), K - 1);
            __builtin_amdgcn_global_load_lds((gas)(Bb + ((long)k * p.ldb + (b_beg + min(bc, b_cnt - 1)) * CE) * ES),
                                             (las)(b_smem + (t * 4 + wave) * 1024), 16, 0, 0);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // every wave reads back what it requested itself

    pred_clear(x, wave, lane);

    // ---- a and b of the range
    uint32_t mag = 0, magb = 0;
    pred_sums<DT>(x, wave, on_b ? part_b + (wave - wa) * 64 : part_a + wave * 64, &mag);
    int b_parts = 4 - wa;
    // K x N: columns past N and rows of k past K cleared
    auto kn_piece = [&](int t) __attribute__((always_inline)) {
        const int cols = bc < b_cnt ? N - (b_beg + bc) * CE : 0;
        const bool in = t * RB + bk < KR && k0 + t * RB + bk < K;
        return mask_chunk(*reinterpret_cast<const i32x4 *>(b_mine + t * PRED_STEP_BYTES), in && cols > 0 ? cols * ES : 0);
    };
    if constexpr (!TRANSB) {
        b_parts = W > 64 ? W >> 6 : 1;
        float mx = 0.f;
        for (int t = 0; t < p.b_steps; ++t) {
            const i32x4 v = kn_piece(t);
            acc_t s = T::zero();
#pragma unroll
            for (int q = 0; q < CE; ++q) {
                const acc_t x = T::elem(v, q);
                s = add_t(s, x);
                if (!T::IS_INT) mx = fmaxf(mx, fabsf((float)x));
            }
            s = seg_sum(s, W < 64 ? W : 64);
            if ((bc & 63) == 0 && t * RB + bk < KR) part_b[(bc >> 6) * 64 + t * RB + bk] = as_word(s);
        }
        if (!T::IS_INT) magb = __float_as_uint(wave_max(mx));
    }
    if (!T::IS_INT && lane == 0) {
        misc[wave] = on_b ? 0u : mag;
        misc[4 + wave] = on_b ? mag : magb;
    }
    __syncthreads();
    bool slow_a = false, slow_b = false;
    uint32_t maga = 0;
    if constexpr (!T::IS_INT) {
        maga = max(max(misc[0], misc[1]), max(misc[2], misc[3]));
        magb = max(max(misc[4], misc[5]), max(misc[6], misc[7]));
        slow_a = maga >= pred_inf<DT>();
        slow_b = TRANSB && magb >= pred_inf<DT>();
        maga = __float_as_uint(pred_mag<DT>(maga));
        if (TRANSB) magb = __float_as_uint(pred_mag<DT>(magb));
        if (slow_a || slow_b) {
            if (slow_a) pred_sums_slow<DT>(a, part_a, misc + 10);
            if (slow_b) pred_sums_slow<DT>(b, part_b, misc + 11);
            __syncthreads();
            if (slow_a) maga = misc[10];
            if (slow_b) magb = misc[11];
        }
    }
    const bool first = blk == 0;
    const bool a_share = split_a && !p.a_given, b_share = !split_a && !p.b_given;        // a share only, not the whole
    if (tid < 2 * KR) {
        const bool is_b = tid >= KR;
        const int i = is_b ? tid - KR : tid, k = k0 + i;
        acc_t v = T::zero();
        if (is_b ? p.b_given : p.a_given) {
            v = from_word<acc_t>(given);
        } else {
            const uint32_t *part = is_b ? part_b : part_a;
            const int n = is_b ? b_parts : wa;
            uint32_t w4[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) w4[w] = part[(w < n ? w : 0) * 64 + i];
#pragma unroll
            for (int w = 0; w < 4; ++w) v = w < n ? add_t(v, from_word<acc_t>(w4[w])) : v;
            if (k < K && (first || (is_b ? b_share : a_share))) atomic_add_word((is_b ? p.b_sum : p.a_sum) + (long)bz * K + k, v);
            if (k >= K) v = T::zero();
        }
        (is_b ? b_lds : a_lds)[i] = as_word(v);
        // the same in terms of the operand type (fp16: of the vector scaled so that its largest value is near 2^14)
        if constexpr (DT == DT_F16) {
            float m = fabsf((float)v);
            m = fmaxf(m, dpp_get<0xB1>(m));
            m = fmaxf(m, dpp_get<0x4E>(m));
            m = fmaxf(m, dpp_get<0x141>(m));
            m = fmaxf(m, dpp_get<0x140>(m));
            m = max_xor16(m);                                // over the 32 lanes of a vector
            int ex = (int)(__float_as_uint(m) >> 23) - 127;
            ex = ex < -100 ? -100 : ex;                      // at most 128 (infinity): both scales are normal numbers
            if (i == 0) misc[8 + (is_b ? 1 : 0)] = (uint32_t)(127 + ex - 14) << 23;
            v *= __uint_as_float((uint32_t)(127 - ex + 14) << 23);
        }
        uint8_t *terms = (is_b ? b_terms : a_terms) + i * ES;
        for (int t = 0; t < 4; ++t) {
            const uint32_t h = DT != DT_I8 && t == 3 ? 0u : pred_term<DT>(v);
            if constexpr (T::IS_INT) terms[t * 64] = (uint8_t)h;
            else *reinterpret_cast<uint16_t *>(terms + t * 64) = (uint16_t)h;
        }
    }
    if constexpr (!T::IS_INT) {
        if (tid == 128 && !p.a_given && (first || a_share) && maga != 0)
            atomicMax(p.a_max + bz, maga);
        if (tid == 192 && !p.b_given && (first || b_share) && magb != 0)
            atomicMax(p.b_max + bz, magb);
    }
    __syncthreads();

    // ---- shares of the predictions
    if (wave == 3 && (first || a_share || b_share)) {
        acc_t v = T::zero();
        if (lane < KR) v = mul_t(from_word<acc_t>(a_lds[lane]), from_word<acc_t>(b_lds[lane]));
        v = wave_sum(v);
        if (lane == 0) add_share<DT>(p.s_pacc, bz, v);
    }
    // a product belongs to this workgroup if its rows do (split), or its vector is a share, or it is the first
    if (on_b ? !split_a || first || a_share : split_a || first || b_share) {
        double *out = on_b ? item(cc, b_beg) : item(rc, a_beg);
        if (on_b ? slow_b : slow_a) pred_dots_slow<DT>(x, wave, on_b ? a_lds : b_lds, out);
        else pred_dots<DT>(x, wave, on_b ? a_terms : b_terms, __uint_as_float(misc[on_b ? 8 : 9]), out);
    }
    if constexpr (!TRANSB) {
        if (!split_a || first || a_share) {
            acc_t c[CE];
#pragma unroll
            for (int q = 0; q < CE; ++q) c[q] = T::zero();
            for (int t = 0; t < p.b_steps; ++t) {
                const i32x4 v = kn_piece(t);
                const int kk = t * RB + bk;
                if (kk < KR && k0 + kk < K) {
                    const acc_t a = from_word<acc_t>(a_lds[kk]);
#pragma unroll
                    for (int q = 0; q < CE; ++q) c[q] = add_t(c[q], mul_t(T::elem(v, q), a));
                }
            }
            // rows of k of a wave first, where it holds several
#pragma unroll
            for (int q = 0; q < CE; ++q) {
                if (W <= 8) c[q] = add_t(c[q], dpp_get<0x128>(c[q]));           // row_ror:8
                if (W <= 16) c[q] = add_xor16(c[q]);
                if (W <= 32) c[q] = add_xor32(c[q]);
            }
            __syncthreads();                                                    // nobody reads the pieces any more
            acc_t *red = reinterpret_cast<acc_t *>(smem);
            const int RY = W <= 64 ? 4 : RB, y0 = W <= 64 ? wave : bk;
            if (W >= 64 || lane < W) {
#pragma unroll
                for (int q = 0; q < CE; ++q) red[(y0 * W + bc) * CE + q] = c[q];
            }
            __syncthreads();
            for (int i = tid; i < b_cnt * CE; i += 256) {
                const int col = b_beg * CE + i;
                if (col < N) {
                    acc_t s = red[i];
                    for (int y = 1; y < RY; ++y) s = add_t(s, red[y * W * CE + i]);
                    add_share<DT>(cc, col, s);
                }
            }
        }
    }
}

// Words other workgroups have added to: read where those additions were made.
__device__ __forceinline__ uint32_t shared_word(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int DT> __device__ __forceinline__ uint32_t shared_sum(const double *base, long at)
{
    if constexpr (Traits<DT>::IS_INT) return shared_word(reinterpret_cast<const uint32_t *>(base) + at);
    else return __float_as_uint((float)__hip_atomic_load(base + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

__device__ __forceinline__ uint32_t draw_ticket(uint32_t *t, uint32_t n = 1)
{
    return __hip_atomic_fetch_add(t, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Compares entry i of a side of batch item bz; returns whether it is flagged.
template <int DT> __device__ __forceinline__ bool compare_entry(const PredArgs &p, int bz, bool row, int i, float tol)
{
    using T = Traits<DT>;
    const long o = (long)bz * (row ? p.M : p.N) + i;
    uint32_t obs;
    if constexpr (T::IS_INT) obs = shared_word((row ? p.rc_obs : p.cc_obs) + o);
    else obs = shared_sum<DT>(row ? p.rc_acc : p.cc_acc, o);
    const uint32_t pred = shared_sum<DT>(row ? p.rc_pacc : p.cc_pacc, o);
    const bool fl = mismatch<T::IS_INT>(obs, pred, tol);
    (row ? p.rc_pred : p.cc_pred)[o] = pred;
    if (!T::IS_INT) (row ? p.rc_obs : p.cc_obs)[o] = obs;
    (row ? p.row_flag : p.col_flag)[o] = fl ? 1 : 0;
    return fl;
}

struct UnitTol { float rows, cols; };
template <int DT> __device__ __forceinline__ UnitTol unit_tolerance(const PredArgs &p, int bz, bool keep)
{
    UnitTol t = {0.f, 0.f};
    if constexpr (!Traits<DT>::IS_INT) {
        const float ma = __uint_as_float(shared_word(p.amax_in + bz)), mb = __uint_as_float(shared_word(p.b_max + bz));
        t.rows = p.tau_override > 0.f ? p.tau_override : (1e-3f * (float)p.K) * ma * mb;
        t.cols = p.tau_override_cols > 0.f ? p.tau_override_cols : t.rows;
        if (keep) {
            p.maxabs[(long)bz * 2] = ma;
            p.maxabs[(long)bz * 2 + 1] = mb;
            p.tau[bz] = t.rows;
        }
    }
    return t;
}

// n units compared by this workgroup, nr rows and nc columns of this thread's flagged.  One 64-bit word adds up units done
// and what they flagged; who completes it writes the counts.
__device__ __forceinline__ void units_done(const PredArgs &p, unsigned n, unsigned nr, unsigned nc, uint32_t *smem)
{
    const int tid = threadIdx.x;
    nr = (unsigned)wave_sum((int)(nr | nc << 16));           // ONE_LAUNCH_MAX_LEN < 2^16
    if ((tid & 63) == 0) smem[4 + (tid >> 6)] = nr;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (tid == 0) {
        const unsigned f = smem[4] + smem[5] + smem[6] + smem[7];
        const unsigned long long mine = (unsigned long long)n << 32 | f;
        const unsigned long long all = mine + __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(p.tickets), mine,
                                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((unsigned)(all >> 32) == (unsigned)(p.tiles_m + p.tiles_n) * p.batch) {
            nr = (unsigned)all & 0xFFFFu;
            nc = (unsigned)all >> 16 & 0xFFFFu;
            p.counts[0] = nr;
            p.counts[1] = nc;
            p.counts[2] = status_of(nr, nc);
            p.counts[3] = 0u;
            p.counts[4] = status_of(nr, nc);
        }
    }
}

// The end of tile (tm, tn) of batch item bz.  smem: 8 words.
template <int DT, int BM, int BN>
__device__ __forceinline__ void end_tile(const PredArgs &p, int tm, int tn, int bz, uint32_t *smem)
{
    static_assert(BM + BN <= 256, "a thread for every entry of two units");
    const int tid = threadIdx.x;
    // this workgroup's additions have been made before its tickets are drawn
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (tid < 2) {
        const int unit = tid == 0 ? tm : p.tiles_m + tn;
        uint32_t *t = p.tickets + (unit_line0(p.batch) + (long)bz * (p.tiles_m + p.tiles_n) + unit) * TICKET_LINE;
        uint32_t mine = 0u, w = draw_ticket(t);
        if ((w & UNIT_TILES) == (unsigned)(tid == 0 ? p.tiles_n : p.tiles_m) - 1) {      // the last tile
            for (int i = 0; i < POLLS && !(w & (UNIT_PREDICTED | UNIT_NO_WAIT)); ++i) w = shared_word(t);
            if (!(w & UNIT_PREDICTED)) w = draw_ticket(t, UNIT_LEFT);
            mine = w & UNIT_PREDICTED ? 1u : 0u;
        }
        smem[tid] = mine;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const unsigned rows = smem[0], cols = smem[1];
    if (!(rows | cols)) return;
    const UnitTol tol = unit_tolerance<DT>(p, bz, false);
    bool fr = false, fc = false;
    if (tid < BM) {
        if (rows && tm * BM + tid < p.M) fr = compare_entry<DT>(p, bz, true, tm * BM + tid, tol.rows);
    } else if (tid < BM + BN) {
        if (cols && tn * BN + tid - BM < p.N) fc = compare_entry<DT>(p, bz, false, tn * BN + tid - BM, tol.cols);
    }
    units_done(p, rows + cols, fr, fc, smem);
}

// The end of workgroup e of the n of batch item bz that form its predictions.  smem: 8 + units words.
template <int DT> __device__ __forceinline__ void end_predict(const PredArgs &p, int e, int n, int bz, uint32_t *smem)
{
    const int tid = threadIdx.x, units = p.tiles_m + p.tiles_n;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (tid == 0) {
        bool last;
        if (p.batch == 1 && n >= PRED_TWO_LEVELS) {
            const int grp = e & (PRED_GROUPS - 1), in_grp = (n - grp + PRED_GROUPS - 1) / PRED_GROUPS;
            last = draw_ticket(p.tickets + (2 + grp) * TICKET_LINE) == (unsigned)in_grp - 1;
            if (last) last = draw_ticket(p.tickets + TICKET_LINE) == (unsigned)PRED_GROUPS - 1;
        } else {
            last = draw_ticket(p.tickets + (1 + bz) * TICKET_LINE) == (unsigned)n - 1;
        }
        smem[0] = last ? 1u : 0u;
        smem[1] = 0u;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (smem[0] == 0u) return;
    // the predictions are complete: units whose tiles have given up on them are compared here
    for (int u = tid; u < units; u += 256) {
        uint32_t *t = p.tickets + (unit_line0(p.batch) + (long)bz * units + u) * TICKET_LINE;
        if (draw_ticket(t, UNIT_PREDICTED) & UNIT_LEFT) smem[8 + atomicAdd(smem + 1, 1u)] = (uint32_t)u;
    }
    if (tid == 0) p.s_pred[bz] = shared_sum<DT>(p.s_pacc, bz);
    const UnitTol tol = unit_tolerance<DT>(p, bz, tid == 0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const unsigned mine = smem[1];
    if (mine == 0u) return;
    unsigned nr = 0, nc = 0;
    // 256 / 64 or / 128 units at a time: a thread's entry of its unit
    const int per = p.bn > 64 ? 128 : 64;
    for (unsigned j = tid / per; j < mine; j += 256 / per) {
        const int u = (int)smem[8 + j], q = tid & (per - 1);
        const bool row = u < p.tiles_m;
        const int i = row ? u * p.bm + q : (u - p.tiles_m) * p.bn + q;
        if (q < (row ? p.bm : p.bn) && i < (row ? p.M : p.N)) {
            const bool fl = compare_entry<DT>(p, bz, row, i, row ? tol.rows : tol.cols);
            nr += fl && row;
            nc += fl && !row;
        }
    }
    units_done(p, mine, nr, nc, smem);
}

}  // namespace abft
