// Batches of small problems, N > 128 (Q K^T): a wave owns columns of its item.  See gemm_item.h for
// what is common.
//
// B of the item and its rows of A lie in LDS (as many rows of A at a time as leave room for a second
// workgroup on the compute unit; the next ones are on their way in registers meanwhile).  Wave w of
// eight takes the blocks of 32 columns w, w + 8, ... over all rows: the column sums of C stay in
// registers for the whole item, a row's sum is one word per wave.  The pass over A is dealt out over the
// waves by blocks of rows.
//
// Measured (384 items 197 x 197 x 64 bf16, Q K^T of 32 images; floor 9.8 us): 32.0 us with four waves per item, C
// through an LDS stage and the sums along K in vector instructions, 21.2 so, 18.5 since the phases read their own arguments (item_args), 12.9
// unprotected (before: 18.0).  An item takes what its waves' instructions take (a SIMD issues one in 0.44 of the cycles): reading the main loop's fragments a piece ahead, or
// dealing the pass over B to all waves, which each cost some more of them, gained nothing (21.4, and 2 to 4 % slower elsewhere).
// int8 1024 x 577 x 577 x 64 (1.44 GB, floor 285 us): 432 us, so 378 (on another
// card 412 and 349); bound by the stores of C, whose rows
// are 16-byte aligned only.
#include "gemm_item.h"

namespace abft {

constexpr int COLS_NW = 8, COLS_NT = 64 * COLS_NW;

// The last block of columns hangs over the edge of C and takes twice as long to store as another: where a wave has no block, it
// takes the second half of that block's rows.  (197 columns, seven blocks: the other waves waited 5900 of an item's 30000
// clocks for the seventh, 2700 so.  bf16 197 x 197 x 64, 128 items 17.0 -> 15.6 us, 384 items 21.6 -> 21.3, unprotected 13.2 -> 12.6.)
static __host__ __device__ bool shares_last_block(int NB, int N) { return NB < COLS_NW && NB * 32 > N; }
// The kernel that can share it.  The other one has 50 to 110 instructions and up to 16 bytes of spilled registers less, and takes the
// items without such a block: 197 x 224 x 64, 384 items, fp16 21.6 -> 21.1 us, with stored sums (192 columns) 33.2 -> 31.1, int8 22.4 -> 22.1.
// Not in bf16 with B stored K x N, nor with stored sums and B stored N x K: there the compiler spills more scalar registers in it (256 items 197 x
// 224 x 64: 18.3 us against 17.4 by this one; 384 items 197 x 160 x 64 with stored sums 32.9 against 31.6).
static bool takes_sharing_kernel(int dt, bool transB, bool protect, bool sto, int NB, int N)
{
    return NB <= COLS_NW && (shares_last_block(NB, N) || (dt == DT_BF16 && protect && sto == transB));
}

// Offsets (words) of the vectors behind B and A.
struct ColsLds {
    int KP, Mr, Nr, RC, a, b, apart, terms, rcobs, rcpred, rspart, ccobs, misc, rcsto, rsspart, ccsto, total;
    __host__ __device__ ColsLds(const ItemArgs &g, int es, bool sto, bool shared)
    {
        KP = g.steps * (es == 2 ? 16 : 32);
        Mr = g.MB * 32; Nr = (g.NB + (shared && g.NB < COLS_NW ? 1 : 0)) * 32; RC = g.rch * 32;      // (the sums of a shared block's second half behind the others)
        int o = 0;
        a = o; o += KP;
        b = o; o += KP;
        apart = o; o += COLS_NW * KP;
        terms = o; o += KP * es;                 // [4][KP] elements
        rcobs = o; o += Mr;
        rcpred = o; o += Mr;
        rspart = o; o += COLS_NW * RC;
        ccobs = o; o += Nr;
        misc = o; o += 48;                       // 0..7 max|A|, 8..15 max|B|, 16..23 a.b per wave; 24..39 flag counts; 40..47 max|C as stored|
        rcsto = o; o += sto ? Mr : 0;
        rsspart = o; o += sto ? COLS_NW * RC : 0;
        ccsto = o; o += sto ? Nr : 0;
        total = o;
    }
};

// SHARED: the last block of columns may be two waves' (TPW = 1).
template <int DT, int TPW, bool PROT, bool TRANSB, bool STO, bool SHARED>
__global__ __launch_bounds__(COLS_NT, TPW == 1 && !STO ? 4 : 2) void item_cols_kernel(ItemArgs)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    typedef typename T::accv_t accv_t;
    typedef FragB<DT, TRANSB, 0> Frag;
    fetch_args<ItemArgs>();
    constexpr int ES = T::ES;
    constexpr int R = TPW == 1 ? 2 : 1;         // blocks of rows at a time
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned nr_w = 0, nc_w = 0;

    for (int bz = blockIdx.x;; bz += gridDim.x) {
        const int tid = item_opaque(threadIdx.x), lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
        // rows of A, from row row0 of the item on
        auto a_stage = [&](const ItemArgs &g, const ColsLds &L, int row0) __attribute__((always_inline)) {
            ItemStage as;
            as.ldbytes = (int)g.lda * ES; as.rowbytes = g.K * ES;
            as.src = stage_source(g.A + ((long)bz * g.sA + (long)row0 * g.lda) * ES, g.M - row0, as.ldbytes, as.rowbytes);
            as.rows_total = L.RC; as.chunks = 2 * g.steps; as.lg = g.a_lg; as.pitch = g.pa;
            return as;
        };
        i32x4 va[ITEM_U];                        // rows of A on their way: one batch holds a chunk (see item_cols_lds)
        {
            const ItemArgs &g = item_args();
            const ColsLds L(g, ES, STO, SHARED);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
            const ItemStage as = a_stage(g, L, 0), bs = b_stage<DT, TRANSB>(g, bz);
            i32x4 vb[ITEM_U];
            stage_load(as, 0, COLS_NT, tid, va);
            stage_load(bs, 0, COLS_NT, tid, vb);
            if (PROT)
                for (int k = tid; k < COLS_NW * L.KP; k += COLS_NT) vec[L.apart + k] = 0u;
            stage_store(as, 0, COLS_NT, tid, smem + g.lds_a, va);
            stage_store(bs, 0, COLS_NT, tid, smem, vb);
            stage_rest(bs, stage_batch_rows(bs, COLS_NT), COLS_NT, tid, smem);
        }
        item_barrier();
        if (PROT) {
            const ItemArgs &g = item_args();
            const ColsLds L(g, ES, STO, SHARED);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
            uint8_t *terms = reinterpret_cast<uint8_t *>(vec + L.terms);
            uint32_t bmax = 0;
            if (g.cached_b) {
                b_cached<DT>(g, bz, vec + L.b, terms, L.KP, tid, COLS_NT);
            } else {
                const Frag fb(smem, g.pb, lane);
                const uint8_t *Bb = g.B + (long)bz * g.sB * ES;
                const long ldb_bytes = g.ldb * ES;
                b_pass<DT>(g, fb, Ident<DT>(lane), vec + L.b, terms, L.KP, Bb, TRANSB ? ES : ldb_bytes, TRANSB ? ldb_bytes : ES, wave, COLS_NW, lane, &bmax);
                item_max_out<DT>(bmax, Bb, ldb_bytes, TRANSB ? g.N : g.K, TRANSB ? g.K : g.N, lane, vec + L.misc + 8 + wave);
            }
            item_barrier();
        }

        uint32_t amax = 0;
        acc_t cs[TPW][16];                       // column sums: register i of the blocks this wave owns, by lane's row
        float cs_s[STO ? TPW : 1][16], cmax = 0.f;
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) { cs[t][i] = T::zero(); cs_s[STO ? t : 0][i] = 0.f; }

        for (int c = 0;; ++c) {
            bool more;
            {
                const ItemArgs &g = item_args();
                const ColsLds L(g, ES, STO, SHARED);
                more = c + 1 < g.nchunk;
                // (the last chunk may be shorter: rows past M are zero)
                if (more) stage_load(a_stage(g, L, (c + 1) * g.rch * 32), 0, COLS_NT, tid, va);
            }
            if (PROT) {
                // the pass over A: a wave takes every eighth block of rows
                const ItemArgs &g = item_args();
                const ColsLds L(g, ES, STO, SHARED);
                uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec), *my_a = vec + L.apart + wave * L.KP, *b_lds = vec + L.b;
                uint8_t *terms = reinterpret_cast<uint8_t *>(vec + L.terms);
                const int rb0 = c * g.rch, rb1 = min(rb0 + g.rch, g.MB), np = g.steps / 2, M = g.M;
                const Ident<DT> id(lane);
                for (int rb = rb0 + ((wave - rb0) & (COLS_NW - 1)); rb < rb1; rb += COLS_NW) {
                    const uint8_t *pa = smem + g.lds_a + ((rb - rb0) * 32 + l32) * g.pa + lh * 16;
                    SplitDot<DT> sdot;
                    Dot<DT> vdot;
                    const uint8_t *my_terms = split_b_lane<DT>(terms, L.KP, lane);
                    for (int p = 0; p < np; ++p) {
                        const i32x4 x0 = *reinterpret_cast<const i32x4 *>(pa + p * 64);
                        const i32x4 x1 = *reinterpret_cast<const i32x4 *>(pa + p * 64 + 32);
                        Turned<DT> turned;
                        turned.add(x0, x1, id);
                        mag_max<DT>(x0, &amax);
                        mag_max<DT>(x1, &amax);
                        if constexpr (split_b<DT>()) {
                            sdot.add(*reinterpret_cast<const i32x4 *>(my_terms + p * 64), x0);
                            sdot.add(*reinterpret_cast<const i32x4 *>(my_terms + p * 64 + 32), x1);
                        } else {
                            vdot.add(x0, b_lds + p * (64 / ES) + lh * (16 / ES));
                            vdot.add(x1, b_lds + p * (64 / ES) + 32 / ES + lh * (16 / ES));
                        }
                        a_sums<DT>(turned, my_a, p * (T::IS_INT ? 64 : 32), lane);
                        if constexpr (T::IS_INT) {
                            Turned<DT> next;
                            next.add(x1, x1, id);
                            a_sums<DT>(next, my_a, p * 64 + 32, lane);
                        }
                    }
                    acc_t dot;
                    if constexpr (split_b<DT>()) dot = sdot.dot();
                    else dot = vdot.sum();
                    if (lane < 32 && rb * 32 + lane < M) dot = dot_or_again<DT>(dot, g.A + ((long)bz * g.sA + (long)(rb * 32 + lane) * g.lda) * ES, b_lds, g.K);
                    if (lane < 32) vec[L.rcpred + rb * 32 + lane] = as_word(dot);
                }
            }
            {
            // One block of columns per wave: two blocks of rows at a time, two independent chains of MFMAs and
            // of what follows them.
            const ItemArgs &g = item_args();
            const ColsLds L(g, ES, STO, SHARED);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec), *my_rs = vec + L.rspart + wave * L.RC;
            const int rb0 = c * g.rch, rb1 = min(rb0 + g.rch, g.MB), np = g.steps / 2;
            const bool shared = SHARED && shares_last_block(g.NB, g.N);
            const int nb_first = shared && wave == g.NB ? g.NB - 1 : wave;
            const int half = ((rb1 - rb0 + 1) / 2 + R - 1) / R * R;         // a shared block: rows of its owner
            // a lane's place in a block of rows of A, in a fragment of B and in a block of C
            const uint8_t *pa_lane = smem + g.lds_a + l32 * g.pa + lh * 16;
            const ItemOut co = item_out<DT>(g, bz, lane);
            for (int rb = rb0; rb < rb1; rb += R) {
                const Frag fb(smem, g.pb, TRANSB ? lane : item_opaque(lane));        // (B stored K x N: no registers to keep it in)
                const bool two = R == 2 && rb + 1 < rb1;
                const uint8_t *pa0 = pa_lane + (rb - rb0) * 32 * g.pa;
                const uint8_t *pa1 = two ? pa0 + 32 * g.pa : pa0;
                // Wide rows of C: the waves stay within a block of rows of each other, and the lines of C
                // that two of them share are completed while the L2 holds them (int8 1024 x 577 x 577 x 64,
                // protected / unprotected: 489 / 588 us without, 381 / 414 with).
                if (TPW > 1) asm volatile("s_barrier" ::: "memory");
                acc_t rs[2] = {T::zero(), T::zero()};
                float rs_s[2] = {0.f, 0.f};
                static_for<0, TPW>([&](auto t_c) {
                    constexpr int t = decltype(t_c)::value;
                    const int nb = nb_first + COLS_NW * t;
                    if (nb < g.NB && !(shared && nb == g.NB - 1 && (rb - rb0 >= half) != (wave == g.NB))) {
                        accv_t acc[R];
                        auto piece = [&](auto first_c, int p) __attribute__((always_inline)) {
                            constexpr bool FIRST = decltype(first_c)::value;
                            i32x4 xb[2], x0[2], x1[R];
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                xb[u] = fb.get(nb, fb.off(2 * p + u));
                                x0[u] = *reinterpret_cast<const i32x4 *>(pa0 + (2 * p + u) * 32);
                                if (R == 2) x1[u & (R - 1)] = *reinterpret_cast<const i32x4 *>(pa1 + (2 * p + u) * 32);
                            }
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                acc[0] = T::mfma(xb[u], x0[u], FIRST && u == 0 ? item_zero<DT>() : acc[0]);
                                if (R == 2) acc[R - 1] = T::mfma(xb[u], x1[u & (R - 1)], FIRST && u == 0 ? item_zero<DT>() : acc[R - 1]);
                            }
                        };
                        piece(std::true_type{}, 0);
                        for (int p = 1; p < np; ++p) piece(std::false_type{}, p);
                        const int n0 = nb * 32;
                        static_for<0, R>([&](auto r_c) {
                            constexpr int r = decltype(r_c)::value;
                            if (r == 0 || two) {
                                const int m0 = (rb + r) * 32;
                                if (PROT) {
                                    if (bz == g.inj_b && g.inj_row >= m0 && g.inj_row < m0 + 32) item_flip<DT>(g, acc[r], m0, n0, lane);
#pragma unroll
                                    for (int i = 0; i < 16; ++i) cs[t][i] = add_t(cs[t][i], (acc_t)acc[r][i]);
                                    rs[r] = add_t(rs[r], sum16<acc_t>(acc[r]));
                                }
                                if constexpr (T::IS_INT) {
                                    uint32_t w[16];
#pragma unroll
                                    for (int i = 0; i < 16; ++i) w[i] = (uint32_t)acc[r][i];
                                    store_block<DT>(co, w, m0, n0, lane);
                                } else {
                                    uint32_t w[8];
                                    pack_block<DT>(acc[r], w);
                                    if constexpr (STO) {
#pragma unroll
                                        for (int j = 0; j < 8; ++j) {
                                            const float y0 = unpack_lo<DT>(w[j]), y1 = unpack_hi<DT>(w[j]);
                                            rs_s[r] += y0 + y1;
                                            cs_s[t][2 * j] += y0;
                                            cs_s[t][2 * j + 1] += y1;
                                            cmax = fmaxf(cmax, fmaxf(fabsf(y0), fabsf(y1)));
                                        }
                                    }
                                    store_block<DT>(co, w, m0, n0, lane);
                                }
                            }
                        });
                    }
                });
                if (PROT) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        if (r == 0 || two) {
                            const int at = (rb + r - rb0) * 32 + l32;
                            my_rs[at] = as_word(add_xor32(rs[r]));     // (both halves of the wave)
                            if (STO) vec[L.rsspart + wave * L.RC + at] = __float_as_uint(add_xor32(rs_s[r]));
                        }
                    }
                }
            }
            }
            if (PROT && !more) {
                // what the last waves are waited for anyway: the largest |element| of A, the column sums of C over the lanes
                const ItemArgs &g = item_args();
                const ColsLds L(g, ES, STO, SHARED);
                uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
                item_max_out<DT>(amax, g.A + (long)bz * g.sA * ES, g.lda * ES, g.M, g.K, lane, vec + L.misc + wave);
                if (STO) {
                    const float m = wave_max(cmax);
                    if (lane == 0) vec[L.misc + 40 + wave] = __float_as_uint(m);
                }
                const int blocks = g.NB + (SHARED && shares_last_block(g.NB, g.N) ? 1 : 0);
                static_for<0, TPW>([&](auto t_c) {
                    constexpr int t = decltype(t_c)::value;
                    const int nb = wave + COLS_NW * t;
                    if (nb < blocks) {
                        const acc_t v = fold16<acc_t>(cs[t], lane);
                        if ((lane & 1) == 0) vec[L.ccobs + nb * 32 + fold16_column(lane)] = as_word(v);
                        if (STO) {
                            const float x = fold16<float>(cs_s[STO ? t : 0], lane);
                            if ((lane & 1) == 0) vec[L.ccsto + nb * 32 + fold16_column(lane)] = __float_as_uint(x);
                        }
                    }
                });
            }
            item_barrier();
            const ItemArgs &g = item_args();
            const ColsLds L(g, ES, STO, SHARED);
            if (PROT) {
                uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
                const int r0 = c * g.rch * 32, rows = min(g.rch, g.MB - c * g.rch) * 32;
                for (int r = tid; r < rows; r += COLS_NT) {
                    vec[L.rcobs + r0 + r] = as_word(sum_copies<acc_t>(vec + L.rspart + r, L.RC, COLS_NW));
                    if (STO) vec[L.rcsto + r0 + r] = __float_as_uint(sum_copies<float>(vec + L.rsspart + r, L.RC, COLS_NW));
                }
            }
            if (!more) break;
            stage_store(a_stage(g, L, 0), 0, COLS_NT, tid, smem + g.lds_a, va);
            item_barrier();
        }
        const bool last = bz + (int)gridDim.x >= item_args().batch;
        if (PROT) {
            {
                const ItemArgs &g = item_args();
                const ColsLds L(g, ES, STO, SHARED);
                uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
                const int ract = g.MB < COLS_NW ? g.MB : COLS_NW;            // waves that have a share of the pass over A
                // (by the last waves: the first ones add up the rows' sums)
                for (int k = COLS_NT - 1 - tid; k < L.KP; k += COLS_NT) {
                    acc_t v = sum_copies<acc_t>(vec + L.apart + k, L.KP, ract);
                    if (k < g.K) v = finite_or_again<DT>(v, g.A + ((long)bz * g.sA + k) * ES, g.lda * ES, g.M);
                    vec[L.a + k] = as_word(v);
                }
            }
            item_barrier();
            const ItemArgs &g = item_args();
            const ColsLds L(g, ES, STO, SHARED);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec), *misc = vec + L.misc, *a_lds = vec + L.a;
            const int N = g.N;
            const bool shared = SHARED && shares_last_block(g.NB, N);
            const Frag fb(smem, g.pb, lane);
            const ItemTol tt = item_tolerance<DT>(g, misc, COLS_NW, bz);
            const float tol_c = g.tau_override_cols > 0.f ? g.tau_override_cols : tt.tol;
            // a B from the resident B (the last waves first: the first ones have the rows)
            for (int nb = COLS_NW - 1 - wave; nb < g.NB; nb += COLS_NW) {
                Dot<DT> vdot;
                for (int s = 0; s < g.steps; ++s) vdot.add(fb.get(nb, fb.at(s)), a_lds + s * (32 / ES) + lh * (16 / ES));
                const acc_t d = vdot.sum();
                const int n = nb * 32 + l32;
                bool fl = false;
                if (lane < 32 && n < N) {
                    const long o = (long)bz * N + n;
                    const bool two = shared && nb == g.NB - 1;
                    uint32_t obs = vec[L.ccobs + n];
                    if (two) obs = as_word(add_t(from_word<acc_t>(obs), from_word<acc_t>(vec[L.ccobs + n + 32])));
                    g.cc_pred[o] = as_word(d);
                    g.cc_obs[o] = obs;
                    if (STO) g.cc_sto[o] = two ? __float_as_uint(__uint_as_float(vec[L.ccsto + n]) + __uint_as_float(vec[L.ccsto + n + 32])) : vec[L.ccsto + n];
                    fl = mismatch<T::IS_INT>(obs, as_word(d), tol_c);
                    g.col_flag[o] = fl ? 1 : 0;
                }
                nc_w += __popcll(__ballot(fl));
            }
            nr_w += item_rows_out<DT>(g, bz, COLS_NT, tid, vec + L.rcobs, vec + L.rcpred, STO ? vec + L.rcsto : nullptr, a_lds, vec + L.b, tt.tol,
                                      misc + 16 + wave);
            if (last && lane == 0) { misc[24 + wave] = nr_w; misc[24 + COLS_NW + wave] = nc_w; }
            item_barrier();
            // (past this barrier only these scalars' words are read: the next item may begin)
            if (tid == 64) item_scalars_out<DT, STO>(g, bz, misc, COLS_NW, tt);
            if (last && tid == 0) item_ticket(g, misc + 24, COLS_NW);
        }
        // (unprotected: the barrier behind the last chunk is the one before the next item's first store)
        if (last) return;
    }
}

// ------------------------------------------------------------------------------------------
// The sums of a shared block's second half lie behind the others: a block is shared where they fit beside the chunk of rows and the number
// of workgroups that the item has without.  (512 items of 367 x 161 x 128, bf16: 36.8 us, 46.7 with a chunk more.)
static size_t cols_bytes(const ItemArgs &g, int es, bool protect, bool sto, bool shared)
{
    return (size_t)g.lds_vec + (protect ? (size_t)ColsLds(g, es, sto, shared).total * 4 : 0);
}

size_t item_cols_lds(int dt, const Shape &s, bool protect, bool sto, ItemArgs *g)
{
    const int es = elem_size(dt);
    if (g->NB > 3 * COLS_NW || (sto && g->NB > COLS_NW)) return 0;
    // one batch of loads must hold a chunk of A
    const int most = ((COLS_NT >> g->a_lg) * ITEM_U) / 32;
    const size_t budgets[2] = {(size_t)ITEM_LDS_LIMIT / 2, (size_t)ITEM_LDS_LIMIT};
    for (size_t budget : budgets)
        for (int n = (g->MB + most - 1) / most; n <= g->MB; ++n) {
            g->rch = (g->MB + n - 1) / n;
            g->nchunk = (g->MB + g->rch - 1) / g->rch;
            g->lds_a = (g->b_rows * g->pb + 15) / 16 * 16;
            g->lds_vec = g->lds_a + g->rch * 32 * g->pa;
            const size_t bytes = cols_bytes(*g, es, protect, sto, false);
            if (bytes <= budget) {
                const size_t sharing = cols_bytes(*g, es, protect, sto, true);
                return takes_sharing_kernel(dt, s.transB, protect, sto, g->NB, s.N) && sharing <= budget ? sharing : bytes;
            }
            // smaller chunks cost more in barriers than a second workgroup gives (one block: see gemm_item_eligible)
            if (g->rch <= (budget < (size_t)ITEM_LDS_LIMIT ? 2 : 1)) break;
        }
    return 0;
}

template <int DT, int TPW, bool PROT, bool TRANSB, bool STO>
static hipError_t cols_one(const ItemArgs &g, size_t smem, hipStream_t st)
{
    auto kern = item_cols_kernel<DT, TPW, PROT, TRANSB, STO, false>;
    if constexpr (TPW == 1)
        if (takes_sharing_kernel(DT, TRANSB, PROT, STO, g.NB, g.N) && smem >= cols_bytes(g, Traits<DT>::ES, PROT, STO, true)) kern = item_cols_kernel<DT, TPW, PROT, TRANSB, STO, true>;
    hipError_t e = ensure_max_lds(reinterpret_cast<const void *>(kern), ITEM_LDS_LIMIT);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)(g.batch < ITEM_MAX_BLOCKS ? g.batch : ITEM_MAX_BLOCKS);
    // Wide rows of C: one workgroup per compute unit.  Two keep twice as many lines of C open, and the L2
    // lets go of more of them half written (int8 1024 x 577 x 577 x 64, protected / unprotected: 378 / 412 us
    // with two, 349 / 370 with one).
    if (TPW > 1 && smem <= (size_t)ITEM_LDS_LIMIT / 2) smem = (size_t)ITEM_LDS_LIMIT / 2 + 1024;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(COLS_NT), smem, st, g);
    return hipGetLastError();
}
template <int DT, bool TRANSB>
static hipError_t cols_mode(bool protect, const ItemArgs &g, size_t smem, hipStream_t st)
{
    if (g.NB > COLS_NW) return protect ? cols_one<DT, 3, true, TRANSB, false>(g, smem, st) : cols_one<DT, 3, false, TRANSB, false>(g, smem, st);
    if (!protect) return cols_one<DT, 1, false, TRANSB, false>(g, smem, st);
    if constexpr (DT != DT_I8)
        if (g.cc_sto) return cols_one<DT, 1, true, TRANSB, true>(g, smem, st);
    return cols_one<DT, 1, true, TRANSB, false>(g, smem, st);
}
hipError_t launch_item_cols(int dt, bool protect, bool transB, const ItemArgs &g, size_t smem, hipStream_t st)
{
    switch (dt) {
    case DT_I8:   return transB ? cols_mode<DT_I8, true>(protect, g, smem, st) : cols_mode<DT_I8, false>(protect, g, smem, st);
    case DT_BF16: return transB ? cols_mode<DT_BF16, true>(protect, g, smem, st) : cols_mode<DT_BF16, false>(protect, g, smem, st);
    case DT_F16:  return transB ? cols_mode<DT_F16, true>(protect, g, smem, st) : cols_mode<DT_F16, false>(protect, g, smem, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace abft
