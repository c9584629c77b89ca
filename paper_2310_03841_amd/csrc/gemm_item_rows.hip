// Batches of small problems, N <= 128 (attn V, and Q K^T of few tokens): a wave owns rows of its item.
// See gemm_item.h for what is common.
//
// B of the item lies in LDS.  Each of the four or eight waves takes blocks of 32 rows of A in turn, and
// fetches their fragments from global memory straight into registers, eight steps of K ahead: every
// element of A is used by one wave only, so a trip through LDS would buy nothing, and no wave waits
// for another between the start of an item and its checks.  Four steps, 128 bytes of each row, are
// requested together (two by two the L1 loses half of a line before it is used: int8 577 x 64 x 577,
// 1024 items 161 us, so 152).  From a fragment come its MFMAs, its share of a = e^T A and of A b; row
// sums and the row dot stay with the lane that owns the row.
//
// Measured (384 items 197 x 64 x 197 bf16, attn V of 32 images; floor 9.8 us): 45.8 us with one workgroup
// of four computing waves and a loading wave per item and the sums along K in vector instructions, 21.6
// so, 19.8 since the phases read their own arguments (item_args), 11.5 unprotected (before: 21.5).  What bounds it: an item is one chain of some
// 2000 instructions per wave (load B, b, the row blocks, the checks) and the 384 items are 1.5 for each compute unit.
#include "gemm_item.h"

namespace abft {

// pitch of a B stored K x N: an odd number of 32-byte (int8: 16-byte) pieces
__host__ __device__ constexpr int rows_kn_pitch(int es, int tpw) { return es == 2 ? tpw * 64 + 32 : tpw * 32 + 16; }

// Copies of a = e^T A that the waves add to: one each, so that the order of additions is fixed; of integers two for all, which leaves
// deep items the LDS for a second workgroup on the compute unit (577 x 64 x 577: 87 KB with eight copies, 71 so).
__host__ __device__ constexpr int rows_a_copies(int es, int nw) { return es == 1 ? 2 : nw; }

constexpr int ROWS_RING = 4;                     // pieces of two steps of A a wave keeps in flight

// Offsets (words) of the vectors behind B.
struct RowsLds {
    int KP, Mr, Nr, rcobs, rcpred, a, b, terms, apart, cspart, ccpred, misc, rcsto, csspart, total;
    __host__ __device__ RowsLds(const ItemArgs &g, int es, int nw, bool sto)
    {
        KP = g.steps * (es == 2 ? 16 : 32);
        Mr = g.MB * 32; Nr = g.NB * 32;
        int o = 0;
        a = o; o += KP;
        b = o; o += KP;
        terms = o; o += KP * es;                 // [4][KP] elements
        apart = o; o += rows_a_copies(es, nw) * KP;
        rcobs = o; o += Mr;
        rcpred = o; o += Mr;
        cspart = o; o += nw * Nr;
        ccpred = o; o += Nr;
        misc = o; o += 48;                       // 0..7 max|A|, 8..15 max|B|, 16..23 a.b per wave; 24..39 flag counts; 40..47 max|C as stored|
        rcsto = o; o += sto ? Mr : 0;
        csspart = o; o += sto ? nw * Nr : 0;
        total = o;
    }
};

template <int DT, int TPW, bool PROT, bool TRANSB, bool STO>
__global__ __launch_bounds__(512, TPW == 2 && !STO ? 4 : 2) void item_rows_kernel(ItemArgs)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    typedef typename T::accv_t accv_t;
    fetch_args<ItemArgs>();
    constexpr int ES = T::ES;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane_id = threadIdx.x & 63, nt = blockDim.x, nw = nt >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    typedef FragB<DT, TRANSB, rows_kn_pitch(ES, TPW)> Frag;
    unsigned nr_w = 0, nc_w = 0;

    for (int bz = blockIdx.x;; bz += gridDim.x) {
        const int tid = item_opaque(threadIdx.x), lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
        const uint8_t *Ab;
        long lda_bytes;
        int M, MB, last_ch;
        i32x4 fa[ROWS_RING][2];
        // piece p of a row block: rows past M and chunks past K fetch the last valid ones, cleared below
        const uint8_t *arow;
        auto row_of = [&](int rb) __attribute__((always_inline)) {
            int r = rb * 32 + l32;
            r = r < M ? r : M - 1;
            arow = Ab + (long)r * lda_bytes;
        };
        auto fetch = [&](int p, i32x4 (&f)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                int ch = 2 * (2 * p + u);
                asm volatile("" : "+s"(ch));
                ch += lh;
                ch = ch < last_ch ? ch : last_ch;
                f[u] = *reinterpret_cast<const i32x4 *>(arow + ch * 16);
            }
        };
        {
            const ItemArgs &g = item_args();
            Ab = g.A + (long)bz * g.sA * ES;
            lda_bytes = g.lda * ES;
            M = g.M; MB = g.MB; last_ch = g.nch - 1;
            arow = Ab;
            if (wave < MB) {
                row_of(wave);
                static_for<0, ROWS_RING>([&](auto j_c) { fetch(decltype(j_c)::value, fa[decltype(j_c)::value]); });
            }
            const RowsLds L(g, ES, nw, STO);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
            const ItemStage bs = b_stage<DT, TRANSB>(g, bz);
            i32x4 v[ITEM_U];
            stage_load(bs, 0, nt, tid, v);
            if (PROT) {
                for (int k = tid; k < rows_a_copies(ES, nw) * L.KP; k += nt) vec[L.apart + k] = 0u;
                for (int n = tid; n < L.Nr; n += nt) vec[L.ccpred + n] = 0u;
            }
            stage_store(bs, 0, nt, tid, smem, v);
            stage_rest(bs, stage_batch_rows(bs, nt), nt, tid, smem);
        }
        item_barrier();
        if (PROT) {
            const ItemArgs &g = item_args();
            const RowsLds L(g, ES, nw, STO);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
            uint8_t *terms = reinterpret_cast<uint8_t *>(vec + L.terms);
            uint32_t bmax = 0;
            if (g.cached_b) {
                b_cached<DT>(g, bz, vec + L.b, terms, L.KP, tid, nt);
            } else {
                const Frag fb(smem, g.pb, lane);
                const uint8_t *Bb = g.B + (long)bz * g.sB * ES;
                const long ldb_bytes = g.ldb * ES;
                b_pass<DT>(g, fb, Ident<DT>(lane), vec + L.b, terms, L.KP, Bb, TRANSB ? ES : ldb_bytes, TRANSB ? ldb_bytes : ES, wave, nw, lane, &bmax);
                item_max_out<DT>(bmax, Bb, ldb_bytes, TRANSB ? g.N : g.K, TRANSB ? g.K : g.N, lane, vec + L.misc + 8 + wave);
            }
            item_barrier();
        }

        uint32_t amax = 0;
        acc_t csum[TPW];                         // column sums, folded: column fold16_column(lane) of each block
        float csum_s[STO ? TPW : 1], cmax = 0.f;
#pragma unroll
        for (int t = 0; t < TPW; ++t) { csum[t] = T::zero(); csum_s[STO ? t : 0] = 0.f; }
        const Ident<DT> id(lane);
        for (int rb = wave; rb < MB; rb += nw) {
            const ItemArgs &g = item_args();
            const RowsLds L(g, ES, nw, STO);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec), *my_a = vec + L.apart + (T::IS_INT ? wave & 1 : wave) * L.KP, *b_lds = vec + L.b;
            uint8_t *terms = reinterpret_cast<uint8_t *>(vec + L.terms);
            const int np = g.steps / 2, kbytes = g.K * ES;
            const int lane = item_opaque(lane_id), l32 = lane & 31, lh = lane >> 5;
            const Frag fb(smem, g.pb, lane);
            const int m0 = rb * 32;
            const bool edge = m0 + 32 > M;
            accv_t acc[TPW];
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][i] = T::zero();
            SplitDot<DT> sdot;
            Dot<DT> vdot;
            const uint8_t *my_terms = split_b_lane<DT>(terms, L.KP, lane);
            // Pieces of A are fetched ROWS_RING ahead.  Every load is issued unconditionally, so that the
            // waits count exactly: in the last group of a row block they are those of the wave's next
            // one, and where there is none all lanes ask for the same 16 bytes.
            for (int p0 = 0; p0 < np; p0 += ROWS_RING) {
                int f0 = p0 + ROWS_RING;
                if (f0 >= np) {
                    f0 = 0;
                    if (rb + nw < MB) row_of(rb + nw);
                    else { arow = Ab; last_ch = 0; }
                }
                static_for<0, ROWS_RING>([&](auto j_c) {
                    constexpr int j = decltype(j_c)::value;
                    const int p = p0 + j;
                    if (p < np) {
                        int s = 2 * p;
                        asm volatile("" : "+s"(s));             // addresses of a piece are formed at the piece
                        i32x4 bf[2][TPW], x[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int at = fb.at(s + u);
#pragma unroll
                            for (int t = 0; t < TPW; ++t) bf[u][t] = fb.get(t, at);
                            x[u] = fa[j][u];
                            if (edge) x[u] = m0 + l32 < M ? x[u] : i32x4{0, 0, 0, 0};
                            if ((s + u + 1) * 32 > kbytes) x[u] = mask_chunk(x[u], kbytes - (2 * (s + u) + lh) * 16);
                        }
                        Turned<DT> turned;
                        if (PROT) {
                            turned.add(x[0], x[1], id);
                            mag_max<DT>(x[0], &amax);
                            mag_max<DT>(x[1], &amax);
                            if constexpr (split_b<DT>()) {
#pragma unroll
                                for (int u = 0; u < 2; ++u) sdot.add(*reinterpret_cast<const i32x4 *>(my_terms + (s + u) * 32), x[u]);
                            } else {
#pragma unroll
                                for (int u = 0; u < 2; ++u) vdot.add(x[u], b_lds + (s + u) * (32 / ES) + lh * (16 / ES));
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int t = 0; t < TPW; ++t) acc[t] = T::mfma(bf[u][t], x[u], acc[t]);
                        if (PROT) {
                            a_sums<DT, T::IS_INT>(turned, my_a, T::IS_INT ? s * 32 : s * 16, lane);
                            if constexpr (T::IS_INT) {
                                Turned<DT> next;
                                next.add(x[1], x[1], id);
                                a_sums<DT, T::IS_INT>(next, my_a, s * 32 + 32, lane);
                            }
                        }
                    }
                    if constexpr (j & 1) { fetch(f0 + j - 1, fa[j - 1]); fetch(f0 + j, fa[j]); }     // 128 bytes of a row in a row
                });
                if (PROT) {
                    if constexpr (split_b<DT>()) sdot.flush();
                    else vdot.flush();
                }
            }
            // ---- the block row leaves
            const ItemOut co = item_out<DT>(g, bz, lane);
            acc_t rs = T::zero();
            float rs_s = 0.f;
            static_for<0, TPW>([&](auto t_c) {
                constexpr int t = decltype(t_c)::value;
                if (t < g.NB) {
                    if (PROT) {
                        if (bz == g.inj_b && g.inj_row >= m0 && g.inj_row < m0 + 32) item_flip<DT>(g, acc[t], m0, t * 32, lane);
                        rs = add_t(rs, sum16<acc_t>(acc[t]));
                        csum[t] = add_t(csum[t], fold16<acc_t>(acc[t], lane));
                    }
                    if constexpr (T::IS_INT) {
                        uint32_t w[16];
#pragma unroll
                        for (int i = 0; i < 16; ++i) w[i] = (uint32_t)acc[t][i];
                        store_block<DT>(co, w, m0, t * 32, lane);
                    } else {
                        uint32_t w[8];
                        pack_block<DT>(acc[t], w);
                        if constexpr (STO) {
                            float sv[16];
#pragma unroll
                            for (int j = 0; j < 8; ++j) { sv[2 * j] = unpack_lo<DT>(w[j]); sv[2 * j + 1] = unpack_hi<DT>(w[j]); }
#pragma unroll
                            for (int j = 0; j < 8; ++j) cmax = fmaxf(cmax, fmaxf(fabsf(sv[2 * j]), fabsf(sv[2 * j + 1])));
                            rs_s += sum16<float>(sv);
                            csum_s[t] += fold16<float>(sv, lane);
                        }
                        store_block<DT>(co, w, m0, t * 32, lane);
                    }
                }
            });
            if (PROT) {
                const acc_t rsum = add_xor32(rs);
                acc_t dot;
                if constexpr (split_b<DT>()) dot = sdot.dot();
                else dot = vdot.sum();
                if (lane < 32 && m0 + lane < M) dot = dot_or_again<DT>(dot, Ab + (long)(m0 + lane) * lda_bytes, b_lds, g.K);
                if (STO) rs_s = add_xor32(rs_s);
                if (lane < 32) {
                    vec[L.rcobs + m0 + lane] = as_word(rsum);
                    vec[L.rcpred + m0 + lane] = as_word(dot);
                    if (STO) vec[L.rcsto + m0 + lane] = __float_as_uint(rs_s);
                }
            }
        }
        const bool last = bz + (int)gridDim.x >= item_args().batch;
        if (PROT) {
            {
                const ItemArgs &g = item_args();
                const RowsLds L(g, ES, nw, STO);
                uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec), *misc = vec + L.misc, *my_cs = vec + L.cspart + wave * L.Nr;
                if ((lane & 1) == 0) {
#pragma unroll
                    for (int t = 0; t < TPW; ++t)
                        if (t < g.NB) {
                            my_cs[t * 32 + fold16_column(lane)] = as_word(csum[t]);
                            if (STO) vec[L.csspart + wave * L.Nr + t * 32 + fold16_column(lane)] = __float_as_uint(csum_s[t]);
                        }
                }
                item_max_out<DT>(amax, Ab, lda_bytes, M, g.K, lane, misc + wave);
                if (STO) {
                    const float m = wave_max(cmax);
                    if (lane == 0) misc[40 + wave] = __float_as_uint(m);
                }
            }
            item_barrier();
            const int wact = MB < nw ? MB : nw;  // waves that have rows
            {
                const ItemArgs &g = item_args();
                const RowsLds L(g, ES, nw, STO);
                uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec);
                const int K = g.K;
                for (int k = tid; k < L.KP; k += nt) {
                    acc_t v = sum_copies<acc_t>(vec + L.apart + k, L.KP, T::IS_INT ? 2 : wact);
                    if (k < K) v = finite_or_again<DT>(v, Ab + (long)k * ES, lda_bytes, M);
                    vec[L.a + k] = as_word(v);
                }
            }
            item_barrier();
            const ItemArgs &g = item_args();
            const RowsLds L(g, ES, nw, STO);
            uint32_t *vec = reinterpret_cast<uint32_t *>(smem + g.lds_vec), *misc = vec + L.misc, *ccpred = vec + L.ccpred, *a_lds = vec + L.a;
            const int N = g.N;
            // ---- a B from the resident B: a wave takes every nw-th step of K
            {
                const Frag fb(smem, g.pb, lane);
                Dot<DT> d[TPW];
                for (int s = wave; s < g.steps; s += nw) {
                    const int at = fb.at(s);
#pragma unroll
                    for (int t = 0; t < TPW; ++t)
                        if (t < g.NB) d[t].add(fb.get(t, at), a_lds + s * (32 / ES) + lh * (16 / ES));
                }
                if (wave < g.steps) {
#pragma unroll
                    for (int t = 0; t < TPW; ++t) {
                        const acc_t v = d[t].sum();
                        if (t < g.NB && lane < 32) lds_add_word(ccpred + t * 32 + lane, v);
                    }
                }
            }
            const ItemTol tt = item_tolerance<DT>(g, misc, nw, bz);
            nr_w += item_rows_out<DT>(g, bz, nt, tid, vec + L.rcobs, vec + L.rcpred, STO ? vec + L.rcsto : nullptr, a_lds, vec + L.b, tt.tol, misc + 16 + wave);
            item_barrier();
            if (tid < L.Nr) {
                bool fl = false;
                if (tid < N) {
                    const long o = (long)bz * N + tid;
                    const acc_t obs = sum_copies<acc_t>(vec + L.cspart + tid, L.Nr, wact);
                    const uint32_t pred = ccpred[tid];
                    g.cc_pred[o] = pred;
                    g.cc_obs[o] = as_word(obs);
                    if (STO) g.cc_sto[o] = __float_as_uint(sum_copies<float>(vec + L.csspart + tid, L.Nr, wact));
                    fl = mismatch<T::IS_INT>(as_word(obs), pred, g.tau_override_cols > 0.f ? g.tau_override_cols : tt.tol);
                    g.col_flag[o] = fl ? 1 : 0;
                }
                nc_w += __popcll(__ballot(fl));
            }
            if (last && lane == 0) { misc[24 + wave] = nr_w; misc[24 + nw + wave] = nc_w; }
            item_barrier();
            // (past this barrier only these scalars' words are read: the next item may begin)
            if (tid == 64) item_scalars_out<DT, STO>(g, bz, misc, nw, tt);
            if (last && tid == 0) item_ticket(g, misc + 24, nw);
        } else {
            item_barrier();                      // LDS is reused by the next item
        }
        if (last) return;
    }
}

// ------------------------------------------------------------------------------------------
static int rows_waves(const ItemArgs &g) { return g.MB <= 4 ? 4 : 8; }

size_t item_rows_lds(int dt, const Shape &s, bool protect, bool sto, ItemArgs *g)
{
    const int es = elem_size(dt);
    if (g->NB > 4) return 0;
    // two or four blocks of columns are multiplied, whether or not the last holds any
    const int tpw = g->NB <= 2 ? 2 : 4;
    if (s.transB) g->b_rows = tpw * 32;
    else { g->pb = rows_kn_pitch(es, tpw); g->b_chunks = tpw * 2 * es; }
    g->b_lg = item_log2(g->b_chunks);
    g->lds_a = 0;
    g->lds_vec = (g->b_rows * g->pb + 15) / 16 * 16;
    const RowsLds L(*g, es, rows_waves(*g), sto);
    const size_t bytes = (size_t)g->lds_vec + (protect ? (size_t)L.total * 4 : 0);
    return bytes <= (size_t)ITEM_LDS_LIMIT ? bytes : 0;
}

template <int DT, int TPW, bool PROT, bool TRANSB, bool STO>
static hipError_t rows_one(const ItemArgs &g, size_t smem, hipStream_t st)
{
    auto kern = item_rows_kernel<DT, TPW, PROT, TRANSB, STO>;
    hipError_t e = ensure_max_lds(reinterpret_cast<const void *>(kern), ITEM_LDS_LIMIT);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)(g.batch < ITEM_MAX_BLOCKS ? g.batch : ITEM_MAX_BLOCKS);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3((unsigned)rows_waves(g) * 64), smem, st, g);
    return hipGetLastError();
}
template <int DT, int TPW, bool TRANSB>
static hipError_t rows_mode(bool protect, const ItemArgs &g, size_t smem, hipStream_t st)
{
    if (!protect) return rows_one<DT, TPW, false, TRANSB, false>(g, smem, st);
    if constexpr (DT != DT_I8)
        if (g.cc_sto) return rows_one<DT, TPW, true, TRANSB, true>(g, smem, st);
    return rows_one<DT, TPW, true, TRANSB, false>(g, smem, st);
}
template <int DT> static hipError_t rows_dt(bool protect, bool transB, const ItemArgs &g, size_t smem, hipStream_t st)
{
    if (g.NB <= 2) return transB ? rows_mode<DT, 2, true>(protect, g, smem, st) : rows_mode<DT, 2, false>(protect, g, smem, st);
    return transB ? rows_mode<DT, 4, true>(protect, g, smem, st) : rows_mode<DT, 4, false>(protect, g, smem, st);
}
hipError_t launch_item_rows(int dt, bool protect, bool transB, const ItemArgs &g, size_t smem, hipStream_t st)
{
    switch (dt) {
    case DT_I8:   return rows_dt<DT_I8>(protect, transB, g, smem, st);
    case DT_BF16: return rows_dt<DT_BF16>(protect, transB, g, smem, st);
    case DT_F16:  return rows_dt<DT_F16>(protect, transB, g, smem, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace abft
