// Which batches of small problems one workgroup per item takes, and how (gemm_item.h).
#include <algorithm>

#include "gemm_item.h"

namespace abft {

// Fewer items leave most compute units without work.  Measured, one workgroup per item / the general
// kernel's tiles and check: bf16 Q K^T 197 x 197 x 64, 24 items 15.2 / 12.4 us, 48 items 15.7 / 15.6, 384 items
// 21.7 / 57.6; int8 attn V 577 x 64 x 577, 16 items 23.8 / 14.7, 48 items 24.4 / 28.9.
constexpr int ITEM_MIN_BATCH = 64;
constexpr int ITEM_MAX_N = 640, ITEM_MAX_M = 1024, ITEM_MAX_THREADS = 512;

// Offsets inside an item are 32-bit numbers (ItemStage, ItemOut): the rows that batches of loads reach, past the last one too, and the row blocks of C
// must end below 2^31 bytes, with a row to spare for what a lane adds along one.  That bounds rows times their distance: up to 1024 rows reached may be 2 MB
// apart (heads side by side, q, k and v of 16 heads x 64 in bf16: 340 images).  Wider ones are for the tiles; 86 images there / here, us: Q K^T 577 x 577 x 64
// 1006 / 355, unprotected 643 / 332, attn V 646 / 340, unprotected 287 / 298.  The kernel by rows reads A by whole addresses.
static bool item_offsets_fit(int dt, const Shape &s, const ItemArgs &g)
{
    const long es = elem_size(dt);
    auto reach = [](int rows, int lg) { const long batch = (long)(ITEM_MAX_THREADS >> lg) * ITEM_U; return (rows + batch - 1) / batch * batch; };
    auto fits = [](long rows, long ld_bytes) { return ld_bytes <= INT32_MAX / (rows + 1); };
    if (!fits(reach(g.b_rows, g.b_lg), s.ldb * es) || !fits((long)g.MB * 32, s.ldc * out_size(dt))) return false;
    return s.N <= 128 || fits(std::max(reach(g.rch * 32, g.a_lg), (long)s.M), s.lda * es);
}

// Fills in the geometry; returns the bytes of LDS, 0 if the item does not fit.
static size_t item_plan(int dt, const Shape &s, bool protect, bool sto, ItemArgs *g)
{
    const int es = elem_size(dt);
    if (s.N > ITEM_MAX_N || s.M > ITEM_MAX_M) return 0;
    // N <= 128: as deep as B fits in LDS (bf16 attn V of 577 tokens, 400 items: 111 us, on tiles 281; 400
    // tokens of head dimension 128, 300 items: 65 / 131).  Wider items hold whole rows of A beside B.
    if ((long)s.K * es > (s.N <= 128 ? 1600 : s.N <= 256 ? 384 : 256)) return 0;
    g->M = s.M; g->N = s.N; g->K = s.K; g->batch = s.batch;
    g->nch = (s.K * es + 15) / 16;
    g->steps = ((s.K * es + 31) / 32 + 1) / 2 * 2;
    g->NB = (s.N + 31) / 32;
    g->MB = (s.M + 31) / 32;
    g->pa = 16 * (2 * g->steps + 1);
    if (s.transB) {
        g->b_rows = g->NB * 32;
        g->b_chunks = 2 * g->steps;
        g->pb = g->pa;
    } else {
        g->b_rows = g->steps * (32 / es);
        g->b_chunks = g->NB * 2 * es;
        g->pb = g->NB * 32 * es + 16 * es;
    }
    g->b_lg = item_log2(g->b_chunks);
    g->a_lg = item_log2(2 * g->steps);
    g->rch = g->MB;
    g->nchunk = 1;
    const size_t smem = s.N <= 128 ? item_rows_lds(dt, s, protect, sto, g) : item_cols_lds(dt, s, protect, sto, g);
    return smem && item_offsets_fit(dt, s, *g) ? smem : 0;
}

// Where B leaves room for one block of rows of A at a time only, an item has a barrier per block and the
// compute unit to itself: it takes more items before that is the faster way.  Measured, item kernel / tiles,
// int8 Q K^T of 478 keys, K = 256: 64 queries, 104 items 20.1 / 31.1 us; 256 queries, 64 items 41.3 / 33.6, 104 items
// 42.0 / 49.1, 256 items 46.4 / 106; 1024 queries, 104 items 125 / 113, 120 items 132 / 132; unprotected 128
// queries, 150 items 18.4 / 16.3; 33 queries, 150 items 9.9 / 7.8; 256 queries, 256 items 32.1 / 44.8.
constexpr int ONE_BLOCK_MIN_BATCH = 104, ONE_BLOCK_MIN_BATCH_TALL = 120, ONE_BLOCK_MIN_BATCH_PLAIN = 256;

// Deep items (N <= 128) hold most of a compute unit's LDS while its waves wait for the whole of B first; without
// checksums to form the tiles are then often the faster way, unless there are rows and items enough (407
// shapes: four are more than 5 % slower by this line than on the item kernel, 58 were slower on it than on the tiles
// of the kernel before): bf16 9 x 128 x 380, 369 items 21.9 us / tiles 9; 577 x 64 x 577, 256 items 36.9 / 52.2.
constexpr int DEEP_MIN_BATCH_PLAIN = 128;

// protect: of two problems of one shape the unprotected one may be tiled
bool gemm_item_eligible(int dt, const Shape &s, bool stored_sums, bool protect)
{
    if (s.batch < ITEM_MIN_BATCH) return false;
    ItemArgs g;
    if (item_plan(dt, s, true, stored_sums && dt != DT_I8, &g) == 0) return false;
    if (s.N <= 128)
        return protect || (long)s.K * elem_size(dt) <= (s.N <= 64 ? 640 : 384) || (g.MB >= 5 && s.batch >= DEEP_MIN_BATCH_PLAIN);
    if (g.rch > 1 || g.MB == 1) return true;
    return protect ? s.batch >= (g.MB <= 8 ? ONE_BLOCK_MIN_BATCH : ONE_BLOCK_MIN_BATCH_TALL)
                   : s.batch >= ONE_BLOCK_MIN_BATCH_PLAIN && g.MB >= 4;
}

hipError_t launch_gemm_item(int dt, bool protect, bool cached_b, bool stored_sums, const void *A, const void *B, void *C,
                            const Shape &s, const Workspace &w, const Verdict *v, const InjectArm &arm,
                            hipStream_t st)
{
    const bool sto = protect && stored_sums && dt != DT_I8;
    if (protect && v == nullptr) return hipErrorInvalidValue;
    ItemArgs g;
    const size_t smem = item_plan(dt, s, protect, sto, &g);
    if (smem == 0) return hipErrorInvalidValue;
    g.A = (const uint8_t *)A; g.B = (const uint8_t *)B; g.C = (uint8_t *)C;
    g.lda = s.lda; g.ldb = s.ldb; g.ldc = s.ldc; g.sA = s.sA; g.sB = s.sB; g.sC = s.sC;
    g.inj_b = arm.batch; g.inj_row = arm.row; g.inj_col = arm.col; g.inj_bit = arm.bit;
    g.cached_b = cached_b ? 1 : 0;
    g.cc_obs = w.cc_obs; g.rc_obs = w.rc_obs; g.rc_pred = w.rc_pred; g.a_sum = w.a_sum; g.a_max = w.a_max;
    g.b_sum = w.b_sum; g.b_max = w.b_max; g.cc_pred = w.cc_pred; g.s_pred = w.s_pred;
    g.cc_sto = sto ? w.cc_sto : nullptr; g.rc_sto = sto ? w.rc_sto : nullptr;
    g.c_max = w.c_max;
    g.maxabs = w.maxabs; g.tau = w.tau;
    g.tau_override = v ? v->tau_override : 0.f;
    g.tau_override_cols = v ? v->tau_override_cols : 0.f;
    g.row_flag = v ? v->row_flag : nullptr; g.col_flag = v ? v->col_flag : nullptr;
    g.counts = v ? v->counts : nullptr;
    g.ticket = w.cmp_ticket; g.group_ticket = w.cmp_ticket + 4;
    return s.N <= 128 ? launch_item_rows(dt, protect, s.transB != 0, g, smem, st)
                      : launch_item_cols(dt, protect, s.transB != 0, g, smem, st);
}

}  // namespace abft
