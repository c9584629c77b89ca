// The streaming pass over an operand that gives its checksum vector (Sec. III-B.1 "Checksums") and
// its largest magnitude: a = e^T A and b = B e, both of length K.  One block sums a window of
// 16-byte chunk columns over a run of rows; the sums of the blocks meet in device-scope atomics.
// Used by the pass over a weight (aux_kernels.hip) and, as extra workgroups beside the tiles, by
// the general GEMM kernel (gemm_tile.hip).
#pragma once
#include "abft_device.h"

namespace abft {

constexpr int ENC_UNROLL = 8;         // independent 16-byte loads in flight per thread, beside the tiles of a GEMM
constexpr int ENC_UNROLL_ALONE = 16;  // the same for a kernel that does nothing else

struct EncPlan { int cw_log2, nwin, rpb, nrb; };

// The stored array has `rows` rows of `cols` elements.  reduce_rows = 1 (A; B stored N x K):
// sum[col] over the rows.  reduce_rows = 0 (B stored K x N): sum[row] over the columns.
struct EncArgs {
    const uint8_t *X;
    long ld, stride;      // elements
    int rows, cols, K;
    int reduce_rows;
    int cw_log2;          // 16-byte chunk columns per block window (power of two <= 64)
    int rpb;              // rows per block
    int nwin, nrb;        // windows, row blocks: nwin * nrb blocks per batch item
    uint32_t *sum;        // [batch][K]  accumulated with atomics: zero before the launch
    uint32_t *max_acc;    // [batch]     largest magnitude as float bits, atomic max: zero before the launch
};

// Window of a streaming pass over a rows x cols array: 8..64 chunk columns, least padding, then widest.
// The rows of a block are the caller's choice.
inline EncPlan plan_window(int rows, int cols, int chunk_elems)
{
    EncPlan p;
    const int chunks = (cols + chunk_elems - 1) / chunk_elems;
    int best_lg = 3;
    long best_waste = -1;
    for (int lg = 3; lg <= 6; ++lg) {
        const int CW = 1 << lg;
        const long waste = (long)((chunks + CW - 1) / CW) * CW - chunks;
        if (best_waste < 0 || waste <= best_waste) { best_waste = waste; best_lg = lg; }
    }
    p.cw_log2 = best_lg;
    p.nwin = (chunks + (1 << best_lg) - 1) >> best_lg;
    p.rpb = rows;
    p.nrb = 1;
    return p;
}

// For a kernel that does nothing else: one batch of ENC_UNROLL_ALONE loads per thread, more when the
// matrix is tall (more than 640 blocks): atomics that hit one cache line are served one after the
// other, so fewer row blocks mean less waiting at the end of the pass.
inline EncPlan plan_alone(int rows, int cols, int chunk_elems)
{
    EncPlan p = plan_window(rows, cols, chunk_elems);
    long rpb = (256L >> p.cw_log2) * ENC_UNROLL_ALONE;
    while (rpb < rows && (long)p.nwin * ((rows + rpb - 1) / rpb) > 640) rpb *= 2;
    p.rpb = (int)rpb;
    p.nrb = (int)((rows + rpb - 1) / rpb);
    return p;
}

// Block `blk` (of nwin * nrb) of batch item bz.  red: 256 * (16 / element size) + 4 words of LDS.
// UNROLL: independent 16-byte loads in flight per thread.
template <int DT, int UNROLL, bool REDUCE_ROWS>
__device__ __forceinline__ void encode_block_dir(const EncArgs &e, int blk, int bz, uint32_t *red_words)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int ES = T::ES, CE = 16 / ES;
    acc_t *red = reinterpret_cast<acc_t *>(red_words);
    const int tid = threadIdx.x;
    const int win = blk % e.nwin, rb = blk / e.nwin;
    const int CW = 1 << e.cw_log2, RL = 256 >> e.cw_log2;
    const int cx = tid & (CW - 1), ry = tid >> e.cw_log2;
    const int col0 = (win * CW + cx) * CE;
    const bool colok = col0 < e.cols;
    const int nvalid = e.cols - col0;                        // elements of this chunk inside the row
    const uint8_t *Xb = e.X + (long)bz * e.stride * ES;
    const int rbeg = rb * e.rpb;
    const int rend = min(rbeg + e.rpb, e.rows);
    const int iters = (rend - rbeg + RL * UNROLL - 1) / (RL * UNROLL);

    acc_t colacc[CE];
#pragma unroll
    for (int q = 0; q < CE; ++q) colacc[q] = T::zero();
    float mx = 0.f;

    for (int it = 0; it < iters; ++it) {
        // a batch of independent loads first: the pass is bound by memory latency otherwise
        i32x4 v[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int r = rbeg + ry + (it * UNROLL + u) * RL;
            v[u] = i32x4{0, 0, 0, 0};
            if (colok && r < rend) v[u] = *reinterpret_cast<const i32x4 *>(Xb + ((long)r * e.ld + col0) * ES);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int r = rbeg + ry + (it * UNROLL + u) * RL;
            i32x4 w = v[u];
            if (nvalid < CE) w = mask_chunk(w, nvalid > 0 ? nvalid * ES : 0);
            acc_t s = T::zero();
#pragma unroll
            for (int q = 0; q < CE; ++q) {
                acc_t x = T::elem(w, q);
                if (!T::IS_INT) mx = fmaxf(mx, fabsf((float)x));
                if constexpr (REDUCE_ROWS) colacc[q] = add_t(colacc[q], x);
                else s = add_t(s, x);
            }
            if constexpr (!REDUCE_ROWS) {
                s = seg_sum(s, CW);
                if (cx == 0 && r < rend) atomic_add_word(e.sum + (long)bz * e.K + r, s);
            }
        }
    }
    // One atomic on max|X| per block, not per wave: they all hit one word, which serves them one after the other.
    float *mx4 = reinterpret_cast<float *>(red_words + 256 * CE);
    if (!T::IS_INT) {
        mx = wave_max(mx);
        if ((tid & 63) == 0) mx4[tid >> 6] = mx;
        if constexpr (!REDUCE_ROWS) __syncthreads();
    }
    if constexpr (REDUCE_ROWS) {
#pragma unroll
        for (int q = 0; q < CE; ++q) red[(ry * CW + cx) * CE + q] = colacc[q];
        __syncthreads();
        // one atomic per column, consecutive lanes on consecutive addresses
        for (int c = tid; c < CW * CE; c += 256) {
            const int col = win * CW * CE + c;
            if (col < e.cols) {
                acc_t t = red[c];
                for (int y = 1; y < RL; ++y) t = add_t(t, red[y * CW * CE + c]);
                atomic_add_word(e.sum + (long)bz * e.K + col, t);
            }
        }
    }
    if (!T::IS_INT && tid == 0) {
        mx = fmaxf(fmaxf(mx4[0], mx4[1]), fmaxf(mx4[2], mx4[3]));
        if (mx > 0.f) atomicMax(e.max_acc + bz, __float_as_uint(mx));
    }
}

template <int DT, int UNROLL>
__device__ __forceinline__ void encode_block(const EncArgs &e, int blk, int bz, uint32_t *red_words)
{
    if (e.reduce_rows) encode_block_dir<DT, UNROLL, true>(e, blk, bz, red_words);
    else encode_block_dir<DT, UNROLL, false>(e, blk, bz, red_words);
}

}  // namespace abft
