// Kernel arguments shared by the GEMM kernels of libabft.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace abft {

// Fast path: workgroups behind the tiles that reduce A (n = nwin * nrb * batch; 0: the tiles do it).
struct BesideArgs { int n, cw_log2, nwin, nrb, rpb; };

struct GemmArgs {
    const uint8_t *A, *B;
    uint8_t *C;
    int M, N, K;
    long lda, ldb, ldc, sA, sB, sC;               // elements
    int tiles_m, tiles_n;
    uint32_t group_inv;                           // map_inverse(tiles_n)
    int n_big, tiles_m_big, tiles_m_small;        // fast path: 256-row tiles and 128-row tiles
    int n_small, batch;                           // fast path: 128-row tiles per batch item; batch items
    int inj_b, inj_row, inj_col, inj_bit;         // armed accumulator flip (inj_b < 0: none)
    const uint32_t *bias;                         // layer bias [N] (float / int32 words) or null
    // protected launches: all of these are accumulated with atomics and start at zero
    uint32_t *cc_obs, *rc_obs;                    // observed sums of C        [batch][N], [batch][M]
    double *cc_acc, *rc_acc;                      // general kernel, floating point: what its tiles add to instead
    uint32_t *rc_pred;                            // A (B e)                    [batch][M]
    uint32_t *a_sum;                              // e^T A                      [batch][K]
    uint32_t *a_max;                              // max|A| as float bits       [batch]
    uint32_t *cc_sto, *rc_sto;                    // sums of C as stored (after rounding), or null
    uint32_t *c_max;                              // max|C as stored| as float bits [batch] (with cc_sto)
    int a_given;                                  // a = e^T A and max|A| come from the caller: the pass over A's
                                                  // slabs forms the row dots only, nothing is added to a_sum / a_max
    const uint32_t *b_sum;                        // B e, complete before the launch [batch][K]
    uint32_t *counts;                             // fast kernel, protected: cleared for the check kernel
    BesideArgs beside;
};

// Workgroup -> tile inside a region of tiles_m x tiles_n tiles: consecutive ids of one XCD
// (workgroups are dealt to the 8 XCDs round-robin) walk GROUP_M tile rows, then the next column,
// so the workgroups that share an L2 work on a compact group of tiles.
// group_inv: 2^32 / (4 tiles_n) rounded down (map_inverse): a quotient by it is the true one or one less.  (Three divisions, of which a scalar unit
// has none, took 830 of the 3200 clocks before a tile's first load.)
constexpr int GROUP_M = 4;              // measured against 2, 3, 6, 8, 16: best or equal on every Linear shape
inline uint32_t map_inverse(int tiles_n) { return (uint32_t)((1ull << 32) / ((uint64_t)GROUP_M * tiles_n)); }
__device__ __forceinline__ void map_tile(int bid, int nb, int tiles_m, int tiles_n, uint32_t group_inv, int *tm, int *tn)
{
    const int q = nb >> 3, r = nb & 7, xcd = bid & 7;
    const int L = xcd * q + (xcd < r ? xcd : r) + (bid >> 3);
    const int per_group = GROUP_M * tiles_n;
    int grp = (int)__umulhi((uint32_t)L, group_inv), in_grp = L - grp * per_group;
    if (in_grp >= per_group) { ++grp; in_grp -= per_group; }
    const int first_m = grp * GROUP_M, gsz = tiles_m - first_m;
    // rows of a group: four, in the last one one to four
    const int col = gsz >= 4 ? in_grp >> 2 : gsz == 3 ? (int)__umulhi((uint32_t)in_grp, 0x55555556u) : gsz == 2 ? in_grp >> 1 : in_grp;
    *tm = first_m + in_grp - col * (gsz < GROUP_M ? gsz : GROUP_M);
    *tn = col;
}

// Fast path (gemm_fast.hip): B stored N x K, K a whole number of 128-byte slabs.
bool gemm_fast_eligible(int dt, int M, int N, int K, bool transB, long lda, long ldb);
hipError_t launch_gemm_fast(int dt, bool protect, GemmArgs &g, int batch, hipStream_t st);
void gemm_fast_tile(int *tm, int *tn);

}  // namespace abft
