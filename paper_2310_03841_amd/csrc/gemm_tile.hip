// Protected GEMM for gfx950, every shape the other two GEMM kernels do not take: problems of a few
// tiles, ragged K, B stored K x N.  C = A B with the observed row and column sums of C taken from
// the accumulators on their way out (epilogue fusion: Sec. IV-C memory paragraph, Sec. V
// "Optimizations" (2)).
//
// What bounds these problems is not arithmetic or bandwidth but the chain of latencies of a call.
// A call of few tiles is therefore one launch (predict_pass.h): workgroups beside the tiles form both predictions, and who
// is last compares.  Call after call, in us, two launches / one (both with the epilogue and the start of before; one now: int8 197 x 768 x 768
// 7.2, bf16 197 x 768 x 3072 14.4): int8 197 x 768 x 768 8.7 / 7.5, 3000 x 128 x 1024 14.2 / 9.3, bf16
// 197 x 768 x 3072 16.4 / 15.4, 64 x 500 x 3072 with B stored K x N 25.1 / 18.9.  (A call takes 3 us before its first and after its
// last workgroup; a second kernel adds that gap, a trip to memory and a reduction.)
// More tiles, or predictions that would take longer than they: the input-side vectors a = e^T A and b = B e, which depend
// on nothing, are formed by extra workgroups of the same launch, beside the tiles; both predictions wait for the check
// kernel behind it (check_kernel, aux_kernels.hip).  Large protected problems: a pass over B
// first and A reduced from the slabs in LDS (fuses_a below).
//
// Tile: BM x BN by four waves of (BM/2) x (BN/2), 32 x 32 MFMA blocks.  K advances in slabs of 128
// bytes per row of A.  Slabs go from global memory straight into LDS (global_load_lds_dwordx4),
// NS buffers deep, so NS - 1 slabs are in flight while one is multiplied; one barrier per slab.
// The fragments of slab s are read while the MFMAs of slab s - 1 run (two register sets).  A slab of a 64 x 64 tile takes some 490 clocks, alone on a compute
// unit; eight buffers instead of four do not change that (fc2 of one image 14.35 -> 14.7 us, 197 x 3072 x 768 10.6 -> 11.0), and loads dealt out between the MFMAs,
// as the fast kernel has them, come too late (14.3 -> 17.0, 10.4 -> 11.0).
//
// LDS: rows of 128 bytes as eight 16-byte chunks, chunk c of row r in slot c ^ ((r >> 1) & 7)
// (sixteen consecutive rows of a fragment read then fall on sixteen different 16-byte bank groups).
// B stored K x N keeps its own orientation in LDS and is transposed on the way to the matrix cores by
// the LDS transpose reads of gfx950 (ds_read_b64_tr_b16 / _b8: sixteen lanes fetch 4 x 16 (8 x 16)
// elements as rows of k and receive columns); its swizzle puts the rows of one such read on
// different banks.  Direct loads land where the lane order says, so every swizzle is applied by
// choosing which global chunk a lane fetches.
//
// Edges: rows and columns past the problem fetch the last valid ones; what they produce is never
// stored or summed.  Past the end of K the fragments of the last slab are cleared in registers.
#include <algorithm>

#include "abft_device.h"
#include "block_out.h"
#include "encode_pass.h"
#include "gemm_apass.h"
#include "gemm_args.h"
#include "gemm_epilogue.h"
#include "predict_pass.h"

namespace abft {

typedef const __attribute__((address_space(1))) void *tile_gas_ptr;
typedef __attribute__((address_space(3))) void *tile_las_ptr;

struct TileArgs {
    GemmArgs g;
    int n_extra;                  // workgroups [0, n_extra) of a batch item: n_enc_a of the pass over A, n_enc_b of the
    int n_enc_a, n_enc_b;         // pass over B, and with a bias one for its sum
    int n_tiles;                  // the workgroups behind them take tiles
    EncArgs ea, eb;
    uint32_t *counts;             // protected: cleared here, completed by the check kernel
    uint32_t *bias_sum;           // protected, with a bias: its sum, formed by one more workgroup
    int aux_off;                  // APASS: where the words of b and of a begin in LDS; ONE: the words of the predictions
    int bias_off;                 // with a bias: where that of a tile's columns lies in LDS, behind all else
};
// What the host fills in.
struct HostArgs : TileArgs {
    PredArgs p;
    int fuse_bm;                  // rows of a tile of the instantiations with APASS, 0: the others
};
// ONE alone takes the arguments of the predictions, and none of the passes beside the tiles: what a launch copies, every call pays for, and
// each line of 64 bytes costs the start of a kernel some 100 clocks.
struct OneArgs {
    GemmArgs g;
    int n_extra, n_tiles, aux_off, bias_off;
    PredArgs p;
};
// Unprotected tiles take none of the passes' either, and ask for the lines ahead of what only protected ones read: three of eight.
struct PlainArgs {
    int n_tiles, bias_off;
    GemmArgs g;
};
template <bool PROT, bool ONE> struct KernelArgs { typedef TileArgs type; };
template <> struct KernelArgs<true, true> { typedef OneArgs type; };
template <> struct KernelArgs<false, false> { typedef PlainArgs type; };
constexpr int PLAIN_ARGS_READ = offsetof(PlainArgs, g) + offsetof(GemmArgs, cc_obs);

// The sums of a tile's rows and columns by wave column and wave row, of the accumulators and of the stored values, and eight words of maxima.
constexpr int tile_epi_bytes(int BM, int BN) { return 4 * (BM + BN) * 4 + 8 * 4; }

// ns: buffers in use, min(NS, slabs of the problem)
__host__ __device__ constexpr int tile_lds_bytes(int BM, int BN, int ns)
{
    const int loop = ns * (BM + BN) * SLAB_BYTES, epi = tile_epi_bytes(BM, BN);
    return loop > epi ? loop : epi;
}

// Swizzle of B stored K x N: 16-byte slot of a row of k <-> chunk of columns.  ROWB: bytes per row.
template <int ES, int ROWB> __device__ __forceinline__ int kn_swizzle(int k)
{
    if constexpr (ES == 2) return ROWB == 128 ? ((k >> 1) & 1) << 2 : (k & 3) << 2;      // 32-byte pieces of 4 rows
    else return ROWB == 64 ? ((k >> 2) & 1) << 1 : ((k >> 1) & 3) << 1;                  // 16-byte pieces of 8 rows
}

// ONE: the whole protected call (predict_pass.h)
template <int DT, int BM, int BN, int NS, bool PROT, bool TRANSB, bool APASS, bool ONE>
__global__ __launch_bounds__(256) void gemm_tile_kernel(typename KernelArgs<PROT, ONE>::type whole)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    typedef typename T::accv_t accv_t;
    constexpr int ES = T::ES, OS = T::OS;
    constexpr int KE = SLAB_BYTES / ES;                          // elements of K per slab
    constexpr int TM = BM / 2, TN = BN / 2, MI = TM / 32, NI = TN / 32;
    constexpr int BUF = (BM + BN) * SLAB_BYTES;
    constexpr int GA = BM / 32, GB = BN / 32;                    // load instructions per wave and slab (8 LDS rows of 128 bytes each)
    constexpr int BROWB = BN * ES;                               // bytes of a row of k (B stored K x N)
    static_assert((NS - 2) * (GA + GB) < 64, "the wait count is an immediate");

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    typedef typename KernelArgs<PROT, ONE>::type Args;
    fetch_args<Args, PROT ? (int)sizeof(Args) : PLAIN_ARGS_READ>();
    // ONE: each argument where it is used (a few of those that the call's end needs and all of the tiles' do not fit the scalar registers; and, from the
    // parameter, the compiler asks for some twenty of them ahead of the line above: int8 873 x 249 x 128 7.5 us, 6.9 so).  The others have scalars
    // enough: 197 x 3072 x 768 and its check 10.5 us, 11.0 with each where it is used.
    const Args &a = ONE ? kernel_args<Args>() : whole;
    const GemmArgs &g = a.g;
    const int bz = blockIdx.y;
    if constexpr (ONE) {
        const size_t first = (size_t)bz * a.p.wgs + blockIdx.x, nw = (size_t)a.p.wgs * a.p.batch;
        for (size_t i = first * 256 + threadIdx.x; i < a.p.zero_words; i += nw * 256) a.p.zero_ptr[i] = 0u;
        for (size_t i = first * 256 + threadIdx.x; i < a.p.zero2_words; i += nw * 256) a.p.zero2_ptr[i] = 0u;
        if ((int)blockIdx.x < a.n_extra) {
            predict_block<DT, TRANSB>(a.p, blockIdx.x, bz, smem, a.aux_off);
            end_predict<DT>(a.p, blockIdx.x, a.n_extra, bz, reinterpret_cast<uint32_t *>(smem));
            return;
        }
    } else if constexpr (PROT) {
        if (blockIdx.x == 0 && bz == 0 && threadIdx.x < 5) a.counts[threadIdx.x] = 0u;
        const int e = blockIdx.x;
        if (e < a.n_extra) {
            if (e == a.n_enc_a + a.n_enc_b) {
                const acc_t t = block_bias_sum<acc_t>(g.bias, g.N, reinterpret_cast<acc_t *>(smem));
                if (threadIdx.x == 0 && bz == 0) *a.bias_sum = as_word(t);
            } else if (e < a.n_enc_a) encode_block<DT, ENC_UNROLL>(a.ea, e, bz, reinterpret_cast<uint32_t *>(smem));
            else encode_block<DT, ENC_UNROLL>(a.eb, e - a.n_enc_a, bz, reinterpret_cast<uint32_t *>(smem));
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;
    int tm, tn;
    int bid = blockIdx.x;
    if constexpr (PROT) bid -= a.n_extra;
    map_tile(bid, a.n_tiles, g.tiles_m, g.tiles_n, g.group_inv, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int M = g.M, N = g.N, K = g.K;
    const int nslab = (K + KE - 1) / KE;
    const int nch = (K * ES + 15) / 16;                          // 16-byte chunks of a row along K that hold data

    const uint8_t *Ab = g.A + (long)bz * g.sA * ES;
    const uint8_t *Bb = g.B + (long)bz * g.sB * ES;

    // ---- sources of the direct loads.  K-contiguous operand: group p of this wave fills LDS rows
    // (4 p + wave) * 8 .. + 8, lane l row l >> 3, slot l & 7.
    const int lrow = lane >> 3;
    const int lchunk = (lane & 7) ^ (((wave & 1) << 2) + (lrow >> 1));
    const uint8_t *arow[GA], *brow[GB];
    int bk[GB], bcb[GB];                                         // B stored K x N: row of k inside the slab, byte offset of the chunk
#pragma unroll
    for (int p = 0; p < GA; ++p) {
        int r = m0 + (4 * p + wave) * 8 + lrow;
        r = r < M ? r : M - 1;
        arow[p] = Ab + (long)r * g.lda * ES;
    }
#pragma unroll
    for (int p = 0; p < GB; ++p) {
        if (TRANSB) {
            int r = n0 + (4 * p + wave) * 8 + lrow;
            r = r < N ? r : N - 1;
            brow[p] = Bb + (long)r * g.ldb * ES;
            bk[p] = bcb[p] = 0;
        } else {
            constexpr int LPR = BROWB / 16, RPG = 64 / LPR;      // lanes per row of k, rows per load instruction
            bk[p] = (4 * p + wave) * RPG + lane / LPR;
            int cb = n0 * ES + (((lane % LPR) ^ kn_swizzle<ES, BROWB>(bk[p])) * 16);
            const int last = ((N - 1) * ES) / 16 * 16;           // last chunk that holds a column
            bcb[p] = cb < last ? cb : last;
            brow[p] = Bb;
        }
    }
    auto issue = [&](int s) __attribute__((always_inline)) {
        uint8_t *dA = smem + (s % NS) * BUF;
        uint8_t *dB = dA + BM * SLAB_BYTES;
        int ch = s * 8 + lchunk;
        ch = ch < nch ? ch : nch - 1;                            // past the end of K: any valid chunk (cleared in registers)
#pragma unroll
        for (int p = 0; p < GA; ++p)
            __builtin_amdgcn_global_load_lds((tile_gas_ptr)(arow[p] + (long)ch * 16),
                                             (tile_las_ptr)(dA + (4 * p + wave) * 8 * SLAB_BYTES), 16, 0, 0);
#pragma unroll
        for (int p = 0; p < GB; ++p) {
            const uint8_t *src;
            if (TRANSB) {
                src = brow[p] + (long)ch * 16;
            } else {
                int k = s * KE + bk[p];
                k = k < K ? k : K - 1;
                src = brow[p] + (long)k * g.ldb * ES + bcb[p];
            }
            __builtin_amdgcn_global_load_lds((tile_gas_ptr)src, (tile_las_ptr)(dB + (4 * p + wave) * 8 * SLAB_BYTES), 16, 0, 0);
        }
    };

    typedef int i32x2 __attribute__((ext_vector_type(2)));
    i32x4 fa[2][4][MI], fb[2][4][NI];
    auto read_frags = [&](int s, auto set_c) __attribute__((always_inline)) {
        constexpr int set = decltype(set_c)::value;
        const uint8_t *sA = smem + (s % NS) * BUF;
        const uint8_t *sB = sA + BM * SLAB_BYTES;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const int sw = ((2 * s4 + lh) ^ ((lane >> 1) & 7)) * 16;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                fa[set][s4][mi] = *reinterpret_cast<const i32x4 *>(sA + (wm * TM + mi * 32 + l32) * SLAB_BYTES + sw);
            if constexpr (TRANSB) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    fb[set][s4][ni] = *reinterpret_cast<const i32x4 *>(sB + (wn * TN + ni * 32 + l32) * SLAB_BYTES + sw);
            }
        }
        if constexpr (!TRANSB) {
            // Sixteen lanes read 4 (8) rows of k of sixteen columns; each gets one column.  A step of
            // 32 bytes of k per lane is two such reads; the four steps of a slab and the halves of a
            // step lie at fixed distances (the swizzle does not change over them).  Written as
            // instructions: in front of the built-in the compiler waits for every outstanding load
            // (800 x 700 x 4096: bf16 36.9 us with the built-in, 19.5 us so).
            constexpr int HALF = (ES == 2 ? 4 : 8) * BROWB, STEP = (ES == 2 ? 16 : 32) * BROWB;
            const int i16 = lane & 15;
            const int kk = ES == 2 ? 8 * lh + (i16 >> 2) : 16 * lh + (i16 >> 1);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int cb = (wn * TN + ni * 32 + 16 * ((lane >> 4) & 1)) * ES + (ES == 2 ? (i16 & 3) : (i16 & 1)) * 8;
                const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint8_t *)(
                    sB + kk * BROWB + (((cb >> 4) ^ kn_swizzle<ES, BROWB>(kk)) * 16) + (cb & 15));
                i32x2 h[8];
#define TILE_TR(T) \
                asm volatile(T " %0, %8\n\t" T " %1, %8 offset:%9\n\t" T " %2, %8 offset:%10\n\t" T " %3, %8 offset:%11\n\t" \
                             T " %4, %8 offset:%12\n\t" T " %5, %8 offset:%13\n\t" T " %6, %8 offset:%14\n\t" T " %7, %8 offset:%15\n\t" \
                             "s_waitcnt lgkmcnt(0)" \
                             : "=&v"(h[0]), "=&v"(h[1]), "=&v"(h[2]), "=&v"(h[3]), "=&v"(h[4]), "=&v"(h[5]), "=&v"(h[6]), "=&v"(h[7]) \
                             : "v"(at), "n"(HALF), "n"(STEP), "n"(STEP + HALF), "n"(2 * STEP), "n"(2 * STEP + HALF), "n"(3 * STEP), \
                               "n"(3 * STEP + HALF) : "memory")
                if constexpr (ES == 2) TILE_TR("ds_read_b64_tr_b16");
                else TILE_TR("ds_read_b64_tr_b8");
#undef TILE_TR
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4)
                    fb[set][s4][ni] = i32x4{h[2 * s4][0], h[2 * s4][1], h[2 * s4 + 1][0], h[2 * s4 + 1][1]};
            }
        }
    };
    auto clear_tail = [&](auto set_c) __attribute__((always_inline)) {
        constexpr int set = decltype(set_c)::value;
        const int base = K * ES - (nslab - 1) * SLAB_BYTES;      // bytes of K in the last slab
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const int keep = base - (2 * s4 + lh) * 16;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) fa[set][s4][mi] = mask_chunk(fa[set][s4][mi], keep);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) fb[set][s4][ni] = mask_chunk(fb[set][s4][ni], keep);
        }
    };
    accv_t acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = T::zero();
    auto mfmas = [&](auto set_c) __attribute__((always_inline)) {
        constexpr int set = decltype(set_c)::value;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] = T::mfma(fb[set][s4][ni], fa[set][s4][mi], acc[mi][ni]);
    };
    typedef std::integral_constant<int, 0> set0;
    typedef std::integral_constant<int, 1> set1;

    // ---- main loop.  Slab s is in place behind "at most the slabs issued after it outstanding"
    // (a wave's loads complete in order) and the barrier; the same barrier says that every wave has
    // its fragments of slab s - 1 in registers, so that buffer takes slab s + NS - 1.
    // APASS: of the tiles that share rows of A, the one in column s mod tiles_n reduces slab s while it is resident
    // (gemm_apass.h).  Its words of b go straight into LDS ahead of the slabs.
    const int owned = (APASS && tn < nslab) ? (nslab - tn + g.tiles_n - 1) / g.tiles_n : 0;
    int aux_off = 0;
    if constexpr (APASS) aux_off = a.aux_off;
    uint32_t *b_lds = reinterpret_cast<uint32_t *>(smem + aux_off), *col_lds = b_lds + owned * KE;
    APassState<DT> ast;
    ast.rdot = T::zero(); ast.amax = 0.f;
    int next_own = tn, own_at = 0;
    if constexpr (APASS) {
        for (int j = wave; j < owned; j += 4)
#pragma unroll
            for (int h = 0; h < KE / 64; ++h) {
                int k = (tn + j * g.tiles_n) * KE + 64 * h + lane;
                k = k < K ? k : K - 1;                           // past the end of K: times zero
                __builtin_amdgcn_global_load_lds((tile_gas_ptr)(g.b_sum + (long)bz * K + k),
                                                 (tile_las_ptr)(b_lds + j * KE + 64 * h), 4, 0, 0);
            }
        for (int i = tid; i < owned * KE; i += 256) col_lds[i] = 0u;
    }
    // the bias of the tile's columns (past the end of N the last one's), straight into LDS of its own, ahead of the slabs: a wait for a slab is
    // one for everything before it
    const uint32_t *bias_lds = reinterpret_cast<const uint32_t *>(smem + a.bias_off);
    if (g.bias && wave < BN / 64) {
        const int gc = n0 + 64 * wave + lane;
        __builtin_amdgcn_global_load_lds((tile_gas_ptr)(g.bias + (gc < N ? gc : N - 1)), (tile_las_ptr)(smem + a.bias_off + 256 * wave), 4, 0, 0);
    }
    for (int s = 0; s < NS - 1; ++s)
        if (s < nslab) issue(s);
    auto arrive = [&](int s) __attribute__((always_inline)) {
        const int ahead = nslab - 1 - s;                         // slabs issued after s: min(ahead, NS - 2)
        constexpr int L = GA + GB;
        if (ahead >= NS - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((NS - 2) * L) : "memory");
        else if (NS > 3 && ahead == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(L) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (s + NS - 1 < nslab) issue(s + NS - 1);
    };
    auto reduce = [&](int s) __attribute__((always_inline)) {
        if constexpr (APASS) {
            if (s != next_own) return;
            const uint8_t *sA = smem + (s % NS) * BUF;
            if (g.a_given)
                a_pass<DT, BM, true>(sA, b_lds + own_at, M - m0, col_lds + own_at, ast, K * ES - s * SLAB_BYTES);
            else
                a_pass<DT, BM, false>(sA, b_lds + own_at, M - m0, col_lds + own_at, ast, K * ES - s * SLAB_BYTES);
            next_own += g.tiles_n;
            own_at += KE;
        }
    };
    const bool ragged = (K * ES) % SLAB_BYTES != 0;
    arrive(0);
    read_frags(0, set0{});
    reduce(0);
    int s = 1;
    for (; s + 1 < nslab; s += 2) {
        arrive(s);
        read_frags(s, set1{});
        mfmas(set0{});
        reduce(s);
        arrive(s + 1);
        read_frags(s + 1, set0{});
        mfmas(set1{});
        reduce(s + 1);
    }
    if (s < nslab) {
        arrive(s);
        read_frags(s, set1{});
        mfmas(set0{});
        reduce(s);
        if (ragged) clear_tail(set1{});
        mfmas(set1{});
    } else {
        if (ragged) clear_tail(set0{});
        mfmas(set0{});
    }

    // ---- epilogue, from the registers (block_out.h): lane l holds row l & 31 of a block and in register i column
    // 8 (i >> 2) + 4 (l >> 5) + (i & 3).  Row sums are in-lane adds, column sums fold lanes and values together, C leaves as segments of 64 bytes of
    // sixteen rows (int32: 128 of eight).  (Each block through a stage in LDS, and from there four columns of four rows to a lane: 3200 of the 13700
    // clocks of a bf16 197 x 3072 x 768.)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // every wave is done with the operand buffers
    if constexpr (APASS) {
        if (!g.a_given) {
            for (int i = tid; i < owned * KE; i += 256) {
                const int k = (tn + i / KE * g.tiles_n) * KE + i % KE;
                if (k < K) atomic_add_word(g.a_sum + (long)bz * K + k, from_word<acc_t>(col_lds[i]));
            }
        }
        const int r = m0 + (tid >> 3) + 32 * (tid & 7);
        if (owned && (tid & 7) < BM / 32 && r < M) atomic_add_word(g.rc_pred + (long)bz * M + r, ast.rdot);
    }
    acc_t *rs_part = reinterpret_cast<acc_t *>(smem);                                // [2][BM] by wave column
    acc_t *cs_part = rs_part + 2 * BM;                                               // [2][BN] by wave row
    float *rs_sto = reinterpret_cast<float *>(cs_part + 2 * BN);                     // the same of the values as stored
    float *cs_sto = rs_sto + 2 * BM;
    float *max_part = cs_sto + 2 * BN;                                               // max|C as stored| by wave, max|A|
    const bool sto = PROT && !T::IS_INT && g.cc_sto != nullptr;
    const bool inj_here = g.inj_b == bz && g.inj_row >= m0 && g.inj_row < m0 + BM && g.inj_col >= n0 && g.inj_col < n0 + BN;
    const bool inside = m0 + BM <= M && n0 + BN <= N;
    float cmax_s = 0.f;
    constexpr bool QUADS = T::IS_INT && !PROT;
    constexpr int NP = out_passes<DT>(), RPP = out_step<DT, QUADS>();    // passes of a block's stores, rows from one to the next
    // this lane's 16 bytes of pass 0 of the wave's first block
    const int orow = m0 + wm * TM + out_row<DT, QUADS>(lane), ocol = n0 + wn * TN + out_col<DT, QUADS>(lane);
    uint8_t *const dst0 = g.C + ((long)bz * g.sC + (long)orow * g.ldc + ocol) * OS;
    const long pass_bytes = (long)RPP * g.ldc * OS;
    // what is left of a lane's 16 bytes at the right edge is the same for all lanes there
    const int left = (N * OS) & 15;
    acc_t cs[NI][16];
    float cs_s[NI][16];
    if (PROT) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) { cs[ni][i] = T::zero(); cs_s[ni][i] = 0.f; }
    }
    static_for<0, MI>([&](auto mi_c) {
        constexpr int mi = decltype(mi_c)::value;
        const int row = m0 + wm * TM + mi * 32 + l32;
        acc_t rsum = T::zero();
        float rsum_s = 0.f;
        static_for<0, NI>([&](auto ni_c) {
            constexpr int ni = decltype(ni_c)::value;
            const int c0 = n0 + wn * TN + ni * 32;
            acc_t v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = acc[mi][ni][i];
            if (inj_here && row == g.inj_row) {
                // the armed flip: one bit of one accumulator, before rounding and before the sums
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (c0 + 8 * (i >> 2) + 4 * lh + (i & 3) == g.inj_col) v[i] = from_word<acc_t>(as_word(v[i]) ^ (1u << g.inj_bit));
            }
            if (g.bias) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const i32x4 b4 = *reinterpret_cast<const i32x4 *>(bias_lds + wn * TN + ni * 32 + 8 * q + 4 * lh);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * q + e] = add_t(v[4 * q + e], from_word<acc_t>((uint32_t)b4[e]));
                }
            }
            if (PROT && !inside) {
                // past the edges: values of the last row and column again, in no sum
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = row < M && c0 + 8 * (i >> 2) + 4 * lh + (i & 3) < N ? v[i] : T::zero();
            }
            if (PROT) {
#pragma unroll
                for (int i = 0; i < 16; ++i) cs[ni][i] = add_t(cs[ni][i], v[i]);
                rsum = add_t(rsum, sum16<acc_t>(v));
            }
            i32x4 out[NP];
            if constexpr (T::IS_INT) {
                uint32_t w[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) w[i] = (uint32_t)v[i];
                if constexpr (QUADS) turn_quads(w, out, lane);
                else turn_block<DT>(w, out);
            } else {
                uint32_t w[8];
                pack_block<DT>(v, w);
                if (sto) {
                    float sv[16];
#pragma unroll
                    for (int j = 0; j < 8; ++j) { sv[2 * j] = unpack_lo<DT>(w[j]); sv[2 * j + 1] = unpack_hi<DT>(w[j]); }
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        cs_s[ni][i] += sv[i];
                        cmax_s = fmaxf(cmax_s, fabsf(sv[i]));
                    }
                    rsum_s += sum16<float>(sv);
                }
                turn_block<DT>(w, out);
            }
            uint8_t *dst = dst0 + (long)(mi * 32) * g.ldc * OS + ni * 32 * OS;
            if (inside) {
#pragma unroll
                for (int p = 0; p < NP; ++p) *reinterpret_cast<i32x4 *>(dst + p * pass_bytes) = out[p];
            } else {
                const int gc = ocol + ni * 32, rows = M - (orow + mi * 32);      // valid rows from this lane's first on
                if (gc + 16 / OS <= N) {
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        if (p * RPP < rows) *reinterpret_cast<i32x4 *>(dst + p * pass_bytes) = out[p];
                } else if (gc < N) {
                    // in falling powers of two, all passes of a size together: few branches
                    if (left & 8) {
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            if (p * RPP < rows) *reinterpret_cast<i32x2 *>(dst + p * pass_bytes) = i32x2{out[p][0], out[p][1]};
                    }
                    if (left & 4) {
                        const int at = left & 8;
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            if (p * RPP < rows) *reinterpret_cast<int *>(dst + p * pass_bytes + at) = at ? out[p][2] : out[p][0];
                    }
                    if (left & 2) {
                        const int at = left & 12;
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            if (p * RPP < rows)
                                *reinterpret_cast<uint16_t *>(dst + p * pass_bytes + at) =
                                    (uint16_t)(at & 8 ? (at & 4 ? out[p][3] : out[p][2]) : (at & 4 ? out[p][1] : out[p][0]));
                    }
                }
            }
        });
        if (PROT) {
            const acc_t r = add_xor32(rsum);
            if (lane < 32) rs_part[wn * BM + wm * TM + mi * 32 + lane] = r;
            if constexpr (!T::IS_INT) {
                if (sto) {
                    const float rs = add_xor32(rsum_s);
                    if (lane < 32) rs_sto[wn * BM + wm * TM + mi * 32 + lane] = rs;
                }
            }
        }
    });
    if (PROT) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const acc_t t = fold16<acc_t>(cs[ni], lane);
            if ((lane & 1) == 0) cs_part[wm * BN + wn * TN + ni * 32 + fold16_column(lane)] = t;
            if constexpr (!T::IS_INT) {
                if (sto) {
                    const float ts = fold16<float>(cs_s[ni], lane);
                    if ((lane & 1) == 0) cs_sto[wm * BN + wn * TN + ni * 32 + fold16_column(lane)] = ts;
                }
            }
        }
        if constexpr (!T::IS_INT) {
            if (sto) {
                cmax_s = wave_max(cmax_s);
                if (lane == 0) max_part[wave] = cmax_s;
            }
            if (APASS && !g.a_given) {
                const float m = wave_max(ast.amax);
                if (lane == 0) max_part[4 + wave] = m;
            }
        }
        // over LDS traffic only: a full barrier would also wait for every store of C
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        for (int t = tid; t < BM + BN; t += 256) {
            const bool isrow = t < BM;
            const int q = isrow ? t : t - BM, gi = (isrow ? m0 : n0) + q, len = isrow ? M : N;
            if (gi < len) {
                const acc_t *src = isrow ? rs_part + q : cs_part + q;
                const long o = (long)bz * len + gi;
                const acc_t sum = add_t(src[0], src[isrow ? BM : BN]);
                if constexpr (T::IS_INT) {
                    atomic_add_word((isrow ? g.rc_obs : g.cc_obs) + o, sum);
                } else {
                    // in doubles: small tiles are many, and the order of their additions must not show
                    unsafeAtomicAdd((isrow ? g.rc_acc : g.cc_acc) + o, (double)sum);
                    if (sto) {
                        const float *ss = isrow ? rs_sto + q : cs_sto + q;
                        unsafeAtomicAdd(reinterpret_cast<float *>(isrow ? g.rc_sto : g.cc_sto) + o, ss[0] + ss[isrow ? BM : BN]);
                    }
                }
            }
        }
        if constexpr (!T::IS_INT) {
            // The largest magnitudes: of C as stored (what a consumer of this C needs as its max|A|), of A.  One
            // atomic per workgroup: on one word they are served one after the other (bf16 3819 x 1465 x 1161 with the
            // stored sums, one per wave: 55.7 us, 38.0 so, 37.0 without the sums)
            auto publish = [&](uint32_t *word, int at) __attribute__((always_inline)) {
                float m = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) m = fmaxf(m, max_part[at + w]);
                if (m > 0.f) atomicMax(word + bz, __float_as_uint(m));
            };
            if (sto && tid == 0) publish(g.c_max, 0);
            if (APASS && !g.a_given && tid == 64) publish(g.a_max, 4);
        }
    }
    if constexpr (ONE) end_tile<DT, BM, BN>(a.p, tm, tn, bz, reinterpret_cast<uint32_t *>(smem));
}

// ------------------------------------------------------------------------------------------
static int slabs_of(int dt, int K) { return (int)(((long)K * elem_size(dt) + SLAB_BYTES - 1) / SLAB_BYTES); }

template <int DT, int BM, int BN, int NS, bool PROT, bool TRANSB, bool APASS = false, bool ONE = false>
static hipError_t launch_one(HostArgs &a, int batch, hipStream_t st)
{
    constexpr int smem_max = APASS || ONE ? 160 * 1024 : tile_lds_bytes(BM, BN, NS) + BN * 4;
    static_assert(tile_lds_bytes(BM, BN, 1) >= 256 * 16 * 4, "the passes over A and B use 16 KB");
    auto kern = gemm_tile_kernel<DT, BM, BN, NS, PROT, TRANSB, APASS, ONE>;
    if (smem_max > 48 * 1024) {
        hipError_t e = ensure_max_lds(reinterpret_cast<const void *>(kern), smem_max);
        if (e != hipSuccess) return e;
    }
    // a problem of fewer slabs than buffers leaves the rest of the LDS to further workgroups
    const int nslab = slabs_of(DT, a.g.K);
    int smem = tile_lds_bytes(BM, BN, nslab < NS ? nslab : NS);
    a.aux_off = smem;
    if (APASS) smem += (int)apass_lds_bytes(DT, nslab, a.g.tiles_n);
    if (ONE) {
        const int pieces = (a.p.a_steps + a.p.b_steps) * PRED_STEP_BYTES;
        a.aux_off = pieces > 256 * 16 * 4 ? pieces : 256 * 16 * 4;
        smem = std::max(smem, a.aux_off + PRED_VEC_WORDS * 4);
        a.p.wgs = a.n_extra + a.n_tiles;
        a.p.tiles_m = a.g.tiles_m; a.p.tiles_n = a.g.tiles_n; a.p.bm = BM; a.p.bn = BN;
    }
    a.bias_off = smem = (smem + 15) & ~15;
    if (a.g.bias) smem += BN * 4;
    dim3 grid((unsigned)(a.n_extra + a.n_tiles), (unsigned)batch, 1);
    if constexpr (ONE) {
        const OneArgs k = {a.g, a.n_extra, a.n_tiles, a.aux_off, a.bias_off, a.p};
        hipLaunchKernelGGL(kern, grid, dim3(256), smem, st, k);
    } else if constexpr (PROT) {
        hipLaunchKernelGGL(kern, grid, dim3(256), smem, st, (const TileArgs &)a);
    } else {
        const PlainArgs k = {a.n_tiles, a.bias_off, a.g};
        hipLaunchKernelGGL(kern, grid, dim3(256), smem, st, k);
    }
    return hipGetLastError();
}

static long tiles_of(int M, int N, int batch, int tm, int tn)
{
    return (long)((M + tm - 1) / tm) * ((N + tn - 1) / tn) * batch;
}

// What a launch of such tiles takes, in us: rounds of 256 compute units, each a slab at a time (what a compute
// unit spends on a slab is its LDS traffic; alone on it, a tile waits for its loads instead) and an end.
// Fitted to 1967 shapes timed with all three (M to 12608, N to 4096, K to 8192 bytes, up to 700 items, three
// types, both layouts of B): the estimate's choice is 0.6 % off the best on average, the rule of
// tile_size alone 1.6 %.
static double tile_cost(int M, int N, int nslab, int batch, int shape)
{
    static const int tm[3] = {64, 64, 128}, tn[3] = {64, 128, 128};
    static const double slab[3] = {0.22, 0.30, 0.45}, slab_alone[3] = {0.25, 0.39, 0.40}, end[3] = {0.25, 0.8, 2.8};
    const long n = (tiles_of(M, N, batch, tm[shape], tn[shape]) + 255) / 256;
    return nslab * (n > 1 ? slab[shape] * n : slab_alone[shape]) + end[shape] * n;
}

// Whether the tiles reduce A from the slabs they hold, behind a pass over B and with A b (APASS), instead of
// extra workgroups that read A and B again and a check that reads A a third time.  Those run in the LDS
// of a tile, one to three to a compute unit, and are for problems that leave the chip room.  From about
// 50 MB of A and B on the tiles' own reduction is the faster way; so / with the extra workgroups: f16 999 x 128
// x 516, 596 items 480 / 903 us; bf16 10496 x 768 x 2819, B cached 82 / 140; below, bf16 8409 x 1717 x 1300
// (26 MB) 108 / 107.  Batches need more (64 MB): their items have few slabs.  B stored K x N: the tiles
// wait for LDS more than for memory, and the reduction does not fit beside (f16 10934 x 1864 x 2268 206 / 193),
// but for large batches of many tiles, unless A is the far smaller operand (200 MB: int8 436 x 128 x 1360, 648 items
// 367 / 1156).
static bool fuses_a(int dt, const Shape &s, int nslab, int *bm)
{
    const double bytes = (double)s.batch * ((double)s.M + s.N) * s.K * elem_size(dt);
    if (nslab < 6 || (dt == DT_I8 && s.N >= 65536)) return false;
    if (s.transB ? bytes < (s.batch == 1 ? 48e6 : 64e6) : s.batch == 1 || bytes < 200e6 || s.M < s.N / 4) return false;
    *bm = tile_cost(s.M, s.N, nslab, s.batch, 1) < 0.8 * tile_cost(s.M, s.N, nslab, s.batch, 2) ? 64 : 128;
    const int tiles_n = (s.N + 127) / 128;
    const long tiles = tiles_of(s.M, s.N, s.batch, *bm, 128);
    return tiles >= 128 && tiles >= (s.transB ? 4 : 24) * apass_owned_slabs(nslab, tiles_n) && tiles / s.batch <= MAX_GRID_X &&
           tile_lds_bytes(*bm, 128, 3) + apass_lds_bytes(dt, nslab, tiles_n) + 128 * 4 <= 160 * 1024;       // (with the bias of a tile's columns)
}

// 64 x 64, 64 x 128 or 128 x 128 tiles.  Wider tiles cost less LDS traffic per product, but a problem of few
// tiles ends sooner the smaller its tiles are: 197 x 768 x 3072 (48 / 24 / 12 tiles) 12.7 / 17.8 / 27.4 us; 1000 x 1000
// x 1024 (256 / 128 / 64) 8.2 / 9.5 / 13.1; 2048 x 1024 x 1024 (512 / 256 / 128) 10.6 / 10.5 / 13.7;
// 6304 x 768 x 3080 with B stored K x N (1188 / 594 / 300) 64.9 / 59.0 / 64.3; 12608 x 1000 x 200
// (3152 / 1576 / 792) 26.3 / 25.0 / 29.5; 6304 x 3072 x 776 (4752 / 2376 / 1200) 74.3 / 69.5 / 62.9.
// Up to two slabs there is no main loop to speak of, and the smallest tile, of which most fit on a
// compute unit, hides the start and the end of its neighbours: 58 x (526 x 526 x 64) 23.4 / 30.8 /
// 49.4 us, 12608 x 1000 x 128 24.0 / 26.1 / 31.4.
// beside: workgroups beside the tiles read A and B in the LDS of a tile, which wide tiles leave little of.
// Without them the tile of the least estimated cost, where that is a tenth less (bf16 10496 x 768 x 2819,
// unprotected 86 -> 68 us).
static void tile_size(int M, int N, int nslab, int batch, bool beside, int *bm, int *bn)
{
    auto tiles = [&](int tm, int tn) { return tiles_of(M, N, batch, tm, tn); };
    *bm = *bn = 128;
    if (tiles(64, 64) / batch > MAX_GRID_X / 2) return;          // more than a launch holds
    int pick = 0;
    if (nslab > 2 && N > 64 && tiles(64, 64) > 256) pick = nslab >= 8 && tiles(128, 128) >= 1024 ? 2 : 1;
    if (!beside) {
        const int rule = pick;
        for (int i = 0; i < 3; ++i)
            if (tile_cost(M, N, nslab, batch, i) < tile_cost(M, N, nslab, batch, pick)) pick = i;
        if (tile_cost(M, N, nslab, batch, pick) > 0.9 * tile_cost(M, N, nslab, batch, rule)) pick = rule;
    }
    if (pick < 2) *bm = 64;
    if (pick < 1) *bn = 64;
}

template <int DT, int BM, int BN, int NS>
static hipError_t launch_cfg(bool protect, bool transB, HostArgs &a, int batch, hipStream_t st)
{
    a.g.tiles_m = (a.g.M + BM - 1) / BM;
    a.g.tiles_n = (a.g.N + BN - 1) / BN;
    a.g.group_inv = map_inverse(a.g.tiles_n);
    const long tiles = (long)a.g.tiles_m * a.g.tiles_n;
    if (tiles + a.n_extra > MAX_GRID_X) return hipErrorInvalidValue;
    a.n_tiles = (int)tiles;
    if constexpr (BN == 128)
        if (a.fuse_bm) return transB ? launch_one<DT, BM, BN, NS, true, true, true>(a, batch, st)
                                     : launch_one<DT, BM, BN, NS, true, false, true>(a, batch, st);
    if constexpr (BM == 64)
        if (a.p.one_launch) return transB ? launch_one<DT, BM, BN, NS, true, true, false, true>(a, batch, st)
                                          : launch_one<DT, BM, BN, NS, true, false, false, true>(a, batch, st);
    if (protect) return transB ? launch_one<DT, BM, BN, NS, true, true>(a, batch, st)
                               : launch_one<DT, BM, BN, NS, true, false>(a, batch, st);
    return transB ? launch_one<DT, BM, BN, NS, false, true>(a, batch, st)
                  : launch_one<DT, BM, BN, NS, false, false>(a, batch, st);
}

// Buffers: where every compute unit has a workgroup at most, four (197 x 768 x 3072: 12.7 us against
// 14.5 with three); otherwise three, for more workgroups on a compute unit (6304 x 768 x 768 on 64 x 64
// tiles: 17.3 us against 20.2 with four).
template <int DT>
static hipError_t launch_tile(bool protect, bool transB, HostArgs &a, int batch, hipStream_t st)
{
    int bm = a.fuse_bm, bn = 128;
    if (!bm) tile_size(a.g.M, a.g.N, slabs_of(DT, a.g.K), batch, protect, &bm, &bn);
    if (bm == 128) return launch_cfg<DT, 128, 128, 3>(protect, transB, a, batch, st);
    if (bn == 128) return launch_cfg<DT, 64, 128, 3>(protect, transB, a, batch, st);
    if ((long)((a.g.M + 63) / 64) * ((a.g.N + 63) / 64) * batch > 256) return launch_cfg<DT, 64, 64, 3>(protect, transB, a, batch, st);
    return launch_cfg<DT, 64, 64, 4>(protect, transB, a, batch, st);
}

bool gemm_fuses_a(int dt, const Shape &s)
{
    int bm;
    return !gemm_takes_fast(dt, s) && fuses_a(dt, s, slabs_of(dt, s.K), &bm);
}

void gemm_tile_shape(int dt, const Shape &s, int *tm, int *tn)
{
    if (gemm_item_eligible(dt, s, false)) {          // one workgroup per batch item
        *tm = s.M;
        *tn = s.N;
        return;
    }
    if (gemm_takes_fast(dt, s)) {
        gemm_fast_tile(tm, tn);
        return;
    }
    *tn = 128;
    if (!fuses_a(dt, s, slabs_of(dt, s.K), tm)) tile_size(s.M, s.N, slabs_of(dt, s.K), s.batch, true, tm, tn);
}

// The fast kernel's 256 x 256 tiles use the matrix cores best and fill the chip worst.  Time in the general kernel over that in the
// fast one, geometric mean over 350 random problems of all types by the number of such tiles, protected / unprotected: 32 to 39 0.76 / 0.84,
// 40 to 47 0.85 / 0.99, 48 to 55 0.81 / 1.05, 56 to 63 0.84 / 1.00, 64 to 79 1.15 / 1.25, 80 to 95 1.18 / 1.33.  (One line for both: a protected
// problem and the same unprotected take the same kernel.)
bool gemm_takes_fast(int dt, const Shape &s)
{
    const long tiles = (long)((s.M + 255) / 256) * ((s.N + 255) / 256) * s.batch;
    return tiles >= 64 && gemm_fast_eligible(dt, s.M, s.N, s.K, s.transB != 0, s.lda, s.ldb);
}

// Beside the tiles: about twelve row blocks, of one to eight batches of loads per thread.  The
// additions of the row blocks meet in the same words, which are served one after the other, and the
// last of them ends the launch: 6304 x 768 x 768 with 99 / 32 / 16 / 8 row blocks of A 26.6 / 22.8 /
// 22.2 / 22.2 us, 1537 x 1001 x 713 with 24 / 16 / 8 of them 15.4 / 13.6 / 13.0 us.
static int beside_batches(const EncPlan &p, int rows)
{
    const int per = 12 * (256 >> p.cw_log2) * ENC_UNROLL;
    return std::min((rows + per - 1) / per, 8);
}

static EncArgs enc_args(const void *X, long ld, long stride, int rows, int cols, int K, int reduce_rows, int dt,
                        uint32_t *sum, uint32_t *max_acc)
{
    EncArgs e;
    e.X = (const uint8_t *)X; e.ld = ld; e.stride = stride; e.rows = rows; e.cols = cols; e.K = K;
    e.reduce_rows = reduce_rows;
    const EncPlan p = plan_window(rows, cols, 16 / elem_size(dt));
    e.cw_log2 = p.cw_log2; e.nwin = p.nwin;
    e.rpb = beside_batches(p, rows) * (256 >> p.cw_log2) * ENC_UNROLL;
    e.nrb = (rows + e.rpb - 1) / e.rpb;
    e.sum = sum; e.max_acc = max_acc;
    return e;
}

// How a problem's predictions are dealt to workgroups (predict_pass.h): the operand that is split and its blocks, so that
// the estimate is least.  Returns that, in us; negative: it does not fit max_steps steps of LDS.  A step of a wave is an LDS
// read, MFMAs and their sums, twice; of a B stored K x N, vector instructions; and the shares of all workgroups
// meet in the same lines, where they queue (f16 4640 x 105 x 320 with 280 workgroups 22.1 us, 11.9 in two launches;
// int8 237 x 2112 x 2112 with 264 / 99 workgroups 23.0 / 10.7).
constexpr double PRED_STEP_US = 0.6, PRED_KN_STEP_US = 0.9, PRED_QUEUE_US = 0.02;
constexpr int PRED_MAX_WGS = 512;
// Workgroups of a launch, tiles and all: with more than one to a compute unit the tiles and the predictions wait for each other.
// One launch / two: 16-bit 1.03 to 1.27 on average, however long the predictions take (up to 256: 0.90 to 0.98); int8 0.88 to 0.94 up
// to 80 k additions, 1.0 to 1.1 beyond, but 0.95 where B is split and b given, so that one block alone forms A b.  16-bit shares
// are added in doubles: the tiles' own wait behind them (up to 120 k 0.92 to 0.97, to 160 k 0.96 to 1.02; 64 x 1536 x 3697, 193 k, 1.35).
constexpr int ONE_LAUNCH_CUS = 256;
constexpr double PRED_MAX_ADDS = 120e3, PRED_MAX_ADDS_SHARED = 80e3;
static double pred_plan(int dt, const Shape &s, bool b_given, int max_steps, long tiles, PredArgs *p)
{
    const int ce = 16 / elem_size(dt), kr = PRED_CHUNKS * ce;
    auto steps = [](int n, int per) { return (n + per - 1) / per; };
    const int nkr = steps(s.K, kr), pieces = steps(s.N, ce);
    double best = -1.0;
    auto offer = [&](int split_b, int units, int nblk, int whole, int split, int wa, int w_log2, double chain) {
        const int len = steps(units, nblk);
        nblk = steps(units, len);
        if (whole + split > max_steps || nkr * nblk > PRED_MAX_WGS) return;
        const double adds = (double)s.batch * nkr * (split_b ? (double)nblk * s.M + s.N : (double)nblk * s.N + s.M);
        const double cost = chain + PRED_QUEUE_US * nkr * nblk;
        const bool shares = tiles + (long)s.batch * nkr * nblk > ONE_LAUNCH_CUS;
        if (dt != DT_I8 ? shares || adds > PRED_MAX_ADDS : shares && adds > PRED_MAX_ADDS_SHARED && !(split_b && b_given)) return;
        if (best >= 0.0 && cost >= best) return;
        best = cost;
        p->nkr = nkr; p->nblk = nblk; p->split_b = split_b; p->blk_len = len;
        p->a_steps = split_b ? whole : split;
        p->b_steps = split_b ? split : whole;
        p->waves_a = wa; p->w_log2 = w_log2;
    };
    // steps of a K x N operand over c pieces of columns: a power of two of pieces of kr rows
    auto kn_log2 = [](int c) {
        int lg = 3;
        while ((1 << lg) < c) ++lg;
        return lg;
    };
    const int a_all = steps(s.M, 64);
    for (int nblk = 1; nblk <= 64; nblk += nblk < 8 ? 1 : 4) {
        if (s.transB) {
            const int split_b = s.N >= s.M, big = std::max(s.M, s.N);
            if (nblk > steps(big, 64)) break;
            const int whole = steps(std::min(s.M, s.N), 64), split = steps(steps(big, nblk), 64);
            for (int w = 1; w <= 3; ++w)                     // waves on the whole operand
                offer(split_b, big, nblk, whole, split, split_b ? w : 4 - w, 3,
                      PRED_STEP_US * std::max(steps(whole, w), steps(split, 4 - w)));
        } else {
            if (nblk <= steps(pieces, 8) && steps(pieces, nblk) <= 256) {
                const int lg = kn_log2(steps(pieces, nblk)), b = std::max(1, (kr << lg) / 256);
                offer(1, pieces, nblk, a_all, b, 4, lg, PRED_STEP_US * steps(a_all, 4) + PRED_KN_STEP_US * b);
            }
            if (nblk <= a_all && pieces <= 256) {
                const int lg = kn_log2(pieces), b = std::max(1, (kr << lg) / 256), a = steps(steps(s.M, nblk), 64);
                offer(0, s.M, nblk, b, a, 4, lg, PRED_STEP_US * steps(a, 4) + PRED_KN_STEP_US * b);
            }
        }
    }
    return best;
}

// Steps of LDS a workgroup of the predictions takes at most: what fits the LDS of the tiles beside it.
static int pred_max_steps(int bm, int bn, int ns) { return (tile_lds_bytes(bm, bn, ns) - PRED_VEC_WORDS * 4) / PRED_STEP_BYTES; }

// One launch, unless the predictions take longer than the tiles by more than the check kernel behind two launches costs: by the
// estimate, `longer` us.  One launch / two, averages over 8000 problems (linear layers, up to 63 attention items, three types, both
// layouts of B, cached or not), on this side of the line and half a us or 64 of K on the other:
//   B stored N x K  int8 0.86 | 0.93 (and up to 1.09); 16-bit 0.93 | 1.01, of a given b with B split, where one block alone forms
//                   A b, 0.93 | 1.02; where a pass over A or B beside the tiles of two launches would outlast them 0.90 | 0.95
//   B stored K x N  by its depth, which the check kernel goes through 512 at a time: 0.66 int8, 0.87 16-bit | 1.04, 1.01; batches
//                   0.95 | 1.0
constexpr int ONE_LAUNCH_MAX_TILES = 512, ONE_LAUNCH_MAX_BATCH_WGS = 440;
static bool one_launch_plan(int dt, const Shape &s, bool b_given, PredArgs *p, int *units)
{
    if (!s.transB && s.K <= (s.batch > 1 ? 512 : 384)) return false;
    if (gemm_takes_fast(dt, s) || s.batch > ONE_LAUNCH_MAX_BATCH || (long)s.batch * s.M > ONE_LAUNCH_MAX_LEN ||
        (long)s.batch * s.N > ONE_LAUNCH_MAX_LEN)
        return false;
    int bm, bn;
    const int nslab = slabs_of(dt, s.K);
    if (fuses_a(dt, s, nslab, &bm)) return false;
    tile_size(s.M, s.N, nslab, s.batch, true, &bm, &bn);
    if (bm != 64) return false;
    const long tiles = tiles_of(s.M, s.N, s.batch, bm, bn);
    *units = ((s.M + bm - 1) / bm + (s.N + bn - 1) / bn) * s.batch;
    if (tiles > ONE_LAUNCH_MAX_TILES || *units > ONE_LAUNCH_MAX_UNITS) return false;
    p->nkr = p->nblk = 0;
    const double pred = pred_plan(dt, s, b_given, pred_max_steps(bm, bn, bn == 64 && tiles <= 256 ? 4 : 3), tiles, p);
    if (s.batch > 1 && tiles + (long)s.batch * p->nkr * p->nblk > ONE_LAUNCH_MAX_BATCH_WGS) return false;
    auto pass = [&](int rows) { return 0.9 * beside_batches(plan_window(rows, s.K, 16 / elem_size(dt)), rows); };
    double longer = 1.75;
    if (s.transB) {
        const double passes = std::max(pass(s.M), b_given ? 0.0 : pass(s.N));
        longer = dt == DT_I8 || (s.batch == 1 && passes > 0.28 * nslab + 3.0) ? 2.0 : b_given && p->split_b && s.batch == 1 ? 1.0 : 0.5;
    }
    return pred >= 0.0 && pred <= 0.28 * nslab + longer;
}

size_t gemm_one_launch(int dt, const Shape &s, bool b_given)
{
    PredArgs p;
    int units;
    return one_launch_plan(dt, s, b_given, &p, &units) ? (size_t)(unit_line0(s.batch) + units) * TICKET_LINE : 0;
}

hipError_t launch_gemm(int dt, bool protect, bool stored_sums, bool encode_b, const void *A, const void *B, void *C,
                       const Shape &s, const Workspace &w, const InjectArm &arm, uint32_t *counts, const OneLaunch *one,
                       hipStream_t st)
{
    // The unprotected item kernels do not look for an armed flip (in them the look cost bf16 400 x 400 x 80,
    // 256 items 24.4 -> 25.0 us): such a call is tiled, C comes out bit for bit the same.
    if (!protect && !w.bias && arm.batch < 0 && gemm_item_eligible(dt, s, false, false))
        return launch_gemm_item(dt, false, false, false, A, B, C, s, w, nullptr, arm, st);
    HostArgs a;
    GemmArgs &g = a.g;
    g.A = (const uint8_t *)A;
    g.B = (const uint8_t *)B;
    g.C = (uint8_t *)C;
    g.M = s.M; g.N = s.N; g.K = s.K;
    g.lda = s.lda; g.ldb = s.ldb; g.ldc = s.ldc;
    g.sA = s.sA; g.sB = s.sB; g.sC = s.sC;
    g.inj_b = arm.batch; g.inj_row = arm.row; g.inj_col = arm.col; g.inj_bit = arm.bit;
    g.cc_obs = w.cc_obs; g.rc_obs = w.rc_obs; g.rc_pred = w.rc_pred; g.cc_acc = w.cc_acc; g.rc_acc = w.rc_acc;
    g.a_sum = w.a_sum; g.a_max = w.a_max; g.b_sum = w.b_sum;
    g.bias = w.bias;
    g.cc_sto = (protect && stored_sums && dt != DT_I8) ? w.cc_sto : nullptr;
    g.rc_sto = g.cc_sto ? w.rc_sto : nullptr;
    g.c_max = g.cc_sto ? w.c_max : nullptr;
    g.a_given = (protect && w.a_given) ? 1 : 0;
    g.tiles_m = g.tiles_n = g.n_big = g.tiles_m_big = g.tiles_m_small = 0;
    g.n_small = 0; g.batch = s.batch;
    g.counts = counts;
    if (gemm_takes_fast(dt, s)) return launch_gemm_fast(dt, protect, g, s.batch, st);
    a.counts = counts;
    a.bias_sum = w.bias_sum;
    a.ea = enc_args(A, s.lda, s.sA, s.M, s.K, s.K, 1, dt, w.a_sum, w.a_max);
    a.eb = s.transB ? enc_args(B, s.ldb, s.sB, s.N, s.K, s.K, 1, dt, w.b_sum, w.b_max)
                    : enc_args(B, s.ldb, s.sB, s.K, s.N, s.K, 0, dt, w.b_sum, w.b_max);
    a.fuse_bm = 0;
    if (protect && !fuses_a(dt, s, slabs_of(dt, s.K), &a.fuse_bm)) a.fuse_bm = 0;
    a.n_enc_a = (protect && !w.a_given && !a.fuse_bm) ? a.ea.nwin * a.ea.nrb : 0;
    a.n_enc_b = (protect && encode_b && !a.fuse_bm) ? a.eb.nwin * a.eb.nrb : 0;
    a.n_extra = a.n_enc_a + a.n_enc_b + (protect && w.bias && !a.fuse_bm ? 1 : 0);
    PredArgs &p = a.p;
    int units = 0;
    p.one_launch = protect && one && one_launch_plan(dt, s, !encode_b, &p, &units) ? 1 : 0;
    if (p.one_launch) {
        p.A = g.A; p.B = g.B;
        p.lda = s.lda; p.ldb = s.ldb; p.sA = s.sA; p.sB = s.sB;
        p.M = s.M; p.N = s.N; p.K = s.K; p.batch = s.batch;
        p.a_given = g.a_given; p.b_given = encode_b ? 0 : 1;
        p.a_vec = w.a_given;
        p.a_sum = w.a_sum; p.b_sum = w.b_sum; p.a_max = w.a_max; p.b_max = w.b_max;
        p.cc_pacc = w.cc_pacc; p.rc_pacc = w.rc_pacc; p.s_pacc = w.s_pacc;
        p.tickets = w.tickets;
        p.amax_in = (w.a_given && w.amax_given) ? w.amax_given : w.a_max;
        p.cc_obs = w.cc_obs; p.rc_obs = w.rc_obs; p.cc_acc = w.cc_acc; p.rc_acc = w.rc_acc;
        p.bias = w.bias;
        p.cc_pred = w.cc_pred; p.rc_pred = w.rc_pred; p.s_pred = w.s_pred; p.maxabs = w.maxabs; p.tau = w.tau;
        p.tau_override = one->v.tau_override; p.tau_override_cols = one->v.tau_override_cols;
        p.row_flag = one->v.row_flag; p.col_flag = one->v.col_flag; p.counts = one->v.counts;
        p.zero_ptr = one->zero_ptr; p.zero_words = one->zero_words;
        p.zero2_ptr = one->zero2_ptr; p.zero2_words = one->zero2_words;
        a.n_extra = p.nkr * p.nblk + (p.bias ? 1 : 0);
    }
    switch (dt) {
    case DT_I8:   return launch_tile<DT_I8>(protect, s.transB != 0, a, s.batch, st);
    case DT_BF16: return launch_tile<DT_BF16>(protect, s.transB != 0, a, s.batch, st);
    case DT_F16:  return launch_tile<DT_F16>(protect, s.transB != 0, a, s.batch, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace abft
