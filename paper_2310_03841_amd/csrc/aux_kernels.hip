// Kernels around the protected GEMM: the pass over B (its checksum vector), check (the predictions
// that are missing, compare, flags), verify (re-sum stored C),
// correct (localise, recompute tiles, re-check) and the bit-flip test hook.
//
// Paper references: the two input-side vectors and the comparison with the
// output sums are the checksum scheme of Sec. III-B.1 ("Checksums"); equality
// for integers and a tolerance for floating point follow item (2) there; the
// tile recompute is the replay correction of Sec. III-B.3 at tile granularity;
// the flip is the fault model of Sec. II-A / III-A.
#include <mutex>

#include "abft_device.h"
#include "encode_pass.h"

namespace abft {

// ======================================================================== per-device launch state
static std::mutex g_launch_lock;

hipError_t ensure_max_lds(const void *kernel, int bytes)
{
    struct Done { const void *kernel; int device; };
    static Done done[512];
    static int n_done = 0;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> hold(g_launch_lock);
    for (int i = 0; i < n_done; ++i)
        if (done[i].kernel == kernel && done[i].device == dev) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    if (n_done < 512) done[n_done++] = Done{kernel, dev};
    return hipSuccess;
}

int device_cu_count(hipError_t *err)
{
    static int cus[64];
    int dev = 0, n = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= 64)) e = hipErrorInvalidDevice;
    if (e == hipSuccess) {
        std::lock_guard<std::mutex> hold(g_launch_lock);
        if (cus[dev] == 0) {
            e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
            if (e == hipSuccess) cus[dev] = n > 0 ? n : 256;
        }
        n = cus[dev];
    }
    if (err) *err = e;
    return e == hipSuccess ? n : 0;
}

// ======================================================================== zero
__global__ void zero_kernel(uint32_t *p, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) p[i] = 0u;
}

hipError_t launch_zero(uint32_t *p, size_t nwords, hipStream_t st)
{
    if (nwords == 0) return hipSuccess;
    size_t blocks = (nwords + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, nwords);
    return hipGetLastError();
}

__global__ void copy_kernel(uint32_t *dst, const uint32_t *src, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) dst[i] = src[i];
}

hipError_t launch_copy(uint32_t *dst, const uint32_t *src, size_t nwords, hipStream_t st)
{
    size_t blocks = (nwords + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, dst, src, nwords);
    return hipGetLastError();
}

// ====================================================================== encode
// Input-side checksum vectors (Sec. III-B.1 "Checksums"): a = e^T A (the input summed over its
// rows) and b = B e (the weight reduced over its output dimension), both of length K, plus
// max|A|, max|B| for the tolerance and the row checksum prediction rc_pred = A b.  Where the GEMM
// kernel reduces A from the slabs it holds in LDS (gemm_apass.h: the fast kernel, the general one for
// large problems), b must be complete before it (A b needs all of b): the pass over B as a kernel of its own.
// For a weight it is done once, offline (remark (2) of the same paragraph).  Otherwise the general kernel
// runs the passes over A and B beside its tiles, and A b is formed by the check kernel.
struct EncBArgs {
    EncArgs e;
    uint32_t *zero_ptr;   // region every block helps to clear (the next kernel's atomics start at zero)
    size_t zero_words;
};

template <int DT>
__global__ __launch_bounds__(256) void encode_b_kernel(EncBArgs a)
{
    fetch_args<EncBArgs>();
    __shared__ uint32_t red[256 * (16 / Traits<DT>::ES) + 4];
    const int tid = threadIdx.x, bz = blockIdx.z;
    {
        const size_t nb = (size_t)gridDim.x * gridDim.z;
        const size_t bid = blockIdx.x + (size_t)gridDim.x * blockIdx.z;
        for (size_t i = bid * 256 + tid; i < a.zero_words; i += nb * 256) a.zero_ptr[i] = 0u;
    }
    encode_block<DT, ENC_UNROLL_ALONE>(a.e, blockIdx.x, bz, red);
}

hipError_t launch_encode_b(int dt, const void *B, const Shape &s, const Workspace &w, uint32_t *zero_ptr,
                           size_t zero_words, hipStream_t st)
{
    EncBArgs a;
    EncArgs &e = a.e;
    e.X = (const uint8_t *)B; e.ld = s.ldb; e.stride = s.sB; e.K = s.K;
    if (s.transB) { e.rows = s.N; e.cols = s.K; e.reduce_rows = 1; }
    else          { e.rows = s.K; e.cols = s.N; e.reduce_rows = 0; }
    const EncPlan p = plan_alone(e.rows, e.cols, 16 / elem_size(dt));
    e.cw_log2 = p.cw_log2; e.nwin = p.nwin; e.rpb = p.rpb; e.nrb = p.nrb;
    e.sum = w.b_sum; e.max_acc = w.b_max;
    a.zero_ptr = zero_ptr; a.zero_words = zero_ptr ? zero_words : 0;
    dim3 grid((unsigned)(e.nwin * e.nrb), 1, (unsigned)s.batch);
    switch (dt) {
    case DT_I8:   hipLaunchKernelGGL(encode_b_kernel<DT_I8>, grid, dim3(256), 0, st, a); break;
    case DT_BF16: hipLaunchKernelGGL(encode_b_kernel<DT_BF16>, grid, dim3(256), 0, st, a); break;
    case DT_F16:  hipLaunchKernelGGL(encode_b_kernel<DT_F16>, grid, dim3(256), 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Largest K of a protected GEMM: the column sums of A's slabs wait in LDS (4 bytes per column
// of K) next to the operand buffers until the epilogue.
int protect_max_k(int dt) { (void)dt; return 4096; }

// A wave found n rows (side 0) or n columns (side 1) that disagree.  counts[side] gains them; counts[2] and
// counts[4] become the status: localised once both sides have flags, suspect while one has.  Only the
// first wave of a side writes it.  It adds first and looks at the other side second, so of the two first
// waves at least one sees both; "localised" goes in whatever is there, "suspect" only replaces "clean".
// (With every wave looking and writing, a bf16 12608 x 3072 x 768 whose every row and column flags took 137 us;
// so 84, and 78 clean: atomics on one line are served one after the other.)
// fix_count: after a correction (counts[4] is the status before it; counts[2] stays where the list was too long).
__device__ __forceinline__ void report_flags(uint32_t *counts, int side, unsigned n, const uint32_t *fix_count = nullptr)
{
    if (atomicAdd(counts + side, n) != 0u) return;
    if (fix_count && fix_count[1]) return;
    if (atomicAdd(counts + (side ^ 1), 0u) != 0u) {
        atomicExch(counts + 2, 1u);
        if (!fix_count) atomicExch(counts + 4, 1u);
    } else {
        atomicCAS(counts + 2, 0u, 2u);
        if (!fix_count) atomicCAS(counts + 4, 0u, 2u);
    }
}

// ===================================================================== compare
// Flags from observed sums against the predictions the last abft_gemm left in the context
// (Sec. III-B.1 item (2): equality for fixed point, tolerance for floating point).  Used by
// abft_verify and abft_correct; abft_gemm compares in its check kernel.
struct CmpArgs {
    const uint32_t *cc_pred, *rc_pred;
    const uint32_t *cc_obs, *rc_obs;
    const float *tau;
    float tau_override;   // > 0: use this tolerance instead of tau[]
    float tau_override_cols;   // > 0: tolerance of the column check
    uint8_t *row_flag, *col_flag;
    uint32_t *counts;
    uint32_t *ticket;     // after a correction: [3]: ticket, flagged rows, flagged cols (self-cleaning)
    uint32_t *fix_count;  // non-null after a correction: [0] tiles listed, [1] overflow (cleared after use, but with counts_ready)
    const int32_t *fix_tiles;          // after a correction: the tiles it recomputed
    uint32_t *cc_sto, *rc_sto;         // non-null: stored-side sums of the GEMM (floating point)
    uint32_t *zero_ptr;   // region every block helps to clear: the re-summing region not in use,
    size_t zero_words;    // so that the next re-sum finds it clean
    int M, N, batch;
    const uint32_t *gate; // non-null: if *gate == 0 (no tile was listed for recomputation) the kernel
                          // leaves flags and counts as the check before it wrote them
    int counts_ready;     // after a correction: resum_touched_kernel has written counts, the list is not cleared
};

template <bool IS_INT>
__global__ __launch_bounds__(256) void compare_kernel(CmpArgs a)
{
    fetch_args<CmpArgs>();
    __shared__ int is_last;
    const int bz = blockIdx.z, tid = threadIdx.x;
    const int idx = blockIdx.x * 256 + tid;
    const int M = a.M, N = a.N;
    {
        const size_t nb = (size_t)gridDim.x * gridDim.z;
        const size_t bid = blockIdx.x + (size_t)gridDim.x * blockIdx.z;
        for (size_t i = bid * 256 + tid; i < a.zero_words; i += nb * 256) a.zero_ptr[i] = 0u;
    }
    if (a.gate && *a.gate == 0u) return;           // uniform over the grid: nobody touches the ticket
    const float tol = IS_INT ? 0.f : (a.tau_override > 0.f ? a.tau_override : a.tau[bz]);
    const float tol_c = (!IS_INT && a.tau_override_cols > 0.f) ? a.tau_override_cols : tol;
    bool frow = false, fcol = false;
    if (!IS_INT && a.fix_count && a.rc_sto && idx < M + N) {
        // After a correction the stored-side sums of the GEMM no longer describe the rows and
        // columns of the recomputed tiles: if the fault was already in the accumulators when the
        // epilogue summed them, those sums contain it, and the repaired values do not.  The fresh
        // re-sum of the repaired rows and columns takes their place.
        unsigned n = a.fix_count[0];
        if (n > (unsigned)MAX_FIX_TILES) n = MAX_FIX_TILES;
        const int mine = (idx < M ? idx : idx - M) / CT, which = idx < M ? 1 : 2;
        bool touched = false;
        for (unsigned t = 0; t < n; ++t)
            touched = touched || (a.fix_tiles[3 * t] == bz && a.fix_tiles[3 * t + which] == mine);
        if (touched) {
            if (idx < M) a.rc_sto[(long)bz * M + idx] = a.rc_obs[(long)bz * M + idx];
            else a.cc_sto[(long)bz * N + idx - M] = a.cc_obs[(long)bz * N + idx - M];
        }
    }
    if (idx < M) {
        frow = mismatch<IS_INT>(a.rc_obs[(long)bz * M + idx], a.rc_pred[(long)bz * M + idx], tol);
        if (!IS_INT && a.rc_sto)
            frow = frow || mismatch<false>(a.rc_obs[(long)bz * M + idx], a.rc_sto[(long)bz * M + idx], STO_TOL_FACTOR * tol);
        a.row_flag[(long)bz * M + idx] = frow ? 1 : 0;
    } else if (idx < M + N) {
        const int j = idx - M;
        fcol = mismatch<IS_INT>(a.cc_obs[(long)bz * N + j], a.cc_pred[(long)bz * N + j], tol_c);
        if (!IS_INT && a.cc_sto)
            fcol = fcol || mismatch<false>(a.cc_obs[(long)bz * N + j], a.cc_sto[(long)bz * N + j], STO_TOL_FACTOR * tol_c);
        a.col_flag[(long)bz * N + j] = fcol ? 1 : 0;
    }
    if (!a.fix_count || a.counts_ready) {
        // the pass over stored C has cleared the counts: only waves that saw a mismatch touch them.  (A ticket per block and
        // a last block that publishes are two trips to memory more: int8 6304 x 768 x 3072, flip, verify and repair
        // 33.7 -> 32.8 us; bf16 6304 x 3072 x 768 with stored sums and verify 80.0 -> 77.1.)
        const unsigned wr = __popcll(__ballot(frow)), wc = __popcll(__ballot(fcol));
        if ((tid & 63) == 0) {
            if (wr) report_flags(a.counts, 0, wr, a.fix_count);
            if (wc) report_flags(a.counts, 1, wc, a.fix_count);
        }
        return;
    }
    const unsigned nr = __syncthreads_count(frow);
    const unsigned nc = __syncthreads_count(fcol);
    if (tid == 0) {
        if (nr | nc) {
            // rare: the counts must be at the coherence point before this block's ticket is, so
            // fetch their old values and wait for them
            unsigned o1 = 0, o2 = 0;
            if (nr) o1 = atomicAdd(a.ticket + 1, nr);
            if (nc) o2 = atomicAdd(a.ticket + 2, nc);
            asm volatile("s_waitcnt vmcnt(0)" :: "v"(o1), "v"(o2) : "memory");
        }
        unsigned total = gridDim.x * gridDim.z;
        unsigned t = atomicAdd(a.ticket, 1u);
        is_last = (t == total - 1);
    }
    __syncthreads();
    if (is_last && tid == 0) {
        uint32_t r = atomicExch(a.ticket + 1, 0u), c = atomicExch(a.ticket + 2, 0u);
        atomicExch(a.ticket, 0u);
        const uint32_t before = a.counts[2];
        a.counts[0] = r;
        a.counts[1] = c;
        // the list is consumed: the next correction starts from an empty one
        const uint32_t tiles = atomicExch(a.fix_count, 0u);
        a.counts[2] = atomicExch(a.fix_count + 1, 0u) ? 3u : status_of(r, c);
        a.counts[3] = tiles > (uint32_t)MAX_FIX_TILES ? (uint32_t)MAX_FIX_TILES : tiles;
        a.counts[4] = before;
    }
}

hipError_t launch_compare(int dt, const Shape &s, const Workspace &w, const Verdict &v, bool after_fix,
                          bool with_sto, uint32_t *zero_ptr, size_t zero_words, hipStream_t st, bool gated, bool counts_ready)
{
    CmpArgs a;
    a.counts_ready = counts_ready ? 1 : 0;
    a.gate = gated ? w.fix_count : nullptr;
    a.zero_ptr = zero_ptr; a.zero_words = zero_ptr ? zero_words : 0;
    a.cc_sto = (with_sto && dt != DT_I8) ? w.cc_sto : nullptr;
    a.rc_sto = a.cc_sto ? w.rc_sto : nullptr;
    a.fix_count = after_fix ? w.fix_count : nullptr;
    a.fix_tiles = w.fix_tiles;
    a.cc_pred = w.cc_pred; a.rc_pred = w.rc_pred;
    a.cc_obs = w.cc_vobs; a.rc_obs = w.rc_vobs;
    a.tau = w.tau; a.tau_override = v.tau_override; a.tau_override_cols = v.tau_override_cols;
    a.row_flag = v.row_flag; a.col_flag = v.col_flag; a.counts = v.counts;
    a.ticket = w.cmp_ticket;
    a.M = s.M; a.N = s.N; a.batch = s.batch;
    dim3 grid((unsigned)((s.M + s.N + 255) / 256), 1, (unsigned)s.batch);
    if (dt == DT_I8) hipLaunchKernelGGL(compare_kernel<true>, grid, dim3(256), 0, st, a);
    else             hipLaunchKernelGGL(compare_kernel<false>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

// ======================================================================= check
// Runs after a GEMM kernel, whose launch has completed a = e^T A, b = B e, the two maxima and the
// observed sums.  Forms the predictions of Sec. III-B.1 that are missing, cc_pred = a B and (unless the GEMM
// kernel formed it from the slabs it holds: rc_ready) rc_pred = A b, each a matrix-vector product over
// one read of its operand, compares and flags.
//
// Bound by latency: a workgroup's critical path is one round of loads and one reduction.  Units of a
// batch item: row units of A, column units of B (a B stored N x K is the same product as A b), one
// unit for the scalar a.b.  There is no last block: the GEMM launch has cleared the counts, and only
// waves that saw a mismatch touch them (report_flags).  (Behind the fast kernel there used to be a kernel
// of its own, with eight rows of B per wave and a ticket per workgroup; a call with a bf16 12608 x 3072 x 768
// then took 80.1 us and takes 77.9, with 6304 x 768 x 3072 in fp16 57.8 and 54.1, with an int8 12608 x 1024 x
// 1024 41.2 and 37.9.)
struct ChkArgs {
    const uint8_t *A, *B;
    long lda, sA, ldb, sB;
    int transB;
    int M, N, K, batch;
    const uint32_t *a_sum, *b_sum, *a_max, *b_max;
    uint32_t *cc_obs, *rc_obs;       // integers: complete; floating point: written here from
    const double *cc_acc, *rc_acc;   // what the tiles added up (null: cc_obs, rc_obs are complete)
    int rc_ready;                    // rc_pred holds A b: the row units compare 256 rows each
    const uint32_t *bias; // layer bias [N] or null: cc_pred gains M bias[n], rc_pred sum(bias), a.b M sum(bias)
    const uint32_t *bias_sum;   // its sum, formed by the general kernel's launch (with rc_ready: formed here)
    uint32_t *cc_pred, *rc_pred, *s_pred;
    float *maxabs, *tau;
    float tau_override, tau_override_cols;
    uint8_t *row_flag, *col_flag;
    uint32_t *counts;
    int row_units, col_units;
    unsigned grid_x;      // workgroups along x
    int ksplit;           // 1, or 4 (deep K): the four waves of a unit share its rows, a quarter of K each
    uint32_t *zero_ptr;   // region every block helps to clear: what the previous protected GEMM of this
    size_t zero_words;    // context accumulated into, so that the next one finds it clean
    uint32_t *zero2_ptr;  // second region to clear: the b slot the next pass over B will accumulate into
    size_t zero2_words;
};

// Dots of RW rows of a K-contiguous operand with a vector of K words: lanes along K, two chunks per
// lane and trip, everything of a trip in flight.  split: this wave takes every fourth run of 128
// chunks.  Every lane returns the wave's share of all RW dots.
// Loads without a lane's branch (around one the compiler waits for those before it): lanes and rows past the end ask for the last
// whole chunk and the last row.  What lies behind the last whole chunk is asked for first, an element a lane.  The vector may
// start on any word: batch items of a ragged K do, and a caller's may.  (The kernel, with a branch around each load / with a path of loads
// without them for whole chunks and aligned vectors, word by word otherwise / so: int8 10624 x 221 x 2360 14.8 / 20.6 / 11.8 us; 570 x 570 x 48, 48
// items, where the second 64 lanes of a trip have nothing, 19.1 / 21.8 / 11.7; bf16 640 x 2880 x 1535 4.7 / 6.6 / 4.8.)
typedef int i32x4_word __attribute__((ext_vector_type(4), aligned(4)));
template <int DT, int RW>
__device__ __forceinline__ void row_dots(const uint8_t *X, long ld, int row0, int rows, int K, const uint32_t *vec,
                                         bool split, typename Traits<DT>::acc_t (&dot)[RW])
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int ES = T::ES, CE = 16 / ES;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nch = K / CE, tail = nch * CE + lane;              // whole chunks; this lane's element behind them
    uint32_t xt[RW], vt;
    if (nch * CE < K) {
        const int k = min(tail, K - 1);
        vt = vec[k];
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            const uint8_t *at = X + ((long)min(row0 + j, rows - 1) * ld + k) * ES;
            if constexpr (ES == 2) xt[j] = *reinterpret_cast<const uint16_t *>(at);
            else xt[j] = *at;
        }
    }
#pragma unroll
    for (int j = 0; j < RW; ++j) dot[j] = T::zero();
    for (int ch0 = split ? wave * 128 : 0; ch0 < nch; ch0 += split ? 512 : 128) {
        i32x4 v[RW][2];
        i32x4_word aw[2][CE / 4];
        auto load = [&](int h) __attribute__((always_inline)) {
            const int ch = min(ch0 + 64 * h + lane, nch - 1);
#pragma unroll
            for (int j = 0; j < RW; ++j)
                v[j][h] = *reinterpret_cast<const i32x4 *>(X + ((long)min(row0 + j, rows - 1) * ld + (long)ch * CE) * ES);
#pragma unroll
            for (int q4 = 0; q4 < CE / 4; ++q4) aw[h][q4] = *reinterpret_cast<const i32x4_word *>(vec + ch * CE + 4 * q4);
        };
        auto add = [&](int h) __attribute__((always_inline)) {
            if (ch0 + 64 * h + lane < nch) {
#pragma unroll
                for (int j = 0; j < RW; ++j)
#pragma unroll
                    for (int q = 0; q < CE; ++q)
                        dot[j] = add_t(dot[j], mul_t(T::elem(v[j][h], q), from_word<acc_t>((uint32_t)aw[h][q >> 2][q & 3])));
            }
        };
        const bool two = ch0 + 64 < nch;
        load(0);
        if (two) load(1);
        add(0);
        if (two) add(1);
    }
    if (tail < K && (!split || wave == 0)) {
#pragma unroll
        for (int j = 0; j < RW; ++j)
            dot[j] = add_t(dot[j], mul_t(T::elem(i32x4{(int)xt[j], 0, 0, 0}, 0), from_word<acc_t>(vt)));
    }
#pragma unroll
    for (int j = 0; j < RW; ++j) dot[j] = wave_sum(dot[j]);
}

constexpr int CHK_KN_LANES = 4;        // chunk columns of a unit over a B stored K x N (64 lanes run along k)

template <int DT, int RW>
__global__ __launch_bounds__(256) void check_kernel(ChkArgs f)
{
    fetch_args<ChkArgs>();
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int ES = T::ES, CE = 16 / ES;
    __shared__ acc_t wred[4];
    __shared__ acc_t part[4][CHK_KN_LANES * CE > RW ? CHK_KN_LANES * CE : RW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int M = f.M, N = f.N, K = f.K;
    // every cache line of the arguments is asked for at once: left alone, the loads wait for the branch below
    asm volatile("" :: "s"(f.A), "s"(f.K), "s"(f.cc_acc), "s"(f.maxabs), "s"(f.zero2_words));
    const unsigned upi = (unsigned)f.row_units + f.col_units + 1;      // units per batch item
    const unsigned id = blockIdx.y * f.grid_x + blockIdx.x;
    if (id >= upi * f.batch) return;
    const int bz = id / upi, u = id - bz * upi;
    const uint32_t *asum = f.a_sum + (long)bz * K, *bsum = f.b_sum + (long)bz * K;
    {
        const size_t nb = (size_t)upi * f.batch;
        for (size_t i = (size_t)id * 256 + tid; i < f.zero_words; i += nb * 256) f.zero_ptr[i] = 0u;
        for (size_t i = (size_t)id * 256 + tid; i < f.zero2_words; i += nb * 256) f.zero2_ptr[i] = 0u;
    }
    // What the comparison needs is requested here and first used behind the dots: a use in between (the
    // tolerance, the conversion of an observed sum) is a wait for memory ahead of the loads of the dots.  (bf16 12608 x 3072 x
    // 768, nothing cached: 76.1 -> 75.7 us; 1537 x 1001 x 713 with B stored K x N: 16.3 -> 15.9; 6304 x 3072 x 768: 81.6 -> 80.0 with sums and verify.)
    uint32_t ma = 0, mb = 0;
    if (!T::IS_INT) { ma = f.a_max[bz]; mb = f.b_max[bz]; }
    auto tolerance = [&]() __attribute__((always_inline)) {
        return T::IS_INT ? 0.f : f.tau_override > 0.f ? f.tau_override : (1e-3f * (float)K) * __uint_as_float(ma) * __uint_as_float(mb);
    };
    auto tolerance_cols = [&]() __attribute__((always_inline)) { return f.tau_override_cols > 0.f ? f.tau_override_cols : tolerance(); };
    const bool acc_obs = !T::IS_INT && f.cc_acc != nullptr;     // the observed sums are still doubles
    // An observed sum as two words (the second one is only looked at if it is a double): loads without a branch, into
    // registers nothing else is written to.
    struct Obs { uint32_t lo, hi; };
    auto request = [&](const double *acc, const uint32_t *sum, long o) __attribute__((always_inline)) {
        const uint32_t *at = acc_obs ? reinterpret_cast<const uint32_t *>(acc + o) : sum + o;
        return Obs{at[0], at[acc_obs ? 1 : 0]};
    };
    auto observed = [&](const Obs &x) __attribute__((always_inline)) {
        return acc_obs ? __float_as_uint((float)__hiloint2double((int)x.hi, (int)x.lo)) : x.lo;
    };
    // sum of the bias
    const uint32_t sb_word = *(f.bias && !f.rc_ready ? f.bias_sum : bsum);
    acc_t sb_block = T::zero();
    if (f.bias && f.rc_ready && (u == (int)upi - 1 || u < f.row_units)) {
        sb_block = block_bias_sum<acc_t>(f.bias, N, wred);
        __syncthreads();
    }
    auto bias_sum = [&]() __attribute__((always_inline)) {
        return !f.bias ? T::zero() : f.rc_ready ? sb_block : from_word<acc_t>(sb_word);
    };
    if (u == (int)upi - 1) {
        // scalar a . b (the single-number check value of Sec. III-B.1)
        acc_t v = T::zero();
        for (int k = tid; k < K; k += 256) v = add_t(v, mul_t(from_word<acc_t>(asum[k]), from_word<acc_t>(bsum[k])));
        v = wave_sum(v);
        if (lane == 0) wred[wave] = v;
        __syncthreads();
        if (tid == 0) {
            f.s_pred[bz] = as_word(add_t(add_t(add_t(wred[0], wred[1]), add_t(wred[2], wred[3])), mul_t((acc_t)M, bias_sum())));
            if (!T::IS_INT) {
                f.maxabs[(long)bz * 2] = __uint_as_float(ma);
                f.maxabs[(long)bz * 2 + 1] = __uint_as_float(mb);
                f.tau[bz] = tolerance();
            }
        }
        return;
    }
    const bool is_row = u < f.row_units;
    if (is_row && f.rc_ready) {
        const int r = u * 256 + tid;
        bool fl = false;
        if (r < M) {
            const long o = (long)bz * M + r;
            uint32_t pred = f.rc_pred[o];
            const Obs x = request(f.rc_acc, f.rc_obs, o);
            const uint32_t obs = observed(x);
            if (acc_obs) f.rc_obs[o] = obs;
            if (f.bias) { pred = as_word(add_t(from_word<acc_t>(pred), sb_block)); f.rc_pred[o] = pred; }
            fl = mismatch<T::IS_INT>(obs, pred, tolerance());
            f.row_flag[o] = fl ? 1 : 0;
        }
        const unsigned nf = __popcll(__ballot(fl));
        if (nf && lane == 0) report_flags(f.counts, 0, nf);
    } else if (is_row || f.transB) {
        // A b against the row sums of C, or a B (rows of B are columns of C) against the column sums
        const int unit = is_row ? u : u - f.row_units;
        const bool split = f.ksplit == 4;
        const int rows = is_row ? M : N;
        const int row0 = split ? unit * RW : (unit * 4 + wave) * RW;
        const bool mine_ok = lane < RW && row0 + lane < rows && (!split || wave == 0);
        const long o = (long)bz * rows + row0 + lane;
        // what the dots are compared with, requested first
        const int at = min(row0 + (lane & (RW - 1)), rows - 1);
        const Obs x = request(is_row ? f.rc_acc : f.cc_acc, is_row ? f.rc_obs : f.cc_obs, (long)bz * rows + at);
        const uint32_t bias = *(f.bias && !is_row ? f.bias + at : bsum);
        acc_t dot[RW];
        row_dots<DT, RW>(is_row ? f.A + (long)bz * f.sA * ES : f.B + (long)bz * f.sB * ES, is_row ? f.lda : f.ldb, row0, rows, K,
                         is_row ? bsum : asum, split, dot);
        if (split) {
            if (lane == 0) {
#pragma unroll
                for (int j = 0; j < RW; ++j) part[wave][j] = dot[j];
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < RW; ++j) dot[j] = add_t(add_t(part[0][j], part[1][j]), add_t(part[2][j], part[3][j]));
        }
        acc_t mine = dot[0];
#pragma unroll
        for (int j = 1; j < RW; ++j) mine = lane == j ? dot[j] : mine;
        if (f.bias) mine = add_t(mine, is_row ? bias_sum() : mul_t((acc_t)M, from_word<acc_t>(bias)));
        const uint32_t obs = observed(x);
        bool fl = false;
        if (mine_ok) {
            (is_row ? f.rc_pred : f.cc_pred)[o] = as_word(mine);
            if (acc_obs) (is_row ? f.rc_obs : f.cc_obs)[o] = obs;
            fl = mismatch<T::IS_INT>(obs, as_word(mine), is_row ? tolerance() : tolerance_cols());
            (is_row ? f.row_flag : f.col_flag)[o] = fl ? 1 : 0;
        }
        const unsigned nf = __popcll(__ballot(fl));
        if (nf && lane == 0) report_flags(f.counts, is_row ? 0 : 1, nf);
    } else {
        // a B over a B stored K x N: CHK_KN_LANES chunk columns, 64 lanes along k
        const int cx = tid % CHK_KN_LANES, ky = tid / CHK_KN_LANES;
        const uint8_t *Bb = f.B + (long)bz * f.sB * ES;
        const int col0 = (u - f.row_units) * CHK_KN_LANES * CE, nst = col0 + cx * CE;
        const bool in = nst < N;
        const int n = col0 + tid;                               // this thread's column in the end
        const bool mine_ok = tid < CHK_KN_LANES * CE && n < N;
        const int at = min(n, N - 1);
        const Obs x = request(f.cc_acc, f.cc_obs, (long)bz * N + at);
        const uint32_t bias = *(f.bias ? f.bias + at : bsum);
        acc_t colp[CE];
#pragma unroll
        for (int q = 0; q < CE; ++q) colp[q] = T::zero();
        constexpr int U = 8;
        for (int k0 = ky; k0 < K; k0 += 64 * U) {
            i32x4 v[U];
            acc_t ak[U];
#pragma unroll
            for (int uu = 0; uu < U; ++uu) {
                const int k = k0 + 64 * uu;
                v[uu] = i32x4{0, 0, 0, 0};
                ak[uu] = T::zero();
                if (k < K && in) {
                    v[uu] = *reinterpret_cast<const i32x4 *>(Bb + ((long)k * f.ldb + nst) * ES);
                    ak[uu] = from_word<acc_t>(asum[k]);
                }
            }
#pragma unroll
            for (int uu = 0; uu < U; ++uu) {
                if (k0 + 64 * uu < K) {
#pragma unroll
                    for (int q = 0; q < CE; ++q) colp[q] = add_t(colp[q], mul_t(T::elem(v[uu], q), ak[uu]));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < CE; ++q) {
            acc_t t = colp[q];
            t = add_t(t, dpp_get<0x124>(t));                    // row_ror:4 inside 16 lanes
            t = add_t(t, dpp_get<0x128>(t));                    // row_ror:8
            t = add_xor16(t);
            t = add_xor32(t);
            if (lane < CHK_KN_LANES) part[wave][cx * CE + q] = t;
        }
        __syncthreads();
        bool fl = false;
        if (mine_ok) {
            acc_t t = add_t(add_t(part[0][tid], part[1][tid]), add_t(part[2][tid], part[3][tid]));
            if (f.bias) t = add_t(t, mul_t((acc_t)M, from_word<acc_t>(bias)));
            const uint32_t obs = observed(x);
            const long o = (long)bz * N + n;
            f.cc_pred[o] = as_word(t);
            if (acc_obs) f.cc_obs[o] = obs;
            fl = mismatch<T::IS_INT>(obs, as_word(t), tolerance_cols());
            f.col_flag[o] = fl ? 1 : 0;
        }
        const unsigned nf = __popcll(__ballot(fl));
        if (nf && lane == 0) report_flags(f.counts, 1, nf);
    }
}

hipError_t launch_check(int dt, bool after_fast, bool rc_ready, const void *A, const void *B, const Shape &s, const Workspace &w, const Verdict &v,
                        uint32_t *zero_ptr, size_t zero_words, uint32_t *zero2_ptr, size_t zero2_words, hipStream_t st)
{
    constexpr int RW = 4;                                       // rows per wave
    ChkArgs f;
    f.A = (const uint8_t *)A; f.B = (const uint8_t *)B;
    f.lda = s.lda; f.sA = s.sA; f.ldb = s.ldb; f.sB = s.sB; f.transB = s.transB;
    f.M = s.M; f.N = s.N; f.K = s.K; f.batch = s.batch;
    f.a_sum = w.a_given ? w.a_given : w.a_sum;
    f.a_max = (w.a_given && w.amax_given) ? w.amax_given : w.a_max;
    f.b_sum = w.b_sum; f.b_max = w.b_max; f.cc_obs = w.cc_obs; f.rc_obs = w.rc_obs;
    f.cc_acc = after_fast ? nullptr : w.cc_acc; f.rc_acc = after_fast ? nullptr : w.rc_acc;
    f.rc_ready = rc_ready ? 1 : 0;
    f.bias = w.bias; f.bias_sum = w.bias_sum;
    f.cc_pred = w.cc_pred; f.rc_pred = w.rc_pred; f.s_pred = w.s_pred; f.maxabs = w.maxabs; f.tau = w.tau;
    f.tau_override = v.tau_override; f.tau_override_cols = v.tau_override_cols;
    f.row_flag = v.row_flag; f.col_flag = v.col_flag; f.counts = v.counts;
    f.zero_ptr = zero_ptr; f.zero_words = zero_ptr ? zero_words : 0;
    f.zero2_ptr = zero2_ptr; f.zero2_words = zero2_ptr ? zero2_words : 0;
    const int ce = 16 / elem_size(dt);
    const int nch = (s.K + ce - 1) / ce;
    f.ksplit = nch > 128 ? 4 : 1;                               // more than one trip of 128 chunks per row
    const int rpb = f.ksplit == 4 ? RW : 4 * RW;
    f.row_units = rc_ready ? (s.M + 255) / 256 : (s.M + rpb - 1) / rpb;
    f.col_units = s.transB ? (s.N + rpb - 1) / rpb : (s.N + CHK_KN_LANES * ce - 1) / (CHK_KN_LANES * ce);
    const long units = ((long)f.row_units + f.col_units + 1) * s.batch;
    if (units > 0x7FFFFFFFL) return hipErrorInvalidValue;
    const unsigned gx = (unsigned)(units < MAX_GRID_X ? units : MAX_GRID_X);
    f.grid_x = gx;
    const dim3 grid(gx, (unsigned)((units + gx - 1) / gx), 1);
    switch (dt) {
    case DT_I8:   hipLaunchKernelGGL((check_kernel<DT_I8, RW>), grid, dim3(256), 0, st, f); break;
    case DT_BF16: hipLaunchKernelGGL((check_kernel<DT_BF16, RW>), grid, dim3(256), 0, st, f); break;
    case DT_F16:  hipLaunchKernelGGL((check_kernel<DT_F16, RW>), grid, dim3(256), 0, st, f); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ================================================================= discrepancy
// Statistics of d = observed - predicted over the rows and over the columns of one GEMM: what
// the paper's "Eps Generation" (Sec. III-B.1) fits its thresholds to.  One block per batch
// item; out[bz] = { sum d, sum d^2, max|d|, count } for the rows, then the same for the columns.
struct DiscArgs {
    const uint32_t *cc_pred, *rc_pred, *cc_src, *rc_src;
    int M, N;
    float *out;           // [batch][8]
};

__global__ __launch_bounds__(256) void discrepancy_kernel(DiscArgs a)
{
    __shared__ float red[4][3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, bz = blockIdx.x;
    for (int side = 0; side < 2; ++side) {
        const int n = side == 0 ? a.M : a.N;
        const uint32_t *src = (side == 0 ? a.rc_src : a.cc_src) + (long)bz * n;
        const uint32_t *pred = (side == 0 ? a.rc_pred : a.cc_pred) + (long)bz * n;
        float s = 0.f, s2 = 0.f, mx = 0.f;
        for (int i = tid; i < n; i += 256) {
            const float dd = __uint_as_float(src[i]) - __uint_as_float(pred[i]);
            s += dd;
            s2 = __builtin_fmaf(dd, dd, s2);
            mx = fmaxf(mx, fabsf(dd));
        }
        s = wave_sum(s);
        s2 = wave_sum(s2);
        mx = wave_max(mx);
        __syncthreads();
        if (lane == 0) { red[wave][0] = s; red[wave][1] = s2; red[wave][2] = mx; }
        __syncthreads();
        if (tid == 0) {
            float *o = a.out + (long)bz * 8 + side * 4;
            o[0] = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
            o[1] = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
            o[2] = fmaxf(fmaxf(red[0][2], red[1][2]), fmaxf(red[2][2], red[3][2]));
            o[3] = (float)n;
        }
    }
}

hipError_t launch_discrepancy(const Shape &s, const Workspace &w, bool stored, float *out, hipStream_t st)
{
    DiscArgs a;
    a.cc_pred = w.cc_pred; a.rc_pred = w.rc_pred;
    a.cc_src = stored ? w.cc_vobs : w.cc_obs;
    a.rc_src = stored ? w.rc_vobs : w.rc_obs;
    a.M = s.M; a.N = s.N; a.out = out;
    hipLaunchKernelGGL(discrepancy_kernel, dim3((unsigned)s.batch), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ====================================================================== verify
// Column and row sums of the stored C (streaming reduction, HBM-bound).
struct VerArgs {
    const uint8_t *C;
    long ldc, sC;
    int M, N;
    int cw_log2, rpb, nwin, nrb;
    uint32_t *cc_vobs, *rc_vobs;
    const uint32_t *gate; // non-null: nothing to do if *gate == 0 (no tile was recomputed: C is as it was checked)
    uint32_t *counts;     // non-null: cleared for the compare kernel
};

// value q of a 16-byte chunk of stored C
template <int DT> __device__ __forceinline__ typename Traits<DT>::acc_t out_elem(const i32x4 &v, int q)
{
    if (DT == DT_I8) return from_word<typename Traits<DT>::acc_t>((uint32_t)v[q]);
    uint32_t w = (uint32_t)v[q >> 1];
    uint32_t h = (q & 1) ? (w >> 16) : (w & 0xFFFFu);
    if (DT == DT_BF16) return from_word<typename Traits<DT>::acc_t>(h << 16);
    return from_word<typename Traits<DT>::acc_t>(__float_as_uint(f16_bits_to_f32(h)));
}

template <int DT>
__global__ __launch_bounds__(256) void verify_kernel(VerArgs a)
{
    fetch_args<VerArgs>();
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int OS = T::OS, CE = 16 / OS;
    __shared__ acc_t red[256 * CE];
    const int tid = threadIdx.x, bz = blockIdx.z;
    if (a.gate && *a.gate == 0u) return;
    if (a.counts && blockIdx.x == 0 && bz == 0 && tid < 5) a.counts[tid] = 0u;
    const int win = blockIdx.x % a.nwin, rb = blockIdx.x / a.nwin;
    const int CW = 1 << a.cw_log2, RL = 256 >> a.cw_log2;
    const int cx = tid & (CW - 1), ry = tid >> a.cw_log2;
    const int col0 = (win * CW + cx) * CE;
    const bool colok = col0 < a.N;
    const int nvalid = a.N - col0;
    const uint8_t *Cb = a.C + (long)bz * a.sC * OS;
    const int rbeg = rb * a.rpb, rend = min(rbeg + a.rpb, a.M);
    acc_t colacc[CE];
#pragma unroll
    for (int q = 0; q < CE; ++q) colacc[q] = T::zero();
    // A thread takes UN consecutive rows at a time: their sums meet in eight lanes, which add sixteen neighbouring
    // words in two atomics (a row at a time, one lane each, the row sums were most of the pass).
    constexpr int UN = ENC_UNROLL_ALONE;
    const uint8_t *src = Cb + (colok ? (long)col0 * OS : 0);
    for (int r0 = rbeg; r0 < rend; r0 += RL * UN) {
        const int rt = r0 + ry * UN;
        i32x4 v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u)                             // past the end: the last row, cleared below
            v[u] = *reinterpret_cast<const i32x4 *>(src + (long)min(rt + u, a.M - 1) * a.ldc * OS);
        acc_t part[CE], m0 = T::zero(), m1 = T::zero();
#pragma unroll
        for (int q = 0; q < CE; ++q) part[q] = T::zero();
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            i32x4 w = v[u];
            if (!colok || rt + u >= rend) w = i32x4{0, 0, 0, 0};
            else if (nvalid < CE) w = mask_chunk(w, nvalid * OS);
            acc_t s = T::zero();
#pragma unroll
            for (int q = 0; q < CE; ++q) {
                const acc_t x = out_elem<DT>(w, q);
                part[q] = add_t(part[q], x);
                s = add_t(s, x);
            }
            s = seg_sum(s, CW);
            if (cx == (u & 7)) { if (u < 8) m0 = s; else m1 = s; }
        }
#pragma unroll
        for (int q = 0; q < CE; ++q) colacc[q] = add_t(colacc[q], part[q]);
        if (cx < 8) {
            uint32_t *d = a.rc_vobs + (long)bz * a.M + rt + cx;
            if (rt + cx < rend) atomic_add_word(d, m0);
            if (rt + cx + 8 < rend) atomic_add_word(d + 8, m1);
        }
    }
#pragma unroll
    for (int q = 0; q < CE; ++q) red[(ry * CW + cx) * CE + q] = colacc[q];
    __syncthreads();
    for (int c = tid; c < CW * CE; c += 256) {
        const int col = win * CW * CE + c;
        if (col < a.N) {
            acc_t t = red[c];
            for (int y = 1; y < RL; ++y) t = add_t(t, red[y * CW * CE + c]);
            atomic_add_word(a.cc_vobs + (long)bz * a.N + col, t);
        }
    }
}

hipError_t launch_verify_sums(int dt, const void *C, const Shape &s, const Workspace &w, uint32_t *counts, hipStream_t st, bool gated)
{
    VerArgs a;
    a.counts = counts;
    a.gate = gated ? w.fix_count : nullptr;
    a.C = (const uint8_t *)C; a.ldc = s.ldc; a.sC = s.sC; a.M = s.M; a.N = s.N;
    a.cc_vobs = w.cc_vobs; a.rc_vobs = w.rc_vobs;
    const EncPlan plan = plan_alone(s.M, s.N, 16 / out_size(dt));
    a.cw_log2 = plan.cw_log2; a.nwin = plan.nwin; a.rpb = plan.rpb; a.nrb = plan.nrb;
    dim3 grid((unsigned)(a.nwin * a.nrb), 1, (unsigned)s.batch);
    switch (dt) {
    case DT_I8:   hipLaunchKernelGGL(verify_kernel<DT_I8>, grid, dim3(256), 0, st, a); break;
    case DT_BF16: hipLaunchKernelGGL(verify_kernel<DT_BF16>, grid, dim3(256), 0, st, a); break;
    case DT_F16:  hipLaunchKernelGGL(verify_kernel<DT_F16>, grid, dim3(256), 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ===================================================================== correct
// Step 1: list flagged rows / columns per batch item, map their cross product to CT x CT tiles.
struct LocArgs {
    const uint8_t *row_flag, *col_flag;
    int M, N;
    int32_t *fix_tiles;
    uint32_t *fix_count;
};

constexpr int LOC_THREADS = 1024;

// note(i) for every non-zero byte i of flag[0..n), by NT threads.  Sixteen flags per load where the address allows: flags are almost
// all zero, and the scan is bound by the latency of its loads.
template <int NT, typename NOTE> __device__ __forceinline__ void scan_flags(const uint8_t *flag, int n, int tid, NOTE &&note)
{
    const int head = min(n, (int)((16u - (unsigned)((uintptr_t)flag & 15u)) & 15u));
    const int nchunk = (n - head) / 16;
    const int tail0 = head + nchunk * 16;
    if (tid < head && flag[tid]) note(tid);
    if (tid < n - tail0 && flag[tail0 + tid]) note(tail0 + tid);
    const i32x4 *body = reinterpret_cast<const i32x4 *>(flag + head);
    for (int c0 = 0; c0 < nchunk; c0 += 4 * NT) {
        i32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * NT + tid;
            v[u] = i32x4{0, 0, 0, 0};
            if (c < nchunk) v[u] = body[c];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if ((v[u][0] | v[u][1] | v[u][2] | v[u][3]) == 0) continue;
            const int c = c0 + u * NT + tid;
#pragma unroll 1
            for (int q = 0; q < 16; ++q) {
                const unsigned w = (unsigned)(q < 8 ? q < 4 ? v[u][0] : v[u][1] : q < 12 ? v[u][2] : v[u][3]);
                if ((w >> (8 * (q & 3))) & 0xFFu) note(head + c * 16 + q);
            }
        }
    }
}
// Appends the CT-tile index of every flagged entry to list (at most MAX_LIST kept; *count keeps counting).
__device__ inline void list_flagged(const uint8_t *flag, int n, int *list, int *count, int tid)
{
    scan_flags<LOC_THREADS>(flag, n, tid, [&](int i) {
        int p = atomicAdd(count, 1);
        if (p < MAX_LIST) list[p] = i / CT;
    });
}

__global__ __launch_bounds__(LOC_THREADS) void locate_kernel(LocArgs a)
{
    __shared__ int rows[MAX_LIST], cols[MAX_LIST];
    __shared__ int nr, nc;
    const int bz = blockIdx.x, tid = threadIdx.x;
    if (tid == 0) { nr = 0; nc = 0; }
    __syncthreads();
    list_flagged(a.row_flag + (long)bz * a.M, a.M, rows, &nr, tid);
    list_flagged(a.col_flag + (long)bz * a.N, a.N, cols, &nc, tid);
    __syncthreads();
    if (tid != 0) return;
    if (nr == 0 || nc == 0) return;                     // clean, or one-sided: nothing to recompute
    bool overflow = nr > MAX_LIST || nc > MAX_LIST;
    int r = nr > MAX_LIST ? MAX_LIST : nr, c = nc > MAX_LIST ? MAX_LIST : nc;
    // unique tile rows / tile cols (lists are short under the single-error model)
    int ur = 0, uc = 0;
    for (int i = 0; i < r; ++i) {
        bool dup = false;
        for (int q = 0; q < ur; ++q) dup |= (rows[q] == rows[i]);
        if (!dup) rows[ur++] = rows[i];
    }
    for (int j = 0; j < c; ++j) {
        bool dup = false;
        for (int q = 0; q < uc; ++q) dup |= (cols[q] == cols[j]);
        if (!dup) cols[uc++] = cols[j];
    }
    for (int i = 0; i < ur; ++i)
        for (int j = 0; j < uc; ++j) {
            unsigned p = atomicAdd(a.fix_count, 1u);
            if (p < (unsigned)MAX_FIX_TILES) {
                a.fix_tiles[3 * p + 0] = bz;
                a.fix_tiles[3 * p + 1] = rows[i];
                a.fix_tiles[3 * p + 2] = cols[j];
            } else overflow = true;
        }
    if (overflow) atomicExch(a.fix_count + 1, 1u);
}

// Step 2, many tiles: one workgroup recomputes one CT x CT tile of C over the whole K.  Its first wave issues
// every MFMA, the same instruction in the same ascending-k order as the GEMM kernel, so a
// floating-point tile comes back with the bits the GEMM produced.  What bounds the step is the
// latency of the operand loads (a wave keeps 2 * FIX_UB 16-byte loads per lane in flight), so
// FIX_WAVES further waves load, each a different run of FIX_UB k-steps, and hand the operands to
// the first wave through LDS, in the lane layout they are consumed in; while it works through one
// group of runs the loads of the next group are in flight.
constexpr int FIX_WAVES = 8;                    // waves that load (the workgroup has one more)
constexpr int FIX_UB = 8;                       // k-steps a wave loads per group
constexpr size_t FIX_LDS_BYTES = (size_t)FIX_WAVES * FIX_UB * 2 * 64 * 16;

struct FixArgs {
    const uint8_t *A, *B;
    uint8_t *C;
    int M, N, K, transB;
    long lda, ldb, ldc, sA, sB, sC;
    int32_t *fix_tiles;
    uint32_t *fix_count;
    uint32_t *cc_vobs;      // non-null: the re-summed column sums of the tile's columns are cleared (they are
                            // accumulated again by resum_touched_kernel)
    const uint32_t *bias;   // layer bias [N] or null
    const uint8_t *row_flag, *col_flag;      // FIND: where the tiles are found
};

// Few tiles: sixteen workgroups share a tile, 8 x 8 elements each.  A compute unit takes in some 27 GB/s of rows that are a few
// whole lines each, and a tile's operands are 64 rows; a part's are sixteen, and eight lanes read 128 bytes of one, where a
// fragment's lanes read 32.  The MFMAs are the same, in the same order, on rows and columns repeated four times over: an
// element's bits depend on its own row and column only.  (Of integers the order does not matter: four waves take a quarter each.)
// int8 6304 x 768 x 3072: a launch 10.2 us and 3.3 for the list ahead of it, 8.3 with the search in it; flip, verify and repair 30.4 -> 24.8, f16 37.6 ->
// 27.7.
constexpr int FIX_PARTS = 16, FIX_PART = 8;     // parts of a tile, rows and columns of one
constexpr int FIX_GROUP = FIX_WAVES * 8;        // slabs in LDS at a time: 512 bytes for each step of 32 bytes of K
static_assert(FIX_GROUP * 4 * 512 == FIX_LDS_BYTES, "the parts' steps fill what a whole tile's run takes");
template <int DT>
__device__ __forceinline__ void recompute_part(const FixArgs &a, uint8_t *lds, int bz, int tr, int tc, int part)
{
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int ES = T::ES, KE = SLAB_BYTES / ES;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, lh = lane >> 5;
    const int row0 = tr * CT + (part >> 2) * FIX_PART, col0 = tc * CT + (part & 3) * FIX_PART;
    const int kbytes = a.K * ES, slabs = (kbytes + SLAB_BYTES - 1) / SLAB_BYTES, lw = wave - 1;
    const uint8_t *Ab = a.A + (long)bz * a.sA * ES, *Bb = a.B + (long)bz * a.sB * ES;
    if (a.cc_vobs && part < 4 && threadIdx.x < FIX_PART && col0 + (int)threadIdx.x < a.N) a.cc_vobs[(long)bz * a.N + col0 + threadIdx.x] = 0u;
    // a lane's place in a slab: row lane >> 3 of the part, chunk lane & 7; in LDS step 4 slab + (chunk >> 1)
    const int r8 = lane >> 3, ch = lane & 7, last_ch = (kbytes - 1) / 16 * 16;
    const uint8_t *pa = Ab + (long)min(row0 + r8, a.M - 1) * a.lda * ES, *pb = Bb + (long)min(col0 + r8, a.N - 1) * a.ldb * ES;
    const int at = (ch >> 1) * 512 + r8 * 32 + (ch & 1) * 16;
    // columns of a B stored K x N: a chunk holds all of the part's (past the end: the last whole chunk)
    const uint8_t *pk = Bb + min(col0, (a.N - 1) / FIX_PART * FIX_PART) * ES;
    // slabs s0 + FIX_WAVES u, u < U; what lies past the end of K is cleared
    auto stage = [&](auto u_c, int s0, int g0) __attribute__((always_inline)) {
        constexpr int U = decltype(u_c)::value;
        typedef int i32x2 __attribute__((ext_vector_type(2)));
        i32x4 x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + FIX_WAVES * u, kb = min(s * SLAB_BYTES + ch * 16, last_ch);
            x[u] = *reinterpret_cast<const i32x4 *>(pa + kb);
            if (a.transB) {
                y[u] = *reinterpret_cast<const i32x4 *>(pb + kb);
            } else if constexpr (ES == 2) {
                y[u] = *reinterpret_cast<const i32x4 *>(pk + (long)min(s * KE + lane, a.K - 1) * a.ldb * ES);
            } else {
                const i32x2 lo = *reinterpret_cast<const i32x2 *>(pk + (long)min(s * KE + 2 * lane, a.K - 1) * a.ldb);
                const i32x2 hi = *reinterpret_cast<const i32x2 *>(pk + (long)min(s * KE + 2 * lane + 1, a.K - 1) * a.ldb);
                y[u] = i32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + FIX_WAVES * u;
            if (s >= slabs) break;
            uint8_t *d = lds + (s - g0) * 4 * 512;
            const int keep = kbytes - (s * SLAB_BYTES + ch * 16);
            if ((s + 1) * SLAB_BYTES > kbytes) {
                x[u] = mask_chunk(x[u], keep);
                if (a.transB) y[u] = mask_chunk(y[u], keep);
            }
            *reinterpret_cast<i32x4 *>(d + at) = x[u];
            if (a.transB) {
                *reinterpret_cast<i32x4 *>(d + at + 256) = y[u];
            } else {
                // element (k, column c) goes to row c of the step that holds k
#pragma unroll
                for (int e = 0; e < 16 / ES; ++e) {
                    const int k = ES == 2 ? lane : 2 * lane + (e >> 3), c = e & 7;
                    const unsigned bits = (unsigned)y[u][e * ES / 4] >> (8 * ES * (e % (4 / ES)));
                    uint8_t *to = d + (k * ES >> 5) * 512 + 256 + c * 32 + (k * ES & 31);
                    const bool in = s * KE + k < a.K;
                    if constexpr (ES == 2) *reinterpret_cast<uint16_t *>(to) = in ? (uint16_t)bits : 0;
                    else *to = in ? (uint8_t)bits : 0;
                }
            }
        }
    };
    typename T::accv_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = T::zero();
    for (int g0 = 0; g0 < slabs; g0 += FIX_GROUP) {
        if (g0) __syncthreads();
        if (lw >= 0) {
            if (slabs - g0 <= 4 * FIX_WAVES) stage(std::integral_constant<int, 4>{}, g0 + lw, g0);
            else stage(std::integral_constant<int, 8>{}, g0 + lw, g0);
        }
        __syncthreads();
        // whole runs of eight steps (of those past the end of K, which hold nothing, only slabs that hold something are read)
        const int steps = min(FIX_GROUP, slabs - g0) * 4;
        const int share = T::IS_INT ? ((steps + 15) / 16) * 4 : steps, first = T::IS_INT ? wave * share : 0, end = min(steps, first + share);
        if (wave < (T::IS_INT ? 4 : 1)) {
            const uint8_t *src = lds + (l32 & 7) * 32 + lh * 16;
            constexpr int RU = 4;
            i32x4 x0[RU], y0[RU], x1[RU], y1[RU];
            auto read = [&](int t, i32x4 (&x)[RU], i32x4 (&y)[RU]) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < RU; ++u) {
                    x[u] = *reinterpret_cast<const i32x4 *>(src + (t + u) * 512);
                    y[u] = *reinterpret_cast<const i32x4 *>(src + (t + u) * 512 + 256);
                }
            };
            if (first < end) read(first, x0, y0);
            for (int t = first; t < end; t += 2 * RU) {
                if (t + RU < end) read(t + RU, x1, y1);
#pragma unroll
                for (int u = 0; u < RU; ++u) acc = T::mfma(y0[u], x0[u], acc);   // B first: lane = row of C, registers = columns
                if (t + RU < end) {
                    if (t + 2 * RU < end) read(t + 2 * RU, x0, y0);
#pragma unroll
                    for (int u = 0; u < RU; ++u) acc = T::mfma(y1[u], x1[u], acc);
                }
            }
        }
    }
    // rows 0..7 of the block are the part's rows, columns 0..7 its columns: register i < 4, column 4 (lane >> 5) + i
    acc_t v[4] = {(acc_t)acc[0], (acc_t)acc[1], (acc_t)acc[2], (acc_t)acc[3]};
    if constexpr (T::IS_INT) {
        __syncthreads();                                        // every wave has read its steps
        i32x4 *meet = reinterpret_cast<i32x4 *>(lds);
        if (wave > 0 && wave < 4 && l32 < FIX_PART) meet[(wave * 2 + lh) * FIX_PART + l32] = i32x4{v[0], v[1], v[2], v[3]};
        __syncthreads();
        if (wave == 0 && l32 < FIX_PART) {
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const i32x4 o = meet[(w * 2 + lh) * FIX_PART + l32];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += o[e];
            }
        }
    }
    if (wave != 0 || l32 >= FIX_PART || row0 + l32 >= a.M) return;
    uint8_t *Cb = a.C + (long)bz * a.sC * T::OS;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int gc = col0 + 4 * lh + e;
        if (gc < a.N) T::store_c(Cb, (long)(row0 + l32) * a.ldc + gc, a.bias ? add_t(v[e], from_word<acc_t>(a.bias[gc])) : v[e]);
    }
}

// FIND: the tiles of a single problem, found by every workgroup for itself from the flags (at most FIND_FLAGS of them: a load or
// four to a thread), which saves the launch that lists them: what that writes is read a trip to memory later.  The tile rows and tile columns with a
// flag, in ascending order, so that all workgroups agree; the first one also leaves the list for the kernels behind.
constexpr int FIND_FLAGS = 32768;
struct FoundTiles {
    int flagged[2], unique[2];                  // rows, columns; tile rows, tile columns
    uint32_t bits[2][FIND_FLAGS / CT / 32];
    int tile[2][MAX_LIST];
};
__device__ __forceinline__ unsigned find_tiles(const FixArgs &a, FoundTiles *f)
{
    constexpr int NT = 64 * (FIX_WAVES + 1);
    const int tid = threadIdx.x;
    for (int i = tid; i < (int)(offsetof(FoundTiles, tile) / 4); i += NT) reinterpret_cast<uint32_t *>(f)[i] = 0u;
    __syncthreads();
    auto note = [&](int side, int i) {
        atomicAdd(&f->flagged[side], 1);
        const int t = i / CT;
        if (!(atomicOr(&f->bits[side][t >> 5], 1u << (t & 31)) >> (t & 31) & 1u)) {
            const int p = atomicAdd(&f->unique[side], 1);
            if (p < MAX_LIST) f->tile[side][p] = t;
        }
    };
    scan_flags<NT>(a.row_flag, a.M, tid, [&](int i) { note(0, i); });
    scan_flags<NT>(a.col_flag, a.N, tid, [&](int i) { note(1, i); });
    __syncthreads();
    const int nr = f->flagged[0], nc = f->flagged[1], ur = f->unique[0], uc = f->unique[1];
    unsigned n = 0;
    bool overflow = false;
    if (nr && nc) {
        // in ascending order; of more than are kept, the first ones
        int mine = 0, rank = 0;
        const int side = tid / MAX_LIST, i = tid % MAX_LIST, count = side == 0 ? ur : uc;
        const bool sorts = side < 2 && count <= MAX_LIST && i < count;
        if (sorts) {
            mine = f->tile[side][i];
            for (int q = 0; q < count; ++q) rank += f->tile[side][q] < mine ? 1 : 0;
        }
        __syncthreads();
        if (sorts) f->tile[side][rank] = mine;
        else if (side < 2 && i == 0 && count > MAX_LIST) {
            int p = 0;
            for (int t = 0; p < MAX_LIST; ++t)
                if (f->bits[side][t >> 5] >> (t & 31) & 1u) f->tile[side][p++] = t;
        }
        __syncthreads();
        const int kr = min(ur, MAX_LIST), kc = min(uc, MAX_LIST);
        n = (unsigned)(kr * kc);
        // (by tiles, not by flags: a hundred flagged columns of one row are four tiles or five, and all of them are recomputed)
        overflow = ur > MAX_LIST || uc > MAX_LIST || n > (unsigned)MAX_FIX_TILES;
        f->unique[0] = kr; f->unique[1] = kc;           // (every thread writes the same, and reads them behind the next barrier or itself)
    }
    if (blockIdx.x == 0) {
        if (tid == 0) { a.fix_count[0] = n; a.fix_count[1] = overflow ? 1u : 0u; }
        const int kc = min(uc, MAX_LIST);
        for (int t = tid; t < (int)min(n, (unsigned)MAX_FIX_TILES); t += NT) {
            a.fix_tiles[3 * t] = 0;
            a.fix_tiles[3 * t + 1] = f->tile[0][t / kc];
            a.fix_tiles[3 * t + 2] = f->tile[1][t % kc];
        }
    }
    return n;
}

template <int DT, bool FIND>
__global__ __launch_bounds__(64 * (FIX_WAVES + 1)) void recompute_kernel(FixArgs a)
{
    fetch_args<FixArgs>();
    using T = Traits<DT>;
    typedef typename T::accv_t accv_t;
    constexpr int ES = T::ES, CE = 16 / ES;
    constexpr int UB = FIX_UB;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    i32x4 *stage = reinterpret_cast<i32x4 *>(lds);          // [FIX_WAVES * UB k-steps][A, B][64 lanes]
    __shared__ FoundTiles found;
    unsigned n;
    if constexpr (FIND) n = find_tiles(a, &found);
    else n = a.fix_count[0];
    if (n > (unsigned)MAX_FIX_TILES) n = MAX_FIX_TILES;
    // the whole workgroup leaves, or takes a part of a tile, or a tile
    const bool parts = n * FIX_PARTS <= (unsigned)MAX_FIX_TILES;
    if (blockIdx.x >= (parts ? n * FIX_PARTS : n)) return;
    const int tile = __builtin_amdgcn_readfirstlane(parts ? blockIdx.x / FIX_PARTS : blockIdx.x);
    int bz = 0, tr, tc;
    if constexpr (FIND) {
        const int kc = found.unique[1];
        tr = __builtin_amdgcn_readfirstlane(found.tile[0][tile / kc]);
        tc = __builtin_amdgcn_readfirstlane(found.tile[1][tile % kc]);
    } else {
        bz = a.fix_tiles[3 * tile]; tr = a.fix_tiles[3 * tile + 1]; tc = a.fix_tiles[3 * tile + 2];
    }
    if (__builtin_expect(parts, 1)) {
        recompute_part<DT>(a, lds, bz, tr, tc, blockIdx.x % FIX_PARTS);
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5;
    const int row = tr * CT + l32, col = tc * CT + l32;
    const uint8_t *Ab = a.A + (long)bz * a.sA * ES, *Bb = a.B + (long)bz * a.sB * ES;
    const int K = a.K;
    if (a.cc_vobs && wave == 1 && lane < CT && col < a.N) a.cc_vobs[(long)bz * a.N + col] = 0u;
    accv_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = T::zero();
    const int steps = (K + 2 * CE - 1) / (2 * CE);
    // Loads without a branch: what lies past the end asks for the last row, column or chunk.  (Under a branch each, or masked at
    // once, every load is waited for before the next.)  Rows and columns past the end need no more: what they give is not
    // stored.  Past the end of K a run is cleared once all of it is under way, by masks that both operands share: this code runs
    // once per call, so its instructions come from memory and a long straight path costs what it saves.  (Flip, verify and
    // repair, with a branch per load / with masks for rows, columns and K of every tile at an edge / so: f16 318 x 41 x 3456 36.0 /
    // 37.7 / 33.3 us; bf16 231 x 310 x 3305 34.2 / 36.1 / 32.8.)
    const long rowc = min(row, a.M - 1), colc = min(col, a.N - 1);
    const int last_kb = (K - 1) / CE * CE;
    auto load_run = [&](int ks0, i32x4 (&av)[UB], i32x4 (&bv)[UB]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int kb = min((ks0 + u) * 2 * CE + lh * CE, last_kb);
            av[u] = *reinterpret_cast<const i32x4 *>(Ab + (rowc * a.lda + kb) * ES);
        }
        if (a.transB) {
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int kb = min((ks0 + u) * 2 * CE + lh * CE, last_kb);
                bv[u] = *reinterpret_cast<const i32x4 *>(Bb + (colc * a.ldb + kb) * ES);
            }
        } else {
            // B stored K x N: gather one column element per k, the elements of QU k-steps in flight
            constexpr int QU = ES == 2 ? UB / 2 : UB / 4;
#pragma unroll
            for (int u0 = 0; u0 < UB; u0 += QU) {
                uint32_t raw[QU][CE];
#pragma unroll
                for (int u = 0; u < QU; ++u)
#pragma unroll
                    for (int q = 0; q < CE; ++q) {
                        const long k = min((ks0 + u0 + u) * 2 * CE + lh * CE + q, K - 1);
                        const uint8_t *at = Bb + (k * a.ldb + colc) * ES;
                        if constexpr (ES == 2) raw[u][q] = *reinterpret_cast<const uint16_t *>(at);
                        else raw[u][q] = *at;
                    }
#pragma unroll
                for (int u = 0; u < QU; ++u)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        if constexpr (ES == 2) bv[u0 + u][w] = (int)(raw[u][2 * w] | raw[u][2 * w + 1] << 16);
                        else bv[u0 + u][w] = (int)(raw[u][4 * w] | raw[u][4 * w + 1] << 8 | raw[u][4 * w + 2] << 16 | raw[u][4 * w + 3] << 24);
                    }
            }
        }
    };
    // every wave takes the same number of trips: the barriers are reached by all
    for (int g0 = 0; g0 < steps; g0 += FIX_WAVES * UB) {
        const int lw = wave - 1;                            // loading wave 0 .. FIX_WAVES - 1
        const int ks0 = g0 + lw * UB;
        i32x4 av[UB], bv[UB];
        const bool loads = wave != 0 && ks0 < steps;
        if (loads) {
            // The straight path stands first: laid out behind the other one, its instructions are another trip to memory
            // (int8 6304 x 768 x 3072: kernel 11.5 us, 10.7 so)
            const bool whole = (ks0 + UB) * 2 * CE <= K;
            if (__builtin_expect(a.transB && whole, 1)) {
                const uint8_t *pa = Ab + (rowc * a.lda + ks0 * 2 * CE + lh * CE) * ES;
                const uint8_t *pb = Bb + (colc * a.ldb + ks0 * 2 * CE + lh * CE) * ES;
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    av[u] = *reinterpret_cast<const i32x4 *>(pa + 32 * u);
                    bv[u] = *reinterpret_cast<const i32x4 *>(pb + 32 * u);
                }
            } else {
                load_run(ks0, av, bv);
                if (!whole) {
                    // (the mask of the last chunk is formed here: hoisted, it comes ahead of every call's loads)
                    int left = (K - last_kb) * ES;
                    asm volatile("" : "+s"(left));
                    const i32x4 last_mask = mask_chunk(i32x4{-1, -1, -1, -1}, left);
#pragma unroll
                    for (int u = 0; u < UB; ++u) {
                        const int kb = (ks0 + u) * 2 * CE + lh * CE;
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            const int keep = kb < last_kb ? -1 : kb == last_kb ? last_mask[w] : 0;
                            av[u][w] &= keep;
                            bv[u][w] &= keep;
                        }
                    }
                }
            }
        }
        __syncthreads();                                    // the first wave is done with the previous group
        if (loads) {
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                stage[((lw * UB + u) * 2 + 0) * 64 + lane] = av[u];
                stage[((lw * UB + u) * 2 + 1) * 64 + lane] = bv[u];
            }
        }
        __syncthreads();
        if (wave == 0) {
            // whole runs of UB k-steps (a run's k-steps past the end of K hold zeros and add nothing);
            // the operands of the next run are read while the chain of dependent MFMAs of this one runs
            const int nrun = min(FIX_WAVES, (steps - g0 + UB - 1) / UB);
            auto read_run = [&](int r, i32x4 (&x)[UB], i32x4 (&y)[UB]) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    x[u] = stage[((r * UB + u) * 2 + 0) * 64 + lane];
                    y[u] = stage[((r * UB + u) * 2 + 1) * 64 + lane];
                }
            };
            i32x4 x0[UB], y0[UB], x1[UB], y1[UB];
            read_run(0, x0, y0);
            for (int r = 0; r < nrun; r += 2) {
                read_run(min(r + 1, FIX_WAVES - 1), x1, y1);
#pragma unroll
                for (int u = 0; u < UB; ++u) acc = T::mfma(y0[u], x0[u], acc);   // B first: lane = row of C, registers = columns
                if (r + 1 < nrun) {
                    read_run(min(r + 2, FIX_WAVES - 1), x0, y0);
#pragma unroll
                    for (int u = 0; u < UB; ++u) acc = T::mfma(y1[u], x1[u], acc);
                }
            }
        }
    }
    if (wave != 0) return;
    uint8_t *Cb = a.C + (long)bz * a.sC * T::OS;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int gc = tc * CT + 8 * (i >> 2) + 4 * lh + (i & 3);
        if (row < a.M && gc < a.N) {
            typename T::acc_t v = acc[i];
            if (a.bias) v = add_t(v, from_word<typename T::acc_t>(a.bias[gc]));
            T::store_c(Cb, (long)row * a.ldc + gc, v);
        }
    }
}

// Step 3 when the sums of the stored C are at hand (abft_verify ran on this C): only the rows and
// the columns of the recomputed tiles changed, so only their sums are formed again.  Workgroup
// (t, p) serves listed tile t: p < CT sums row p of the tile over all N and stores it; every p sums
// the tile's CT columns over its share of the M rows and adds that to the column sums, which
// recompute_kernel has cleared.  A tile row or tile column listed more than once is summed by
// its first tile only.
constexpr int TOUCH_PARTS = 64;
constexpr int TOUCH_TILES = 8;           // workgroups per part: listed tiles served at a time

struct TouchArgs {
    const uint8_t *C;
    long ldc, sC;
    int M, N;
    const int32_t *fix_tiles;
    const uint32_t *fix_count;
    uint32_t *cc_vobs, *rc_vobs;
    uint32_t *counts;       // non-null: made ready for a compare without a ticket
};

template <int DT>
__global__ __launch_bounds__(256) void resum_touched_kernel(TouchArgs a)
{
    fetch_args<TouchArgs>();
    using T = Traits<DT>;
    typedef typename T::acc_t acc_t;
    constexpr int OS = T::OS, CE = 16 / OS;
    constexpr int CPR = CT / CE;                            // 16-byte chunks across a tile
    constexpr int RL = 256 / CPR;                           // rows a pass of the workgroup covers
    __shared__ acc_t red[256 * CE];
    unsigned n = a.fix_count[0];
    if (n > (unsigned)MAX_FIX_TILES) n = MAX_FIX_TILES;
    const int part = blockIdx.y, tid = threadIdx.x;
    if (a.counts && blockIdx.x == 0 && part == TOUCH_PARTS - 1 && tid == 0) {
        const uint32_t before = a.counts[2];
        a.counts[0] = 0u;
        a.counts[1] = 0u;
        a.counts[2] = a.fix_count[1] ? 3u : 0u;
        a.counts[3] = n;
        a.counts[4] = before;
    }
    // the grid has TOUCH_TILES workgroups per part; listed tiles beyond that many take further trips
    for (int t = blockIdx.x; t < (int)n; t += gridDim.x) {
        const int bz = a.fix_tiles[3 * t], tr = a.fix_tiles[3 * t + 1], tc = a.fix_tiles[3 * t + 2];
        bool first_row = true, first_col = true;
        for (int q = 0; q < t; ++q)
            if (a.fix_tiles[3 * q] == bz) {
                first_row = first_row && a.fix_tiles[3 * q + 1] != tr;
                first_col = first_col && a.fix_tiles[3 * q + 2] != tc;
            }
        const uint8_t *Cb = a.C + (long)bz * a.sC * OS;
        const int M = a.M, N = a.N;

        const int row = tr * CT + part;
        if (first_row && part < CT && row < M) {
            acc_t s = T::zero();
            const int nch = (N + CE - 1) / CE;
            for (int c = tid; c < nch; c += 256) {
                const i32x4 v = *reinterpret_cast<const i32x4 *>(Cb + ((long)row * a.ldc + (long)c * CE) * OS);
                const int nvalid = N - c * CE;
#pragma unroll
                for (int q = 0; q < CE; ++q)
                    if (q < nvalid) s = add_t(s, out_elem<DT>(v, q));
            }
            s = wave_sum(s);
            if ((tid & 63) == 0) red[tid >> 6] = s;
            __syncthreads();
            if (tid == 0) a.rc_vobs[(long)bz * M + row] = as_word(add_t(add_t(red[0], red[1]), add_t(red[2], red[3])));
            __syncthreads();                                    // red is used again below
        }
        if (!first_col) continue;

        const int mc = (M + TOUCH_PARTS - 1) / TOUCH_PARTS;
        const int rbeg = part * mc, rend = min(rbeg + mc, M);
        const int cx = tid % CPR, ry = tid / CPR;
        const int col0 = tc * CT + cx * CE;
        const int nvalid = N - col0;
        acc_t colacc[CE];
#pragma unroll
        for (int q = 0; q < CE; ++q) colacc[q] = T::zero();
        for (int r0 = rbeg + ry; r0 < rend; r0 += RL * ENC_UNROLL) {
            i32x4 v[ENC_UNROLL];
#pragma unroll
            for (int u = 0; u < ENC_UNROLL; ++u) {
                const int r = r0 + u * RL;
                v[u] = i32x4{0, 0, 0, 0};
                if (nvalid > 0 && r < rend) v[u] = *reinterpret_cast<const i32x4 *>(Cb + ((long)r * a.ldc + col0) * OS);
            }
#pragma unroll
            for (int u = 0; u < ENC_UNROLL; ++u) {
                if (r0 + u * RL < rend) {
#pragma unroll
                    for (int q = 0; q < CE; ++q)
                        if (q < nvalid) colacc[q] = add_t(colacc[q], out_elem<DT>(v[u], q));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < CE; ++q) red[ry * CT + cx * CE + q] = colacc[q];
        __syncthreads();
        if (tid < CT) {
            const int col = tc * CT + tid;
            if (col < N && rbeg < rend) {
                acc_t s = red[tid];
                for (int y = 1; y < RL; ++y) s = add_t(s, red[y * CT + tid]);
                atomic_add_word(a.cc_vobs + (long)bz * N + col, s);
            }
        }
        __syncthreads();                                        // red is free for the next tile
    }
}

template <int DT>
static hipError_t launch_recompute(const FixArgs &f, hipStream_t st)
{
    auto kern = f.row_flag ? recompute_kernel<DT, true> : recompute_kernel<DT, false>;
    hipError_t e = ensure_max_lds(reinterpret_cast<const void *>(kern), (int)FIX_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(MAX_FIX_TILES), dim3(64 * (FIX_WAVES + 1)), FIX_LDS_BYTES, st, f);
    return hipGetLastError();
}

// One problem of not too many flags: the recompute finds its tiles itself, and leaves their list behind.
bool correct_finds(const Shape &s) { return s.batch == 1 && s.M + s.N <= FIND_FLAGS; }

hipError_t launch_correct(int dt, const void *A, const void *B, void *C, const Shape &s,
                          const Workspace &w, const Verdict &v, bool with_sto, bool clear_list, bool targeted,
                          size_t stale_words, uint32_t *zero_ptr, size_t zero_words, hipStream_t st, bool skip_if_clean)
{
    hipError_t e = hipSuccess;
    const bool find = correct_finds(s);
    if (!find) {
        if (clear_list && (e = launch_zero(w.fix_count, 2, st)) != hipSuccess) return e;
        LocArgs l;
        l.row_flag = v.row_flag; l.col_flag = v.col_flag; l.M = s.M; l.N = s.N;
        l.fix_tiles = w.fix_tiles; l.fix_count = w.fix_count;
        hipLaunchKernelGGL(locate_kernel, dim3((unsigned)s.batch), dim3(LOC_THREADS), 0, st, l);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }

    FixArgs f;
    f.row_flag = find ? v.row_flag : nullptr; f.col_flag = find ? v.col_flag : nullptr;
    f.A = (const uint8_t *)A; f.B = (const uint8_t *)B; f.C = (uint8_t *)C;
    f.M = s.M; f.N = s.N; f.K = s.K; f.transB = s.transB;
    f.lda = s.lda; f.ldb = s.ldb; f.ldc = s.ldc; f.sA = s.sA; f.sB = s.sB; f.sC = s.sC;
    f.fix_tiles = w.fix_tiles; f.fix_count = w.fix_count;
    f.cc_vobs = targeted ? w.cc_vobs : nullptr;
    f.bias = w.bias;
    switch (dt) {
    case DT_I8:   e = launch_recompute<DT_I8>(f, st); break;
    case DT_BF16: e = launch_recompute<DT_BF16>(f, st); break;
    case DT_F16:  e = launch_recompute<DT_F16>(f, st); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if (targeted) {
        TouchArgs t;
        t.C = (const uint8_t *)C; t.ldc = s.ldc; t.sC = s.sC; t.M = s.M; t.N = s.N;
        t.fix_tiles = w.fix_tiles; t.fix_count = w.fix_count; t.cc_vobs = w.cc_vobs; t.rc_vobs = w.rc_vobs;
        t.counts = find ? v.counts : nullptr;
        const dim3 grid(TOUCH_TILES, TOUCH_PARTS);
        switch (dt) {
        case DT_I8:   hipLaunchKernelGGL(resum_touched_kernel<DT_I8>, grid, dim3(256), 0, st, t); break;
        case DT_BF16: hipLaunchKernelGGL(resum_touched_kernel<DT_BF16>, grid, dim3(256), 0, st, t); break;
        default:      hipLaunchKernelGGL(resum_touched_kernel<DT_F16>, grid, dim3(256), 0, st, t); break;
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        return launch_compare(dt, s, w, v, true, with_sto, nullptr, 0, st, false, find);
    }
    // re-check without earlier sums of this C: the stored C is re-summed as a whole (a streaming
    // pass at HBM speed) and compared with the predictions
    if (stale_words && (e = launch_zero(w.cc_vobs, stale_words, st)) != hipSuccess) return e;
    if ((e = launch_verify_sums(dt, C, s, w, nullptr, st, skip_if_clean)) != hipSuccess) return e;
    return launch_compare(dt, s, w, v, true, with_sto, zero_ptr, zero_words, st, skip_if_clean);
}

// ====================================================================== checksum-only correction
// Integers: one block per batch item.  With exactly one flagged row i and one flagged column j
// whose discrepancies d (re-summed stored C minus prediction, in Z/2^32) agree, the corrupted
// element is C[i][j] and C[i][j] - d its value (the classic scheme of Sec. II-B; no operand is
// read, nothing is recomputed).  The re-summed vectors and the flags of the item are updated
// with it; any other pattern is left as it is.  The last block writes counts and status.
struct ArithArgs {
    uint8_t *row_flag, *col_flag;
    uint32_t *counts;
    uint32_t *ticket;            // [4]: ticket, flagged rows left, flagged cols left, elements fixed (self-cleaning)
    const uint32_t *cc_pred, *rc_pred;
    uint32_t *cc_vobs, *rc_vobs;
    uint32_t *C;
    long ldc, sC;
    int M, N;
};

__global__ __launch_bounds__(256) void arith_fix_kernel(ArithArgs a)
{
    __shared__ int nr, nc, ri, cj;
    const int bz = blockIdx.x, tid = threadIdx.x;
    if (tid == 0) { nr = 0; nc = 0; ri = 0; cj = 0; }
    __syncthreads();
    for (int i = tid; i < a.M; i += 256)
        if (a.row_flag[(long)bz * a.M + i]) { atomicAdd(&nr, 1); atomicMax(&ri, i); }
    for (int j = tid; j < a.N; j += 256)
        if (a.col_flag[(long)bz * a.N + j]) { atomicAdd(&nc, 1); atomicMax(&cj, j); }
    __syncthreads();
    if (tid != 0) return;
    uint32_t r = (uint32_t)nr, c = (uint32_t)nc, fixed = 0;
    if (r == 1 && c == 1) {
        const long ir = (long)bz * a.M + ri, jc = (long)bz * a.N + cj;
        const uint32_t dr = a.rc_vobs[ir] - a.rc_pred[ir], dc = a.cc_vobs[jc] - a.cc_pred[jc];
        if (dr == dc) {
            a.C[(long)bz * a.sC + (long)ri * a.ldc + cj] -= dr;
            a.rc_vobs[ir] -= dr;
            a.cc_vobs[jc] -= dc;
            a.row_flag[ir] = 0;
            a.col_flag[jc] = 0;
            r = 0; c = 0; fixed = 1;
        }
    }
    if (r) atomicAdd(a.ticket + 1, r);
    if (c) atomicAdd(a.ticket + 2, c);
    if (fixed) atomicAdd(a.ticket + 3, fixed);
    __threadfence();
    if (atomicAdd(a.ticket, 1u) == gridDim.x - 1) {
        const uint32_t rr = atomicExch(a.ticket + 1, 0u), cc = atomicExch(a.ticket + 2, 0u),
                       ff = atomicExch(a.ticket + 3, 0u);
        atomicExch(a.ticket, 0u);
        const uint32_t before = a.counts[2];
        a.counts[0] = rr;
        a.counts[1] = cc;
        a.counts[2] = status_of(rr, cc);
        a.counts[3] = ff;
        a.counts[4] = before;
    }
}

hipError_t launch_arith_fix(void *C, const Shape &s, const Workspace &w, const Verdict &v, hipStream_t st)
{
    ArithArgs a;
    a.row_flag = v.row_flag; a.col_flag = v.col_flag; a.counts = v.counts; a.ticket = w.cmp_ticket;
    a.cc_pred = w.cc_pred; a.rc_pred = w.rc_pred; a.cc_vobs = w.cc_vobs; a.rc_vobs = w.rc_vobs;
    a.C = (uint32_t *)C; a.ldc = s.ldc; a.sC = s.sC; a.M = s.M; a.N = s.N;
    hipLaunchKernelGGL(arith_fix_kernel, dim3((unsigned)s.batch), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ====================================================================== inject
__global__ void flip_kernel(uint8_t *C, long idx, int os, int bit)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    if (os == 4) {
        uint32_t *p = reinterpret_cast<uint32_t *>(C) + idx;
        *p ^= (1u << bit);
    } else if (os == 1) {
        C[idx] = (uint8_t)(C[idx] ^ (uint8_t)(1u << bit));
    } else {
        uint16_t *p = reinterpret_cast<uint16_t *>(C) + idx;
        *p = (uint16_t)(*p ^ (uint16_t)(1u << bit));
    }
}

hipError_t launch_flip_at(void *base, long idx, int elem_bytes, int bit, hipStream_t st)
{
    hipLaunchKernelGGL(flip_kernel, dim3(1), dim3(64), 0, st, (uint8_t *)base, idx, elem_bytes, bit);
    return hipGetLastError();
}

hipError_t launch_flip(void *C, int dt, const Shape &s, long batch_idx, long row, long col, int bit,
                       hipStream_t st)
{
    long idx = batch_idx * s.sC + row * s.ldc + col;
    hipLaunchKernelGGL(flip_kernel, dim3(1), dim3(64), 0, st, (uint8_t *)C, idx, out_size(dt), bit);
    return hipGetLastError();
}

// ====================================================================== report: matrix-pipe ceiling
// Nothing but matrix instructions, in the GEMM kernel's own shape: one wave per SIMD, sixteen
// independent 32 x 32 accumulators (all 256 accumulator registers), operands held in registers.
// What it reaches is the ceiling of the matrix pipe at the clock the chip sustains under that
// load; the fraction of it a GEMM kernel reaches says how well its loop feeds the pipe, apart
// from the clock.  Every wave also reads the shader clock counter and the constant 100 MHz
// counter around its loop, which gives the clock it ran at.
template <int DT>
__global__ __launch_bounds__(256) void mfma_peak_kernel(int iters, unsigned long long *clk, uint32_t *sink)
{
    using T = Traits<DT>;
    typedef typename T::accv_t accv_t;
    // Operands with the bit activity of real data: random signs and mantissas, magnitudes in
    // [1/128, 1), four different register sets taken in turn.  (With operands that never change
    // the matrix pipe toggles few bits, draws little power and keeps a clock no GEMM on real data
    // is granted.)
    uint32_t h = (uint32_t)(blockIdx.x * 256 + threadIdx.x) * 2654435761u + 12345u;
    auto next = [&]() __attribute__((always_inline)) -> int {
        h ^= h << 13; h ^= h >> 17; h ^= h << 5;
        uint32_t w = h;
        if (DT == DT_BF16) w = (w & 0x807F807Fu) | 0x3C003C00u | ((w >> 3) & 0x03800380u);
        if (DT == DT_F16) w = (w & 0x83FF83FFu) | 0x20002000u | ((w >> 3) & 0x1C001C00u);
        return (int)w;
    };
    i32x4 a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        a[q] = i32x4{next(), next(), next(), next()};
        b[q] = i32x4{next(), next(), next(), next()};
    }
    accv_t acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][i] = T::zero();
    const unsigned long long c0 = clock64(), w0 = wall_clock64();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = T::mfma(b[j & 3], a[(j >> 2) & 3], acc[j]);
    }
    const unsigned long long c1 = clock64(), w1 = wall_clock64();
    // keep the accumulators alive
    typename T::acc_t t = T::zero();
#pragma unroll
    for (int j = 0; j < 16; ++j) t = add_t(t, acc[j][j]);
    if (as_word(t) == 0x7FC12345u) sink[threadIdx.x] = as_word(t);
    if (threadIdx.x == 0) {
        clk[2 * blockIdx.x] = c1 - c0;
        clk[2 * blockIdx.x + 1] = w1 - w0;
    }
}

hipError_t launch_mfma_peak(int dt, int blocks, int iters, unsigned long long *clk, uint32_t *sink, hipStream_t st)
{
    switch (dt) {
    case DT_I8:   hipLaunchKernelGGL(mfma_peak_kernel<DT_I8>, dim3(blocks), dim3(256), 0, st, iters, clk, sink); break;
    case DT_BF16: hipLaunchKernelGGL(mfma_peak_kernel<DT_BF16>, dim3(blocks), dim3(256), 0, st, iters, clk, sink); break;
    case DT_F16:  hipLaunchKernelGGL(mfma_peak_kernel<DT_F16>, dim3(blocks), dim3(256), 0, st, iters, clk, sink); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace abft
