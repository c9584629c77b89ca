// Fast path of the protected GEMM for gfx950: B stored N x K (both operands K-contiguous) and
// K a whole number (at least three) of 128-byte slabs.  The data movement:
//   * global -> LDS with buffer loads that go straight there (buffer_load_dwordx4 ... lds): no VGPR staging.  One
//     wave instruction fills 8 LDS rows of 128 bytes; the XOR swizzle of the LDS layout is
//     applied by choosing which global 16-byte chunk each lane fetches.
//   * 256 x 256 tiles by eight waves of 128 x 64 (eight 32x32 MFMA blocks per wave), 128 x 256 tiles by eight of 64 x 64;
//     one barrier per slab, loads spread evenly between the MFMAs.
//   * two waves per SIMD: what one wave spends on issuing loads, fragment reads and the epilogue's vector instructions, the other
//     fills with MFMAs.  With one (four waves of 128 x 128, the LDS traffic of a slab 192 instead of 256 KB) every instruction
//     beside an MFMA costs five clocks of the only wave there is.  What bounded that loop was not LDS bandwidth, which a
//     micro-benchmark puts at 256 bytes per clock for 16-byte fragment reads (64 KB of them per 32 KB loaded cost nothing), but issue:
//     the vector memory path takes a load of 1 KB every 18 clocks per compute unit, and all of a slab's loads in one of its four steps
//     held every wave there.  Four waves / eight, clocks per slab (MFMAs alone 2048 and 1024): 256 x 256
//     2388 / 2152, 128 x 256 1526 / 1130; epilogue of a 256 x 256 tile, unprotected 5500 / 3900, protected 12000 / 10200.
//     bf16, unprotected: 6304 x 768 x 768 11.9 -> 10.7 us, 6304 x 768 x 3072 40.9 -> 32.6, 12608 x 3072 x 768 57.9 -> 55.0, 4096 x 4096 x 4096
//     103 -> 100.  The large ones are power-limited: of the 11 % fewer clocks the chip takes back most by its clock (1.73 -> 1.56
//     GHz over 4096 x 4096 x 4096).
//   * MFMAs take the B fragment first, so a lane owns a row of C (see gemm_epilogue.h).
//   * workgroup -> tile mapping keeps the workgroups that share an XCD (and its L2) on a
//     compact group of tiles.
// Rows of the tile beyond the problem are fetched from a valid row instead of being
// zero-filled: a row of A only influences the same row of C, which is discarded, and the pass
// over A's slabs ignores them.
#include <mutex>
#include <queue>
#include <vector>

#include "abft_device.h"
#include "encode_pass.h"
#include "gemm_args.h"
#include "gemm_epilogue.h"

namespace abft {

typedef const __attribute__((address_space(1))) void *gas_ptr;
typedef __attribute__((address_space(3))) void *las_ptr;

// Unprotected; protected, the tiles reduce A; protected, workgroups beside the tiles do.  A kernel for each: the last
// has no code for owned slabs, the others none for the pass beside them.
enum { FAST_PLAIN, FAST_OWN, FAST_BESIDE };

// LDS of a tile: a slab is MI units of A and 2 NI of B, 64 rows of 128 bytes each: one load instruction of every wave.  Unit mi of A
// holds the rows of block row mi of both wave rows, unit (ni, h) of B those of block column ni of wave columns 2 h and 2 h + 1.
// The first FM units of A and the first 2 FN of B have three buffers, the others two.
template <int BM, int FM, int FN> struct FastLds {
    static constexpr int MI = BM / 64, NI = 2, UNIT = 64 * SLAB_BYTES;
    static constexpr int NLD = MI + 2 * NI;                                // units
    static constexpr int NF = FM + 2 * FN, NR = NLD - NF;                  // those with three buffers, with two
    static constexpr int F_BYTES = NF * UNIT, R_BYTES = NR * UNIT, BYTES = 3 * F_BYTES + 2 * R_BYTES;
    // Load q of a slab: first the units with two buffers, A then B, then those with three.
    static constexpr bool ring3(int q) { return q >= NR; }
    static constexpr bool is_a(int q) { return q < NR ? q < MI - FM : q < NR + FM; }
    static constexpr int unit(int q)                                       // mi, or 2 ni + h
    {
        return q < NR ? (q < MI - FM ? FM + q : 2 * FN + q - (MI - FM)) : q < NR + FM ? q - NR : q - NR - FM;
    }
    // Loads of the four steps from a slab's barrier on: the first of them go where the next barrier needs them.
    static constexpr int by_step(int n) { return n == 0 ? 0 : n == 1 ? (3 * NLD + 7) / 8 : n == 2 ? (5 * NLD + 7) / 8 : n == 3 ? 7 * NLD / 8 : NLD; }
    // where it lies in its buffer
    static constexpr int at(int q) { return (q < NR ? q : q - NR) * UNIT; }
    static constexpr int load_of_a(int mi) { return mi < FM ? NR + mi : mi - FM; }
    static constexpr int load_of_b(int ni) { return ni < FN ? NR + FM + 2 * ni : MI - FM + 2 * (ni - FN); }      // h = 0
};
template <int MODE, int BM> struct FastShape;
template <int MODE> struct FastShape<MODE, 256> { typedef FastLds<256, MODE == FAST_OWN ? 3 : 4, 0> lds; };
template <int MODE> struct FastShape<MODE, 128> { typedef FastLds<128, 2, 2> lds; };
template <int MODE> constexpr int fast_lds_bytes()
{
    const int b = FastShape<MODE, 256>::lds::BYTES, s = FastShape<MODE, 128>::lds::BYTES;
    return b > s ? b : s;
}

// One BM x 256 tile with origin (m0, n0) of batch item bz.
// What the pass over A keeps lies behind the operand buffers.
template <int DT, int BM, int MODE, int STO>
__device__ __forceinline__ void fast_tile(const GemmArgs &g, uint8_t *smem, int m0, int n0, int bz, int tn)
{
    using T = Traits<DT>;
    using L = typename FastShape<MODE, BM>::lds;
    typedef typename T::accv_t accv_t;
    typedef __attribute__((address_space(3))) uint8_t *lds_ptr;
    typedef __attribute__((address_space(3))) void *lds_void;
    typedef const __attribute__((address_space(3))) i32x4 *lds_frag;
    constexpr int ES = T::ES;
    constexpr int KE = SLAB_BYTES / ES;
    constexpr int TM = BM / 2, TN = 64;
    constexpr int MI = L::MI, NI = L::NI, NMF = MI * NI, NFR = MI + NI;
    constexpr int NF = L::NF, NR = L::NR, NLD = L::NLD;
    constexpr bool PROT = MODE != FAST_PLAIN, OWN = MODE == FAST_OWN;

    const int tid = tile_thread_index(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform by construction
    const int wm = wave >> 2, wn = wave & 3;
    const int l32 = lane & 31, lh = lane >> 5;
    const int M = g.M, N = g.N, K = g.K;

    // ---- global sources.  This wave's load of a unit fills its LDS rows 8 wave .. + 8;
    // lane l lands in row + (l >> 3), slot (l & 7), and fetches the chunk for which
    // LDS slot = chunk ^ ((row >> 1) & 7).  (A 16-byte fragment read is served sixteen lanes at a
    // time from 64 banks: sixteen consecutive rows must fall on sixteen different 16-byte bank
    // groups.  Two consecutive 128-byte rows span all 64 banks, so the eight even rows need eight
    // different slots, and so do the eight odd rows; chunk ^ (row & 7) makes rows r and r + 8
    // collide, which the LDS bank-conflict counter showed as half of all LDS cycles.)  Buffer loads: the tile's
    // origin in a descriptor, a lane's offset inside the tile, which never changes, in a register, the slab's in a scalar, so
    // that a load inside the main loop is itself and the word that says where it goes.  Rows of the tile past
    // the end of the matrix fetch the last valid row instead.
    const int lrow = lane >> 3;
    const int lchunk = (lane & 7) ^ (((wave & 1) << 2) + (lrow >> 1));
    constexpr int RSRC_FLAGS = 0x00027000;
    const __amdgpu_buffer_rsrc_t a_src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(g.A + ((long)bz * g.sA + (long)m0 * g.lda) * ES), 0, 0x7FFFFFFF, RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t b_src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(g.B + ((long)bz * g.sB + (long)n0 * g.ldb) * ES), 0, 0x7FFFFFFF, RSRC_FLAGS);
    int off[NLD];
    static_for<0, NLD>([&](auto q_c) {
        constexpr int q = decltype(q_c)::value, u = L::unit(q);
        constexpr bool is_a = L::is_a(q);
        const int in = (wave & 3) * 8 + lrow, last = (is_a ? M - m0 : N - n0) - 1;
        int r = is_a ? (wave >> 2) * TM + u * 32 + in : (2 * (u & 1) + (wave >> 2)) * TN + (u >> 1) * 32 + in;
        r = r < last ? r : last;
        off[q] = r * (int)((is_a ? g.lda : g.ldb) * ES) + lchunk * 16;
    });
    const int a_rows = M - m0;                        // rows of this tile inside A
    const int nslab = K / KE;                         // at least 3 (gemm_fast_eligible)

    // The accumulators are never zero-filled: the first MFMA of every block takes a literal
    // zero as its addend.  Every block is always computed, also where the tile hangs over the
    // edge of the problem: a conditional MFMA would move the accumulators out of their registers.
    accv_t acc[MI][NI];
    accv_t zerov;
#pragma unroll
    for (int i = 0; i < 16; ++i) zerov[i] = T::zero();

    // The buffers of a slab: f of those in rings of three, r of two.
    const lds_ptr lds = (lds_ptr)smem;
    struct Buf { int f, r; };
    auto load = [&](auto q_c, int s, Buf to) __attribute__((always_inline)) {
        constexpr int q = decltype(q_c)::value;
        const lds_ptr dst = lds + ((L::ring3(q) ? to.f : to.r) + wave * 8 * SLAB_BYTES) + L::at(q);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(L::is_a(q) ? a_src : b_src, (lds_void)dst, 16, off[q], s * SLAB_BYTES, 0, 0);
    };
    // ---- main loop, software-pipelined by hand.  A slab is four MFMA steps of 32 bytes of K.
    // The fragments of step t+1 are read from LDS while the MFMAs of step t run (two register
    // sets).  The barrier sits between steps 2 and 3: by then every wave has
    // read its step-3 fragments, so nobody reads this slab's buffers any more.  From there on, over the four steps up to the
    // next slab's barrier, the loads into those buffers are issued: the units with two buffers of slab s + 2, then those with
    // three of slab s + 3.
    i32x4 fa[2][MI], fb[2][NI];
    // a lane's place in a unit of A at step 0 (row l32 of this wave's half); at step t chunk 2 t + lh, so bits 5 and 6 change
    const int frag_at = wm * 32 * SLAB_BYTES + l32 * SLAB_BYTES + (lh ^ ((lane >> 1) & 7)) * 16;
    const int b_from_a = (wn - wm) * 32 * SLAB_BYTES; // the same in a unit of B, from unit h = 0 on
    // fragment j of step t: of B, then of A
    auto fragment = [&](auto j_c, auto t_c, Buf b) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value, t = decltype(t_c)::value, set = t & 1;
        constexpr bool isb = j < NI;
        constexpr int q = isb ? L::load_of_b(isb ? j : 0) : L::load_of_a(isb ? 0 : j - NI);
        const int base = (L::ring3(q) ? b.f : b.r) + (isb ? b_from_a : 0);
        const i32x4 v = *(lds_frag)(lds + ((frag_at ^ (32 * t)) + base) + L::at(q));
        if constexpr (isb) fb[set][isb ? j : 0] = v;
        else fa[set][isb ? 0 : j - NI] = v;
    };
    // MFMA j of step t (set t & 1)
    auto mfma = [&](auto first_c, auto t_c, auto j_c) __attribute__((always_inline)) {
        constexpr int set = decltype(t_c)::value & 1, mi = decltype(j_c)::value / NI, ni = decltype(j_c)::value % NI;
        acc[mi][ni] = T::mfma(fb[set][ni], fa[set][mi], decltype(first_c)::value ? zerov : acc[mi][ni]);
    };
    // Protected tiles reduce the slabs of A they own (slab s belongs to tile column s mod
    // tiles_n) while those are resident: see gemm_apass.h.
    constexpr int AUX_OFF = fast_lds_bytes<MODE>();    // behind the buffers of the larger tile
    static_assert(epi_total_bytes(BM, 256) <= AUX_OFF, "the epilogue reads the column sums there while it fills the LDS ahead of them");
    EpiProt<DT, MI> ep;
    ep.slab0 = tn; ep.slab_step = g.tiles_n; ep.owned = (OWN && tn < nslab) ? (nslab - tn + g.tiles_n - 1) / g.tiles_n : 0;
    ep.col_lds = reinterpret_cast<uint32_t *>(smem + AUX_OFF);
    ep.back = 1.f;
    {
        int next_own = tn, own_at = 0;                 // the next slab to reduce, and its place among the owned
        // column sums, [owned][KE]; terms of b, [2][3][KE]; zeros; words of b, [2][KE]
        constexpr int TERM = SLAB_BYTES, TERMS = 3 * TERM;
        uint8_t *const terms = smem + AUX_OFF + ep.owned * KE * 4;
        uint32_t *const words = reinterpret_cast<uint32_t *>(terms + 2 * TERMS + TERM);
        // b of the j-th owned slab, straight into LDS, two owned slabs ahead.  (A register would be waited for together
        // with every operand load behind it.)
        auto fetch_b = [&](int j) __attribute__((always_inline)) {
            if (wave < KE / 64 && j < ep.owned)
                __builtin_amdgcn_global_load_lds((gas_ptr)(g.b_sum + (long)bz * K + (tn + j * g.tiles_n) * KE + 64 * wave + lane),
                                                 (las_ptr)(words + (j & 1) * KE + 64 * wave), 4, 0, 0);
        };
        if constexpr (OWN) {
            fetch_b(0);
            fetch_b(1);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) ep.pass.dot[mi] = acc4_zero<DT>();
            ep.pass.amax = 0u;
            for (int i = tid; i < ep.owned * KE + SLAB_BYTES / 4; i += 64 * FAST_WAVES)
                reinterpret_cast<uint32_t *>(smem + AUX_OFF)[i < ep.owned * KE ? i : i + 2 * TERMS / 4] = 0u;
        }
        // buffers of slabs s, s + 1, s + 2 (three-buffer units; two-buffer units of s + 2: those of s)
        int f0 = 0, f1 = L::F_BYTES, f2 = 2 * L::F_BYTES, r0 = 3 * L::F_BYTES, r1 = r0 + L::R_BYTES;
        auto next = [&]() __attribute__((always_inline)) {
            const int f = f0, r = r0;
            f0 = f1; f1 = f2; f2 = f;
            r0 = r1; r1 = r;
        };
        static_for<0, NLD>([&](auto q_c) { load(q_c, 0, Buf{f0, r0}); });
        static_for<0, NLD>([&](auto q_c) { load(q_c, 1, Buf{f1, r1}); });
        // Start as soon as slab 0 is in place: loads complete in order, so "at most the loads of the
        // slab behind it outstanding" means everything issued before them has landed.
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(NLD) : "memory");
        static_for<0, NFR>([&](auto j_c) { fragment(j_c, std::integral_constant<int, 0>{}, Buf{f0, r0}); });
        // The barrier of slab s: slab s + 1 is in place; what was requested after it are the units with three buffers of
        // slab s + 2 (or nothing any more).
        auto slab_barrier = [&](auto behind_c) __attribute__((always_inline)) {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(decltype(behind_c)::value ? NF : 0) : "memory");
        };
        // b of the next slab to reduce in terms of the operand type, a slab ahead of it
        float scale = 1.f;
        if constexpr (OWN && DT == DT_F16) b_scale(N, &scale, &ep.back);
        auto put_terms = [&]() __attribute__((always_inline)) {
            if (wave < KE / 64) {
                typename T::acc_t v = from_word<typename T::acc_t>(words[(own_at & 1) * KE + 64 * wave + lane]);
                if constexpr (DT == DT_F16) v *= scale;
                uint8_t *d = terms + (own_at & 1) * TERMS + (64 * wave + lane) * ES;
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const uint32_t h = b_term<DT>(v);
                    if constexpr (ES == 1) d[e * TERM] = (uint8_t)h;
                    else *reinterpret_cast<uint16_t *>(d + e * TERM) = (uint16_t)h;
                }
            }
        };
        if (OWN && tn == 0) {
            put_terms();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        auto own_ahead = [&](int s) __attribute__((always_inline)) {
            if (OWN && s + 1 == next_own) put_terms();
        };
        auto own_done = [&](int s) __attribute__((always_inline)) {
            if (OWN && s == next_own) {
                next_own += g.tiles_n;
                own_at += 1;
                fetch_b(own_at + 1);
            }
        };
        // The pass over a slab this tile owns, ahead of its MFMAs: a wave takes the fragments of step wn once more, of its rows, two at a
        // time: some ninety instructions, beside which the SIMD's other wave multiplies.  (Dealt out in pieces behind the MFMAs of the slab's
        // first three steps it is no faster: pieces / so, us, bf16 12608 x 768 x 3072 72.7 / 72.2, 20000 x 768 x 2048 66.8 / 65.8, f16 12608 x 768 x
        // 768 30.5 / 30.0, int8 36928 x 1024 x 4096 163.5 / 163.0; 72 problems, 1.006 of the time in pieces.)
        auto reduce = [&](int s) __attribute__((always_inline)) {
            if constexpr (OWN) {
                if (s != next_own) return;
                constexpr int NU = T::IS_INT ? 2 : 1;
                // lane: column c = lane & 15 of the product belongs to the rows of half c >> 2, and to term c & 3
                const int ln = tile_thread_index() & 63, c = ln & 15, term = (c >> 2) == ((ln >> 4) & 1) ? c & 3 : 3;  // (formed here, not kept across the tile)
                const uint8_t *src = terms + (term < 3 ? (own_at & 1) * TERMS + term * TERM : 2 * TERMS);
                const i32x4 b = *reinterpret_cast<const i32x4 *>(src + wn * 32 + (ln >> 5) * 16);
                const i32x4 id0 = turn_operand<DT>(ln, 0), id1 = T::IS_INT ? turn_operand<DT>(ln, 1) : id0;
                typename Acc4<DT>::type sums[NU];
                static_for<0, MI / 2>([&](auto h_c) {
                    constexpr int h = decltype(h_c)::value;
                    i32x4 x[2];
                    TurnSums<DT> ts;
                    static_for<0, 2>([&](auto i_c) {
                        constexpr int i = decltype(i_c)::value, q = L::load_of_a(2 * h + i);
                        x[i] = *(lds_frag)(lds + ((frag_at ^ (32 * wn)) + (L::ring3(q) ? f0 : r0)) + L::at(q));
                        // rows past the end hold the last one's elements
                        if (wm * TM + (2 * h + i) * 32 + l32 >= a_rows) x[i] = i32x4{0, 0, 0, 0};
                    });
                    pass_mfmas<DT>(ep.pass.dot[2 * h], ep.pass.dot[2 * h + 1], ts, x, b, id0, id1);
                    if constexpr (!T::IS_INT) {
                        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
                        u16x2 m = __builtin_bit_cast(u16x2, ep.pass.amax);
#pragma unroll
                        for (int i = 0; i < 8; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, x[i >> 2][i & 3] & 0x7FFF7FFF));
                        ep.pass.amax = __builtin_bit_cast(uint32_t, m);
                        ts.c[0] += ts.c[1];
                    }
#pragma unroll
                    for (int u = 0; u < NU; ++u) sums[u] = h == 0 ? ts.c[u] : sums[u] + ts.c[u];
                });
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    typename T::acc_t v = add_t(add_t((typename T::acc_t)sums[u][0], (typename T::acc_t)sums[u][1]),
                                                add_t((typename T::acc_t)sums[u][2], (typename T::acc_t)sums[u][3]));
                    v = add_xor32(add_xor16(v));
                    if (ln < 16) lds_add_word(const_cast<uint32_t *>(ep.col_lds) + own_at * KE + wn * (KE / 4) + 16 * u + ln, v);
                }
            }
        };
        // A slab with loads between its MFMAs, in explicit program order (one group per MFMA, fenced): left
        // alone, the compiler issues all loads in one burst and the matrix pipe waits for them.  first_c: the first slab; all
        // of slab 1 has been requested ahead of it.
        auto slab = [&](auto first_c, int s) __attribute__((always_inline)) {
            constexpr bool FIRST = decltype(first_c)::value;
            if constexpr (FIRST) reduce(s);
            own_ahead(s);
            static_for<0, 4>([&](auto t_c) {
                constexpr int t = decltype(t_c)::value;
                // this step's loads: step 3 begins with those into this slab's buffers, steps 0 to 2 go on with those into the last one's
                constexpr int at = t == 3 ? 0 : t + 1;
                constexpr int q0 = FIRST && t < 3 ? NR + NF * t / 3 : L::by_step(at), q1 = FIRST && t < 3 ? NR + NF * (t + 1) / 3 : L::by_step(at + 1);
                constexpr int RPM = NMF >= NFR ? 1 : 2;                // fragment reads behind an MFMA
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, NMF>([&](auto j_c) {
                    constexpr int j = decltype(j_c)::value;
                    mfma(std::integral_constant<bool, FIRST && t == 0>{}, t_c, j_c);
                    static_for<(j * RPM < NFR ? j * RPM : NFR), (j * RPM + RPM < NFR ? j * RPM + RPM : NFR)>([&](auto r_c) {
                        fragment(r_c, std::integral_constant<int, (t + 1) & 3>{}, t < 3 ? Buf{f0, r0} : Buf{f1, r1});
                    });
                    static_for<q0 + (q1 - q0) * j / NMF, q0 + (q1 - q0) * (j + 1) / NMF>([&](auto q_c) {
                        constexpr int q = decltype(q_c)::value;
                        int to = s + (t == 3 ? 1 : 0) + (q < NR ? 1 : 2);
                        if (FIRST && t == 3 && q >= NR) to = to < nslab ? to : nslab - 1;      // of three slabs: bytes nobody reads
                        load(q_c, to, t == 3 ? Buf{f0, r0} : Buf{f2, r1});
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (t == 2) slab_barrier(std::true_type{});
            });
            own_done(s);
            next();
        };
        // One of the last slabs: the loads that are still to come in groups ahead of a step's MFMAs.
        auto tail_slab = [&](int s) __attribute__((always_inline)) {
            reduce(s);
            own_ahead(s);
            static_for<0, 4>([&](auto t_c) {
                constexpr int t = decltype(t_c)::value;
                constexpr int at = t == 3 ? 0 : t + 1;
                constexpr int q0 = L::by_step(at), q1 = L::by_step(at + 1), qr = q1 < NR ? q1 : NR < q0 ? q0 : NR;
                const int ahead = s + (t == 3 ? 1 : 0);
                if (q0 < qr && ahead + 1 < nslab) static_for<q0, qr>([&](auto q_c) { load(q_c, ahead + 1, Buf{f0, t == 3 ? r0 : r1}); });
                if (qr < q1 && ahead + 2 < nslab) static_for<qr, q1>([&](auto q_c) { load(q_c, ahead + 2, Buf{t == 3 ? f0 : f2, r0}); });
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, NMF>([&](auto j_c) {
                    constexpr int j = decltype(j_c)::value;
                    constexpr int RPM = NMF >= NFR ? 1 : 2;
                    mfma(std::false_type{}, t_c, j_c);
                    // after the last slab: read and never used
                    static_for<(j * RPM < NFR ? j * RPM : NFR), (j * RPM + RPM < NFR ? j * RPM + RPM : NFR)>([&](auto r_c) {
                        fragment(r_c, std::integral_constant<int, (t + 1) & 3>{}, t < 3 ? Buf{f0, r0} : Buf{f1, r1});
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (t == 2) {
                    if (s + 2 < nslab) slab_barrier(std::true_type{});
                    else slab_barrier(std::false_type{});
                }
            });
            own_done(s);
            next();
        };
        slab(std::true_type{}, 0);
        int s = 1;
        // the middle slabs: runs of slabs that are not this workgroup's, each followed by one that is
        const int mid_end = nslab - 3;
        if constexpr (OWN) {
            while (next_own < mid_end) {                   // next_own >= s here
                for (; s < next_own; ++s) slab(std::false_type{}, s);
                reduce(s);
                slab(std::false_type{}, s);
                ++s;
            }
        }
        for (; s < mid_end; ++s) slab(std::false_type{}, s);
        for (; s < nslab; ++s) tail_slab(s);
    }
    __syncthreads();
    gemm_epilogue<DT, BM, PROT, STO>(g, acc, smem, m0, n0, bz, ep);
}

// The grid mixes two tile shapes against wave quantisation: 256 x 256 tiles cover the first
// big_rows rows, 128 x 256 tiles the rest; how many of each is chosen by playing the dispatch
// through (choose_big_rows).  (600 big tiles on 256 CUs would be three rounds for 2.34 rounds
// of work.)
template <int DT, int MODE, int STO>
__global__ __launch_bounds__(64 * FAST_WAVES) void gemm_fast_kernel(GemmArgs whole)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    constexpr bool PROT = MODE != FAST_PLAIN;
    fetch_args<GemmArgs>();
    // Persistent workgroups: one per compute unit, each walks the tile list with the grid's stride.
    // The 128-row tiles come first in the list: the compute units that start with one are half a
    // tile ahead of the others from then on, so the two groups store their tiles of C at different
    // times (a round of the machine that stores in step asks for tens of MB at once) and draw on
    // the matrix pipes at different times.  Measured on 12608 x 3072 x 768 (tiles by four waves): 63 -> 60.5 us.
    for (int t = blockIdx.x;;) {
        // (unprotected, there are scalars enough for all of a launch, and one trip to them is less)
        const GemmArgs &g = PROT ? kernel_args<GemmArgs>() : whole;
        if (PROT && t == 0 && threadIdx.x < 5) g.counts[threadIdx.x] = 0u;               // completed by the check kernel
        const int n_tile = MODE == FAST_BESIDE ? (int)gridDim.x - g.beside.n : (int)gridDim.x;
        if constexpr (MODE == FAST_BESIDE) {
            if ((int)blockIdx.x >= n_tile) {
                a_beside<DT>(g, (int)blockIdx.x - n_tile, smem);
                return;
            }
        }
        const int per_item = g.n_small + g.n_big;
        const int bz = t < per_item ? 0 : t / per_item, bid = t - bz * per_item;
        int tm, tn;
        if (STO != STO_128 && bid >= g.n_small) {
            map_tile(bid - g.n_small, g.n_big, g.tiles_m_big, g.tiles_n, g.group_inv, &tm, &tn);
            if constexpr (STO != STO_128) fast_tile<DT, 256, MODE, STO>(g, smem, tm * 256, tn * 256, bz, tn);
        } else {
            map_tile(bid, g.n_small, g.tiles_m_small, g.tiles_n, g.group_inv, &tm, &tn);
            fast_tile<DT, 128, MODE, STO>(g, smem, g.tiles_m_big * 256 + tm * 128, tn * 256, bz, tn);
        }
        t += n_tile;
        if (t >= per_item * g.batch) break;
        // the epilogue's last reads of LDS precede the next tile's first writes
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}

// ------------------------------------------------------------------------------------------
// How many tile rows get 256-row tiles (the rest of M gets 128-row tiles).  Workgroups are
// dispatched in index order to whichever CU is free, one per CU; a 128 x 256 tile takes 0.57 of the time of a 256 x 256 tile
// (19.6 k of 34.6 k clocks at 12 slabs), protected 0.66 (29.7 k of 45 k): its prologue is the same.  A few candidate splits are
// played through with those two costs and the one that finishes first wins; the result is remembered per shape.  (The ratio falls
// with depth, to 0.54 and 0.57 at 60 slabs.  Costs by a problem's slabs and owned slabs were
// no better: 1.001 of the time over 120 random problems, single ones within 4 % either way.)
static double play_schedule(int big_rows, int M, int tiles_n, int batch, int ncu, double small)
{
    const int rest = M - big_rows * 256;
    const long nb = (long)big_rows * tiles_n, ns = (long)(rest > 0 ? (rest + 127) / 128 : 0) * tiles_n;
    std::priority_queue<double, std::vector<double>, std::greater<double>> cu;
    for (int i = 0; i < ncu; ++i) cu.push(0.0);
    double end = 0.0;
    for (int z = 0; z < batch; ++z)
        for (long t = 0; t < nb + ns; ++t) {
            const double f = cu.top() + (t < ns ? small : 1.0);     // dispatch order: the half-height tiles first
            cu.pop();
            cu.push(f);
            if (f > end) end = f;
        }
    return end;
}

static int choose_big_rows(int M, int tiles_n, int batch, int ncu, bool protect)
{
    struct Memo { int M, tiles_n, batch, ncu, protect, big_rows; };
    static Memo memo[16];
    static int memo_n = 0;
    static std::mutex memo_lock;                 // contexts may be driven from different host threads
    std::lock_guard<std::mutex> hold(memo_lock);
    for (int i = 0; i < memo_n; ++i)
        if (memo[i].M == M && memo[i].tiles_n == tiles_n && memo[i].batch == batch && memo[i].ncu == ncu && memo[i].protect == protect)
            return memo[i].big_rows;
    const double small = protect ? 0.66 : 0.57;
    const int rows_all_big = (M + 255) / 256;
    const long per_row = (long)tiles_n * batch;
    const long total_big = rows_all_big * per_row;
    int cand[4], nc = 0;
    cand[nc++] = rows_all_big;                                   // big tiles only
    cand[nc++] = 0;                                              // half-height tiles only
    long whole = (total_big / ncu) * ncu / per_row;              // whole rounds of big tiles
    if (whole > rows_all_big) whole = rows_all_big;
    cand[nc++] = (int)whole;
    const long fewer = whole - (ncu + per_row - 1) / per_row;    // one round fewer
    if (fewer > 0) cand[nc++] = (int)fewer;
    int best = cand[0];
    double best_t = play_schedule(cand[0], M, tiles_n, batch, ncu, small);
    for (int i = 1; i < nc; ++i) {
        const double t = play_schedule(cand[i], M, tiles_n, batch, ncu, small);
        if (t < best_t - 1e-9) { best_t = t; best = cand[i]; }
    }
    Memo m = {M, tiles_n, batch, ncu, protect, best};
    memo[memo_n < 16 ? memo_n++ : (M + tiles_n) & 15] = m;
    return best;
}

// Workgroups that reduce A on the `idle` compute units the tiles of a single round leave (a_beside).  Windows of 8
// to 64 chunks along K (least padding, then widest), the rows dealt to as few row blocks as end in 0.85 of the time that the
// tiles take: whatever reads A at once takes from the tiles' loads, and on every idle compute unit the pass cost more than it saved
// where those were many.  us, tiles that own slabs / a workgroup on every idle unit / so: bf16 3775 x 1280 x 1600 33.2 / 33.6 / 30.3, f16 1447 x
// 2752 x 2304 41.2 / 42.2 / 36.0, 8014 x 512 x 1344 31.0 / 33.8 / 28.3, 6304 x 768 x 3072 50.5 / 48.4 / 44.7; bf16 5664 x 768 x 3904 58.3 / 49.6 /
// 49.5, int8 4655 x 1664 x 2688 40.2 / 37.8 / 37.5.  210 random problems that the conditions below let in: 0.957 of the time with owned
// slabs (the worst 1.02, as far as two runs differ), 16-bit types 0.964 and int8 0.993 of that with all idle units.
// Times in us of a workgroup's pass (it reads 64 KB at a time) and of a tile beside one, with what the clock comes down to under load.
static double beside_us(int dt, long bytes) { return 4.0 + (double)bytes / (dt == DT_I8 ? 15e3 : 20e3); }
static double tile_us(bool big, int slabs) { return big ? 8.0 + 1.25 * slabs : 6.0 + 0.7 * slabs; }
static BesideArgs plan_beside(int dt, int M, int K, int batch, int slabs, int tiles_n, int idle, bool big)
{
    const BesideArgs none = {0, 0, 0, 0, 0};
    if (dt == DT_I8 ? slabs < 9 || slabs < tiles_n : slabs < 20 || slabs < 3 * tiles_n) return none;
    const EncPlan w = plan_window(M, K, 16 / elem_size(dt));
    const long per_row_block = (long)w.nwin * batch;
    if (per_row_block > idle) return none;
    BesideArgs b;
    b.cw_log2 = w.cw_log2; b.nwin = w.nwin;
    const int rl = (64 * FAST_WAVES >> w.cw_log2) * 8;                      // rows a workgroup takes at a time
    const double tiles_us = tile_us(big, slabs);
    const int most = (int)(idle / per_row_block);
    double us = 0.0;
    for (int n = 1; n <= most; ++n) {
        b.rpb = ((M + n - 1) / n + 15) / 16 * 16;
        if (b.rpb < rl) b.rpb = rl;
        us = beside_us(dt, (long)b.rpb * (16 << w.cw_log2));
        if (us <= 0.85 * tiles_us || b.rpb == rl) break;
    }
    b.nrb = (M + b.rpb - 1) / b.rpb;
    b.n = (int)(b.nrb * per_row_block);
    return us <= 1.2 * tiles_us ? b : none;
}

template <int DT, bool PROT, bool STO>
static hipError_t launch_fast_one(GemmArgs &g, int batch, hipStream_t st)
{
    constexpr int smem_max = 160 * 1024;
    const int slabs = g.K / (SLAB_BYTES / Traits<DT>::ES);
    hipError_t e;
    const int num_cu = device_cu_count(&e);
    if (e != hipSuccess) return e;
    g.tiles_n = (g.N + 255) / 256;
    g.group_inv = map_inverse(g.tiles_n);
    const int big_rows = choose_big_rows(g.M, g.tiles_n, batch, num_cu, PROT);
    g.tiles_m_big = big_rows;
    g.n_big = big_rows * g.tiles_n;
    const int rest = g.M - big_rows * 256;
    g.tiles_m_small = rest > 0 ? (rest + 127) / 128 : 0;
    g.tiles_m = g.tiles_m_big + g.tiles_m_small;
    g.n_small = g.tiles_m_small * g.tiles_n;
    g.batch = batch;
    const long total = (long)(g.n_big + g.n_small) * batch;
    if (total > 0x7FFFFFFFL) return hipErrorInvalidValue;
    dim3 grid((unsigned)(total < num_cu ? total : num_cu), 1, 1);
    g.beside.n = 0;
    if (PROT && total < num_cu) {
        g.beside = plan_beside(DT, g.M, g.K, batch, slabs, g.tiles_n, num_cu - (int)total, g.n_big != 0);
        grid.x += g.beside.n;
    }
    size_t smem;
    // Stored sums: the mix of tiles of any other call, and a kernel of its own where all have 128 rows (gemm_epilogue.h).  us, protected and
    // stored: all of 128 rows / mixed: bf16 12608 x 768 x 3072 103.4 / 81.7, 12608 x 3072 x 768 95.5 / 85.5, 6304 x 3072 x 768 62.0 / 55.0,
    // fp16 12212 x 3712 x 3904 381 / 344.
    constexpr int ALL = STO ? STO_256 : STO_NO, SMALL = STO ? STO_128 : STO_NO;
    auto kern = STO && !big_rows ? gemm_fast_kernel<DT, PROT ? FAST_OWN : FAST_PLAIN, SMALL> : gemm_fast_kernel<DT, PROT ? FAST_OWN : FAST_PLAIN, ALL>;
    if constexpr (PROT) {
        const size_t aux = fast_aux_bytes(DT, slabs, g.tiles_n);
        smem = fast_lds_bytes<FAST_OWN>() + aux;
        if (g.beside.n) {
            kern = STO && !big_rows ? gemm_fast_kernel<DT, FAST_BESIDE, SMALL> : gemm_fast_kernel<DT, FAST_BESIDE, ALL>;
            smem = fast_lds_bytes<FAST_BESIDE>();
        }
    } else {
        smem = fast_lds_bytes<FAST_PLAIN>();
    }
    if (smem > (size_t)smem_max) return hipErrorInvalidValue;
    e = ensure_max_lds(reinterpret_cast<const void *>(kern), smem_max);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(64 * FAST_WAVES), smem, st, g);
    return hipGetLastError();
}

bool gemm_fast_eligible(int dt, int M, int N, int K, bool transB, long lda, long ldb)
{
    const int ke = SLAB_BYTES / elem_size(dt);
    // whole slabs, at least three of them (the main loop is peeled), and 32-bit row offsets
    // inside a tile
    // (int8: N < 65536 keeps |b| <= 128 N below 2^23, which the pass over A's slabs relies on here)
    return transB && (K % ke) == 0 && K >= 3 * ke && M >= 512 && N >= 512 && (dt != DT_I8 || N < 65536) &&
           lda * elem_size(dt) < (1L << 23) && ldb * elem_size(dt) < (1L << 23) &&
           // what the pass over A's slabs keeps per tile fits behind the operand buffers (protected or
           // not: a problem takes the same kernel in every mode)
           fast_lds_bytes<FAST_OWN>() + fast_aux_bytes(dt, K / ke, (N + 255) / 256) <= 160 * 1024;
}

void gemm_fast_tile(int *tm, int *tn) { *tm = 256; *tn = 256; }

template <int DT> static hipError_t launch_fast_type(bool protect, GemmArgs &g, int batch, hipStream_t st)
{
    if (!protect) return launch_fast_one<DT, false, false>(g, batch, st);
    if constexpr (!Traits<DT>::IS_INT)
        if (g.cc_sto) return launch_fast_one<DT, true, true>(g, batch, st);
    return launch_fast_one<DT, true, false>(g, batch, st);
}

hipError_t launch_gemm_fast(int dt, bool protect, GemmArgs &g, int batch, hipStream_t st)
{
    switch (dt) {
    case DT_I8:   return launch_fast_type<DT_I8>(protect, g, batch, st);
    case DT_BF16: return launch_fast_type<DT_BF16>(protect, g, batch, st);
    case DT_F16:  return launch_fast_type<DT_F16>(protect, g, batch, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace abft
