// Operations (2) and (5) of the fused LoRA linear layer (Section 5.1, FusedLoRA Design) on small output tiles:
// the launches whose 256- or 192-row tiles of lf_gemm.hip would leave most compute units without work.
//   (2)  Y  = X W + S' B                     out operand W [N,K], B [N,r]: contiguous along the contraction
//   (5)  dX = dY W^T + mask*q*(dS A^T)       out operand W [N,K], A [r,K]: contraction over the rows
// Every output element is formed by the same MFMAs in the same order as on the large tiles (contraction in steps of
// 32 from zero, then the LoRA term), so Y and dX are bit-identical whichever kernel a launch picks.
//
// What bounds them: the copies out of L2 (a compute unit takes in 120 GB/s when all of them copy, 147 by itself; 128 x 128 tiles,
// one on every compute unit, use 80), and the meeting of the waves once a slab.  Hence: a ring of three to eight slabs in LDS,
// filled several slabs ahead by waves that do nothing else (a copy holds the wave that issues it up until the memory pipeline
// takes it, and a wave that waits for copies to land is late for its MFMAs), one barrier per slab; the computing waves read
// their fragments one sub-step ahead or, in the tiles whose waves have the registers and eight MFMAs or more a sub-step to
// cover the reads with, a whole slab ahead, which leaves nothing but the barrier between two slabs' MFMAs; two workgroups on a
// compute unit for the tiles whose ring leaves room.  Accumulators are vector registers, the MFMAs assembly (see ring_mfma): the
// compiler's own moved every accumulator block in every step (M = 1024, 4096 x 4096: 40 -> 35 us).
// Against copies issued by the computing waves between their MFMAs, us, (2) / (5): 1024 x 4096 x 4096 36.0 -> 33.4 / 36.1 -> 33.3; 1000 rows,
// 14336 -> 4096 110 -> 104 / 109 -> 99; 512 x 4096 x 4096 23.6 -> 22.2 / 24.0 -> 22.9; 256 rows, 17024 -> 17856 247 -> 239 /
// 236 -> 212; 128 rows, 26496 -> 960 54 -> 54.6 / 64 -> 54.5; 256 x 1024 x 1024 5.4 -> 4.8 / 5.8 -> 4.8 (replayed back to back; in a
// trace of whole steps 5.7 and, with the strips, 6.0).
// Measured, one launch, against the 128-row tiles that served these sizes before: 256 x 1024 x 1024 16 -> 6.1 us
// forward, 22 -> 6.7 us backward; 1024 x 4096 x 4096 56 -> 35 and 66 -> 39 us; 77 rows, 4096 -> 14336 51 -> 24 and
// (backward) 174 -> 41 us; 64 rows, 15616 -> 320 176 -> 33 us.
#include <type_traits>

#include "lf_device.h"
#include "lf_gemm_parts.h"
#include "lf_gemm_ring.h"
#include "lf_internal.h"
#include "lf_strips.h"

namespace lf {

// One kernel of the family.  TM x TN output tile, WM x WN computing waves of (TM / WM) x (TN / WN) each, ring of NS LDS stages,
// one slab pair of 64 * D contraction elements per stage.  TW waves copy the token slabs and OW the out slabs; TW = 0: OW waves copy both (the better
// way for the one tile whose out slab is the larger one: 256 rows, 17024 -> 17856, (5) 222 -> 212 us).
template <int TM_, int TN_, int WM_, int WN_, int NS_, int TW_, int OW_, int D_ = 1>
struct Ring {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, NS = NS_, TW = TW_, OW = OW_, CW = TW + OW, D = D_;
    static constexpr int NW = WM * WN, THREADS = 64 * NW;             // waves and threads that compute
    static constexpr int MI = TM / WM / 16, NI = TN / WN / 16;        // 16x16 blocks per wave
    static constexpr int DEPTH = D * BK, SUBS = 2 * D;                // contraction elements and sub-steps of 32 to a stage
    static constexpr int ROWB = DEPTH * 2;                            // bytes of a row in a row-operand slab
    static constexpr int STAGE = (TM + TN) * ROWB;
    static constexpr int LDS = NS * STAGE;
    static constexpr int REGS = 512 / ((NW + CW + 3) / 4);            // of a wave, with a SIMD's share of the workgroup on it
    // fragments of two slabs in registers: where they fit beside the accumulators and some forty others (128 x 64 tiles with the
    // shorter sub-steps of a 2 x 4 split, 512 x 4096 x 4096: 22.4 -> 23.8 us, so not below eight MFMAs)
    static constexpr bool NARROW = D == 1 && TM == 32;                // whole 32 x 64 tiles of one slab to a stage
    static constexpr bool AHEAD = D == 2 || MI * NI >= 8 && MI * NI * 4 + (MI + NI) * 16 + 40 <= REGS;
    static_assert(TM * D / 8 % (TW ? TW : OW) == 0 && TN * D / 8 % OW == 0, "the copies of a slab divide evenly over the waves");
    static_assert(NS >= 2, "ring depth");
    static_assert(TM * TN / 8 % THREADS == 0 || TM * TN / 8 < THREADS, "whole passes on the way out, or one");
    static_assert(TM * TN * 2 <= LDS, "the way out goes through the ring");
};

// Column-operand slab of TN columns: 64 contraction rows of TN * 2 bytes, chunk index XOR-ed so that the 32 lanes of a
// transposing read ({a..a+3, a+8..a+11} x 32 bytes) cover 256 distinct bytes mod 256.  128 columns and more: as in the
// large tiles; 64 (32) columns: two (four) rows share 256 bytes, so only row bits 1 and 3 (bit 3) choose among a row's windows.
template <int TN>
__device__ __forceinline__ int ring_col_swz(int row) {
    return TN >= 128 ? col_slab_swz(row) : TN == 64 ? (row & 2) | ((row & 8) >> 1) : (row & 8) >> 2;
}

// ---- the copying waves -----------------------------------------------------------------------------
// Position of 16-byte chunk `chunk` of row `row` in a row-operand slab: 64 elements to a row as in the large tiles, or 128, where the 16 rows of a
// fragment read are 256 bytes apart and each needs a chunk position of its own.
template <int D>
__device__ __forceinline__ int ring_row_swz(int row) { return D == 1 ? row_slab_swz(row) : row & 15; }

// Where a slab comes from: rows (token: of the tile; out: output columns or, COL, contraction rows) `ld` elements apart, `rows`
// of them valid; chunks: valid 16-byte chunks along the contraction (8 or 16, r / 8 for the LoRA slab), COL: along the columns.
struct RingSource { const char* biased; uint32_t ld; int rows, chunks; };

// Copies of a slab pair by one wave: NT of the token slab, then NO of the out slab (1 KB each); either may be none.  Those of
// a slab share an M0.
template <class C, bool COL, int NT_, int NO_>
struct RingCopies {
    static constexpr int NT = NT_, NO = NO_, N = NT + NO;
    static_assert(NT <= 8 && NO <= 8 && N * (C::NS - 1) < 64, "immediates of the copies; the wait counter has six bits");

    // Source offset of this lane for copy I of wave w, bytes from the slab's first element.
    template <int I>
    static __device__ __forceinline__ uint32_t lane(int w, const RingSource& tok, const RingSource& out) {
        const int l = threadIdx.x & 63;
        uint32_t e;                                                   // < 2^30: at most 256 rows of 2^22 elements
        if constexpr (I < NT) {
            const int pos = (w * NT + I) * 64 + l, row = pos / (8 * C::D);
            e = (uint32_t)min(row, tok.rows - 1) * tok.ld + min((pos % (8 * C::D)) ^ ring_row_swz<C::D>(row), tok.chunks - 1) * 8;
        } else if constexpr (!COL) {
            const int pos = (w * NO + I - NT) * 64 + l, row = pos / (8 * C::D);
            e = (uint32_t)min(row, out.rows - 1) * out.ld + min((pos % (8 * C::D)) ^ ring_row_swz<C::D>(row), out.chunks - 1) * 8;
        } else {
            constexpr int CPR = C::TN / 8;                            // chunks per slab row
            const int pos = (w * NO + I - NT) * 64 + l, row = pos / CPR;
            e = (uint32_t)min(row, out.rows - 1) * out.ld + min((pos % CPR) ^ ring_col_swz<C::TN>(row), out.chunks - 1) * 8;
        }
        return e * 2 + kCopyBias - (I < NT ? pass_imm(NT, I) : pass_imm(NO, I - NT));
    }

    // One slab pair's copies into the stage at LDS address `stage`.  FORM: the lane offsets are formed on the way, each right before
    // its copy (the first slab of a launch waits for nothing else).
    template <bool FORM, int I = 0>
    static __device__ __forceinline__ void issue(int w, const RingSource& tok, const RingSource& out, uint32_t (&off)[N], uint32_t stage) {
        if constexpr (I < N) {
            if constexpr (FORM) off[I] = lane<I>(w, tok, out);
            if constexpr (I < NT) copy16_to_lds<pass_imm(NT, I), I == 0>(tok.biased, off[I], stage + (w * NT + NT / 2) * 1024);
            else copy16_to_lds<pass_imm(NO, I - NT), I == NT>(out.biased, off[I], stage + C::TM * C::ROWB + (w * NO + NO / 2) * 1024);
            if constexpr (FORM) __builtin_amdgcn_sched_barrier(0);
            issue<FORM, I + 1>(w, tok, out, off, stage);
        }
    }

    // Slab `kt` goes into stage kt % NS: a base slab (out_adv bytes further each time), the LoRA slab (kt == nk, if there is one),
    // or nothing.  The barriers are those of the computing waves: one before the first slab, then one per slab, at which the
    // copies of slab kt + 1 have landed and the stage of slab kt is free.
    static __device__ __forceinline__ void run(int w, RingSource tok, RingSource out, int64_t out_adv, const RingSource& ltok,
                                               const RingSource& lout, int slabs, bool has_lora, bool at_once, uint32_t lds) {
        constexpr int NS = C::NS;
        const int nk = (slabs + C::D - 1) / C::D, nkt = nk + has_lora;
        const int half_at = C::D == 2 && (slabs & 1) ? nk - 1 : nk;       // the stage of which half is past the contraction's end
        uint32_t off[N];
        auto slab = [&](int kt, int stage, auto form) {           // (first lane: an M0 value is scalar, whatever else the kernel holds)
            if (kt < half_at) {
                issue<form()>(w, tok, out, off, __builtin_amdgcn_readfirstlane(lds + stage * C::STAGE));
                tok.biased += C::ROWB;
                out.biased += out_adv;
            } else if (C::D == 2 && kt < nk) {
                tok.chunks = 8;
                if constexpr (COL) out.rows = BK;
                else out.chunks = 8;
                issue<true>(w, tok, out, off, __builtin_amdgcn_readfirstlane(lds + stage * C::STAGE));
            } else if (kt < nkt) {
                issue<true>(w, ltok, lout, off, __builtin_amdgcn_readfirstlane(lds + stage * C::STAGE));
            }
        };
        slab(0, 0, std::true_type{});
#pragma unroll
        for (int s = 1; s < NS; ++s) slab(s, s, std::false_type{});
        if (nkt >= NS) wait_slab_loads_but<N*(NS - 1)>();
        else wait_slab_loads();
        asm volatile("s_barrier" ::: "memory");
        int stage = 0, kt = 0;
        // (2) on whole 32 x 64 tiles, while a whole base slab follows, without a branch: the loop below picks its wait and its sources anew in
        // every step, some twenty instructions and four jumps between the barrier and the copies, which the slab of such a tile (0.13 us) waits
        // for.  us, that loop / this, weight cached: 4096 -> 4096, 80 rows 11.9 / 10.7, 128 rows 12.1 / 11.3; 8192 -> 4096, 128 rows 22.1 / 19.3; four
        // adapters of 3 - 10 rows, 16384 -> 4096 54.1 / 47.9; from HBM 17.2 / 16.9, 29.0 / 28.9, 67.9 / 66.1.  Not where the weight outgrows the memory-side
        // cache, whose copies come late anyway and are the worse for coming all at once (eight adapters of 1 - 16 rows, 8896 -> 20480 217 / 223; 16384 ->
        // 9984 104.7 / 105.7; with 242 MB, 11008 -> 11008, three of 9 rows 78.1 / 74.5, from HBM 96.4 / 94.1), nor in (5) (eight adapters of 1 - 18 rows, 9856 to 2368
        // columns 81.9 / 84.4) and on the other tiles (256 rows, 17024 -> 17856 240 / 260; 1500 rows, 4096 -> 4096, backward 68 / 72).
        if constexpr (C::NARROW && !COL) {
            const int whole = at_once ? half_at - NS : 0;
            for (; kt < whole; ++kt) {
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(N * (NS - 2)) : "memory");
                issue<false>(w, tok, out, off, __builtin_amdgcn_readfirstlane(lds + stage * C::STAGE));
                tok.biased += C::ROWB;
                out.biased += out_adv;
                stage = stage + 1 == NS ? 0 : stage + 1;
            }
        }
        for (; kt < nk; ++kt) {
            if (kt + NS <= nkt) wait_slab_loads_but<N*(NS - 2)>();
            else wait_slab_loads();
            asm volatile("s_barrier" ::: "memory");
            slab(kt + NS, stage, std::false_type{});
            stage = stage + 1 == NS ? 0 : stage + 1;
        }
    }
};

template <class C> struct RingFrags { bf16x8 ft[C::MI], fo[C::NI]; };

// Fragment number J of sub-step `sub` (32 contraction elements) of the slab pair at `st`, in the order of first use:
// token block 0, the out blocks, the other token blocks.
template <class C, bool COL, int J>
__device__ __forceinline__ void ring_read_one(RingFrags<C>& f, const char* st, int sub, int wm, int wn) {
    const int l = threadIdx.x & 63;
    const int off = (l & 15) * C::ROWB + (((4 * sub + (l >> 4)) ^ ring_row_swz<C::D>(l & 15)) << 4);
    if constexpr (J == 0 || J > C::NI) {
        constexpr int mi = J == 0 ? 0 : J - C::NI;
        f.ft[mi] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + off + (wm * C::MI + mi) * 16 * C::ROWB));
    } else {
        constexpr int ni = J - 1;
        const char* so = st + C::TM * C::ROWB;
        const int blk = wn * C::NI + ni;
        if constexpr (COL) {
            constexpr int PITCH = C::TN * 2;
            const int row = 8 * (l >> 4) + ((l & 15) >> 2), col = (l & 3) << 2;
            const int o = row * PITCH + (((col >> 3) ^ ring_col_swz<C::TN>(row)) << 4) + ((col & 7) << 1);
            const int a = (o ^ (blk << 5)) + sub * 32 * PITCH;
            f.fo[ni] = join_tr(lds_read_tr(so, a), lds_read_tr(so, a + 4 * PITCH));
        } else {
            f.fo[ni] = __builtin_bit_cast(bf16x8, *(const u32x4*)(so + off + blk * 16 * C::ROWB));
        }
    }
}
template <class C, bool COL, int J = 0, int END = C::MI + C::NI>
__device__ __forceinline__ void ring_read(RingFrags<C>& f, const char* st, int sub, int wm, int wn) {
    if constexpr (J < END) {
        ring_read_one<C, COL, J>(f, st, sub, wm, wn);
        ring_read<C, COL, J + 1, END>(f, st, sub, wm, wn);
    }
}

// MFMAs of a sub-step (block rows FIRST .. of the fragments), from assembly with the accumulators tied in place: with the builtin the compiler moves
// accumulator blocks between registers in every step of the loop.  OPS_FROM_VALU: the operands may come straight from
// the vector ALU (zero_past_rank); the compiler keeps the wait states that needs only for its own MFMAs.
template <class C, bool OPS_FROM_VALU, int FIRST, int ROWS>
__device__ __forceinline__ void ring_mfma(f32x4 (&acc)[ROWS][C::NI], const RingFrags<C>& f) {
#pragma unroll
    for (int mi = 0; mi < ROWS; ++mi)
#pragma unroll
        for (int ni = 0; ni < C::NI; ++ni) {
            if constexpr (OPS_FROM_VALU)
                asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(f.fo[ni]), "v"(f.ft[FIRST + mi]));
            else
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(f.fo[ni]), "v"(f.ft[FIRST + mi]));
        }
}
// ... and the distance to the vector ALU's first read of their results.
template <int MI, int NI>
__device__ __forceinline__ void ring_mfma_done(f32x4 (&acc)[MI][NI]) {
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+v"(acc[mi][ni]));
}

template <class C>
__device__ __forceinline__ void ring_zero_past_rank(RingFrags<C>& f, int sub, int rank_chunks) {
    const int chunk = 4 * sub + ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi) f.ft[mi] = zero_past_rank(f.ft[mi], chunk, rank_chunks);
#pragma unroll
    for (int ni = 0; ni < C::NI; ++ni) f.fo[ni] = zero_past_rank(f.fo[ni], chunk, rank_chunks);
}

// One sub-step of a slab: its MFMAs, and between them the reads of the fragments `nxt` (sub-step nxt_sub of the slab at
// `st`) and, in the second sub-step (HAND), the hand-over to the next slab.  A wave issues in order, so they have to be
// mixed by hand.  With four or fewer MFMAs a sub-step the reads go out in its first half, so
// that the last one has returned when the hand-over (or the next sub-step) needs it, and the hand-over sits a quarter
// into the second sub-step; with more the reads spread evenly.
template <class C> struct RingSlots {
    static constexpr int SLOTS = C::MI * C::NI, READS = C::MI + C::NI;
    static constexpr bool SHORT = SLOTS < 8;
    static constexpr int HAND_AT = SHORT ? SLOTS / 4 : 0;                       // hand-over before this slot's MFMA
    static constexpr int first(bool hand) { return hand ? HAND_AT : 0; }        // first slot that carries reads
    static constexpr int span(bool hand) { return SHORT ? (SLOTS - first(hand) + 1) / 2 : SLOTS; }   // ... and how many do
    static constexpr int reads_before(bool hand, int s) {
        const int k = s - first(hand);
        return k <= 0 ? 0 : k >= span(hand) ? READS : k * READS / span(hand);
    }
};

template <class C, bool COL, bool HAND, int I>
__device__ __forceinline__ void ring_half(f32x4 (&acc)[C::MI][C::NI], const RingFrags<C>& cur, RingFrags<C>& nxt, const char* st,
                                          int nxt_sub, int wm, int wn) {
    using S = RingSlots<C>;
    if constexpr (I < S::SLOTS) {
        constexpr int mi = I / C::NI, ni = I % C::NI;
        // hand-over: every read of the stage is behind this wave; behind the barrier the next slab has landed, too
        if constexpr (HAND && I == S::HAND_AT) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        ring_read<C, COL, S::reads_before(HAND, I), S::reads_before(HAND, I + 1)>(nxt, st, nxt_sub, wm, wn);
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(cur.fo[ni]), "v"(cur.ft[mi]));
        __builtin_amdgcn_sched_barrier(0);
        ring_half<C, COL, HAND, I + 1>(acc, cur, nxt, st, nxt_sub, wm, wn);
    }
}

// Reads FIRST .. END - 1 of a stage's fragments, sub-step by sub-step.
template <class C, bool COL, int FIRST, int END>
__device__ __forceinline__ void ring_read_stage(RingFrags<C> (&f)[C::SUBS], const char* st, int wm, int wn) {
    if constexpr (FIRST < END) {
        constexpr int READS = C::MI + C::NI, sub = FIRST / READS;
        ring_read_one<C, COL, FIRST % READS>(f[sub], st, sub, wm, wn);
        ring_read_stage<C, COL, FIRST + 1, END>(f, st, wm, wn);
    }
}

// A stage with the fragments of two stages in registers (AHEAD): the MFMAs of `cur`, and in their first half the reads of the next
// stage's fragments, from `st`.
template <class C, bool COL, int I>
__device__ __forceinline__ void ring_stage(f32x4 (&acc)[C::MI][C::NI], const RingFrags<C> (&cur)[C::SUBS], RingFrags<C> (&nxt)[C::SUBS],
                                           const char* st, int wm, int wn) {
    constexpr int SLOTS = C::MI * C::NI, READS = C::SUBS * (C::MI + C::NI), SPAN = C::SUBS * SLOTS / 2;
    if constexpr (I < C::SUBS * SLOTS) {
        constexpr int h = I / SLOTS, mi = I % SLOTS / C::NI, ni = I % C::NI;
        constexpr int lo = I * READS / SPAN, hi = (I + 1) * READS / SPAN;
        ring_read_stage<C, COL, lo < READS ? lo : READS, hi < READS ? hi : READS>(nxt, st, wm, wn);
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(cur[h].fo[ni]), "v"(cur[h].ft[mi]));
        __builtin_amdgcn_sched_barrier(0);
        ring_stage<C, COL, I + 1>(acc, cur, nxt, st, wm, wn);
    }
}

template <class C, bool COL, class Args>
__device__ __forceinline__ void ring_tile(const Args& p, char* smem) {
    constexpr int NS = C::NS, MI = C::MI, NI = C::NI;
    int tm, tn;
    tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm, tn);
    RowTile rt;
    if (!find_row_tile_by_lanes(p.tb, C::TM, tm, rt, p.row_lo, p.row_hi)) return;
    const int c0 = tn * C::TN, cols_valid = min(C::TN, p.NC - c0);
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w % C::WM, wn = w / C::WM;
    const bool has_lora = p.r > 0;
    const int nk = p.KC / BK;

    if (w >= C::NW) {
        const int cw = w - C::NW;
        const RingSource tok{(const char*)(p.tok + (int64_t)rt.row_start * p.KC) - kCopyBias, (uint32_t)p.KC, rt.rows, 8 * C::D};
        const RingSource ltok{(const char*)(p.ltok + (int64_t)rt.row_start * p.r) - kCopyBias, (uint32_t)p.r, rt.rows, p.r >> 3};
        const RingSource out = COL ? RingSource{(const char*)(p.out + c0) - kCopyBias, (uint32_t)p.NC, C::DEPTH, cols_valid >> 3}
                                   : RingSource{(const char*)(p.out + (int64_t)c0 * p.KC) - kCopyBias, (uint32_t)p.KC, cols_valid, 8 * C::D};
        const RingSource lout = COL ? RingSource{(const char*)(p.lout + (int64_t)rt.g * p.r * p.NC + c0) - kCopyBias, (uint32_t)p.NC, p.r, cols_valid >> 3}
                                    : RingSource{(const char*)(p.lout + ((int64_t)rt.g * p.NC + c0) * p.r) - kCopyBias, (uint32_t)p.r, cols_valid, p.r >> 3};
        const int64_t out_adv = COL ? (int64_t)C::DEPTH * p.NC * 2 : C::ROWB;
        const uint32_t lds = lds_addr_of(smem);
        const bool at_once = (int64_t)p.KC * p.NC * 2 <= (256ll << 20);     // (the weight fits the memory-side cache)
        if constexpr (C::TW == 0)
            RingCopies<C, COL, C::TM * C::D / 8 / C::OW, C::TN * C::D / 8 / C::OW>::run(cw, tok, out, out_adv, ltok, lout, nk, has_lora, at_once, lds);
        else if (cw < C::TW)
            RingCopies<C, COL, C::TM * C::D / 8 / C::TW, 0>::run(cw, tok, out, out_adv, ltok, lout, nk, has_lora, at_once, lds);
        else
            RingCopies<C, COL, 0, C::TN * C::D / 8 / C::OW>::run(cw - C::TW, tok, out, out_adv, ltok, lout, nk, has_lora, at_once, lds);
        return;
    }

    // (5): keep flags of this lane's elements while the first slabs are on their way.  Block b = mi * NI + ni: bit
    // 2 * (b & 7) + pr of word b >> 3 for element 2 * pr, + 16 for element 2 * pr + 1.
    constexpr int FW = (MI * NI + 7) / 8;
    uint32_t keep[FW];
    if constexpr (COL) {
#pragma unroll
        for (int i = 0; i < FW; ++i) keep[i] = 0xFFFFFFFFu;
        if (has_lora && p.tb.a[rt.g].T) {
            const KeepThreshold th = keep_threshold(p.tb.a[rt.g].T);
            const uint32_t cp0 = (uint32_t)(c0 + wn * NI * 16 + 4 * (l >> 4)) >> 1;
#pragma unroll
            for (int i = 0; i < FW; ++i) keep[i] = 0;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const RowKey rk = row_key(p.tb.a[rt.g].k0, p.tb.a[rt.g].k1,
                                          (uint32_t)(rt.local_row0 + (wm * MI + mi) * 16 + (l & 15)));
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int pr = 0; pr < 2; ++pr) {
                        const int b = mi * NI + ni;
                        const uint32_t m = keep_pair_mask(hash_word(rk, cp0 + ni * 8 + pr), th) & 0x00010001u;
                        keep[b >> 3] |= m << (2 * (b & 7) + pr);
                    }
            }
        }
    }

    f32x4 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

    asm volatile("s_barrier" ::: "memory");

    int stage = 0;
    RingFrags<C> fa[C::SUBS];
    if constexpr (C::AHEAD) {
        // Step kt computes slab kt from registers while it reads slab kt + 1.  At its barrier the copies of that slab have landed,
        // and every wave holds slab kt: the copies of slab kt + NS go into the stage that it has left.  (The last step
        // reads a stage that may hold nothing; without a LoRA term those fragments are not used.)
        RingFrags<C> fb[C::SUBS];
        ring_read_stage<C, COL, 0, C::SUBS * (MI + NI)>(fa, smem, wm, wn);
        const int stages = (nk + C::D - 1) / C::D, half_at = C::D == 2 && (nk & 1) ? stages - 1 : stages;
        auto step = [&](RingFrags<C> (&cur)[C::SUBS], RingFrags<C> (&nxt)[C::SUBS], int kt) {
            // half a stage at the end: the other half of it is zero (a second path with fewer MFMAs would move accumulators)
            if (C::D == 2 && kt == half_at) {
#pragma unroll
                for (int h = C::SUBS / 2; h < C::SUBS; ++h) {
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) cur[h].ft[mi] = bf16x8{};
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) cur[h].fo[ni] = bf16x8{};
                }
            }
            stage = stage + 1 == NS ? 0 : stage + 1;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            ring_stage<C, COL, 0>(acc, cur, nxt, smem + stage * C::STAGE, wm, wn);
        };
        int kt = 0;
        for (; kt + 1 < stages; kt += 2) {
            step(fa, fb, kt);
            step(fb, fa, kt + 1);
        }
        if (kt < stages) {
            step(fa, fb, kt);
#pragma unroll
            for (int h = 0; h < C::SUBS; ++h) fa[h] = fb[h];
        }
    } else {
        // Step kt computes slab kt.  The fragments of its second half are read while the first half's MFMAs run; then every
        // read of the stage is behind this wave, the copies of slab kt + 1 have landed, and one barrier makes both true for the
        // whole workgroup: the copies of slab kt + NS go into the stage just left.
        ring_read<C, COL>(fa[0], smem, 0, wm, wn);
        for (int kt = 0; kt < nk; ++kt) {
            const int next = stage + 1 == NS ? 0 : stage + 1;
            ring_half<C, COL, false, 0>(acc, fa[0], fa[1], smem + stage * C::STAGE, 1, wm, wn);
            ring_half<C, COL, true, 0>(acc, fa[1], fa[0], smem + next * C::STAGE, 0, wm, wn);
            stage = next;
        }
    }
    RingFrags<C>& f0 = fa[0];

    // LoRA term: (2) on the same accumulators; (5) by itself, masked and added
    const int rank_chunks = has_lora ? p.tb.a[rt.g].rank >> 3 : 0;
    if (has_lora) {
        // block rows of the tile from row `first` on into `to`; the fragments of sub-step 0 are in f0
        auto term = [&](auto& to, auto first) {
            constexpr int FIRST = first(), ROWS = sizeof(to) / sizeof(to[0]);
            ring_zero_past_rank<C>(f0, 0, rank_chunks);
            ring_mfma<C, true, FIRST, ROWS>(to, f0);
            if (rank_chunks > 4) {
                ring_read<C, COL>(f0, smem + stage * C::STAGE, 1, wm, wn);
                ring_mfma<C, false, FIRST, ROWS>(to, f0);
            }
            ring_mfma_done<ROWS, NI>(to);
        };
        if constexpr (!COL) {
            term(acc, std::integral_constant<int, 0>{});
        } else {
            ring_mfma_done<MI, NI>(acc);
            // half of the block rows at a time where there are four: t beside the accumulators is what the registers allow
            constexpr int ROWS = MI >= 4 ? MI / 2 : MI;
            auto part = [&](auto first) {
                f32x4 t[ROWS][NI];
#pragma unroll
                for (int mi = 0; mi < ROWS; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) t[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (first() > 0) ring_read<C, COL>(f0, smem + stage * C::STAGE, 0, wm, wn);
                term(t, first);
#pragma unroll
                for (int mi = 0; mi < ROWS; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int b = (first() + mi) * NI + ni, bit = 2 * (b & 7) + (e >> 1) + (e & 1) * 16;
                            const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)keep[b >> 3], bit, 1);
                            const float te = t[mi][ni][e];        // (a copy: bit_cast of a vector element reads element 0)
                            acc[first() + mi][ni][e] += __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, te) & m);
                        }
            };
            part(std::integral_constant<int, 0>{});
            if constexpr (ROWS < MI) part(std::integral_constant<int, ROWS>{});
        }
    } else {
        ring_mfma_done<MI, NI>(acc);
    }

    // Way out: the bf16 tile goes through LDS (rows of TN * 2 bytes, eight-byte slots XOR-ed so that the 16 rows x 2
    // slots a cycle writes are distinct) and whole tile rows are stored, 16 bytes per lane, non-temporally like those of the
    // large tiles: ordinary stores leave the tile in the L2s, to be written back when the kernel ends (one 128 x 256 tile per
    // compute unit: 64 x 2048 over 4096 rows 9.5 -> 8.3 us, 256 x 8192 over 1024 rows 11.6 -> 10.3; geometric mean over 740
    // sizes and all kinds 0.98).  No copy is in flight here: the last step of the loop waited for all of them.
    __syncthreads();
    constexpr int PITCH = C::TN * 2;
    auto swz = [](int row) { return C::TN >= 128 ? (row & 15) << 1 : C::TN == 64 ? ((row >> 1) & 7) << 1 : ((row >> 2) & 3) << 1; };
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int row = (wm * MI + mi) * 16 + (l & 15);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            u32x2 o;
            o.x = pack_bf16x2(acc[mi][ni][0], acc[mi][ni][1]);
            o.y = pack_bf16x2(acc[mi][ni][2], acc[mi][ni][3]);
            const int slot = (wn * NI + ni) * 4 + (l >> 4);
            *(u32x2*)(smem + row * PITCH + ((slot ^ swz(row)) << 3)) = o;
        }
    }
    __syncthreads();
    lora_bf16* res = p.res + (int64_t)rt.row_start * p.NC + c0;
    constexpr int CPR = C::TN / 8;                                    // 16-byte chunks per tile row
#pragma unroll
    for (int i = 0; i < (C::TM * CPR + C::THREADS - 1) / C::THREADS; ++i) {
        const int pos = i * C::THREADS + (int)threadIdx.x, row = pos / CPR, ch = pos % CPR;
        if (C::TM * CPR < C::THREADS && pos >= C::TM * CPR) break;
        const u32x4 v = *(const u32x4*)(smem + row * PITCH + ((ch ^ (swz(row) >> 1)) << 4));
        if (row < rt.rows && ch * 8 < cols_valid) __builtin_nontemporal_store(v, (u32x4*)(res + (int64_t)row * p.NC + ch * 8));
    }
}

template <class C, bool COL, class TB>
__global__ void __launch_bounds__(C::THREADS + 64 * C::CW) ring_gemm_kernel(RingArgsOf<TB> p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    ring_tile<C, COL>(p, smem);
}

// (5) and the strips of (4) and dB, neither of which needs the other, in one launch of DA_THREADS a workgroup (rule and figures at
// kStripsBeside); the waves that a tile has no work for end at once.  Bounded by the latency of one sweep over the contraction.
template <class C, int CB, class TB>
__global__ void __launch_bounds__(DA_THREADS, 4) ring_strips_kernel(RingStripsArgsOf<TB> p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tiles = p.tiles_m * p.tiles_n;
    if ((int)blockIdx.x >= tiles) {
        strip_of<CB>(p, blockIdx.x - tiles, smem);
        return;
    }
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) >= C::NW + C::CW) return;
    ring_tile<C, true>(p, smem);
}

template <class C, int CB>
static hipError_t launch_ring_strips_t(const RingStripsArgs& a, hipStream_t st) {
    static_assert(C::LDS >= strip_lds(CB) && C::THREADS + 64 * C::CW <= DA_THREADS, "a strip in a tile's LDS, a tile in a strip's threads");
    static_assert(2 * C::LDS <= 160 * 1024, "two workgroups on a compute unit (kStripsBeside)");
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = ring_strips_kernel<C, CB, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;                  // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)(b.tiles_m * b.tiles_n + b.a.blocks + b.b.blocks)), dim3(DA_THREADS), C::LDS, st, b);
        return hipGetLastError();
    });
}

template <class C, bool COL>
static hipError_t launch_ring_cfg(const RingArgs& a, hipStream_t st) {
    const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
    if (tiles == 0) return hipSuccess;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = ring_gemm_kernel<C, COL, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;                  // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(C::THREADS + 64 * C::CW), C::LDS, st, b);
        return hipGetLastError();
    });
}

// Which kernel of the family: see kRingTiles.  Two workgroups of kinds 2, 3 and 4 fit on a compute unit (their rings
// take 64 - 80 KB of LDS), one of the others.  Kind 5 is for launches of at most one workgroup per compute unit: the deeper
// ring and the single pass over the weight pay when that comes from HBM (77 rows, 4096 -> 14336, weight not cached: 64 x 128
// tiles 38 us, 128 x 64 tiles 32 us).
// Kind 3, ring of five stages / four, (2): 4096 -> 4096, 160 rows 13.1 / 13.8; (5): 8192 to 8192, 100 rows 29.2 / 28.1, 128 rows 31.2 / 29.6.
// Kind 4, half a tile to a workgroup while every half has a compute unit, in 128-deep stages with both stages' fragments in registers: a sweep is
// bound by the bytes that a slab brings to the compute unit (12 KB in 0.13 us, 8 KB in 0.08; longer rings gain nothing).  us, whole tiles of one slab to a stage /
// halves, (2): 1024 -> 1024, 16 rows 4.73 / 3.77, 256 rows 4.88 / 3.88; 2048 -> 2048, 128 rows 6.74 / 5.00; 4096 -> 4096, 16 rows 11.1 / 7.7, 64 rows
// 11.3 / 8.6; 26496 -> 960, 128 rows 53.9 / 36.5; (5): 1024 -> 1024, 256 rows 4.83 / 4.07; 2048 -> 2048, 128 rows 6.68 / 5.67; 4096 -> 4096, 64 rows
// 13.8 / 12.9; 8192 -> 1024, 64 rows 17.9 / 11.3; 4096 -> 2112, 64 rows 10.4 / 7.8; 2048 -> 960, 250 rows 6.8 / 6.4.
// Whole tiles have one slab to a stage, six of them.  (2): five / six: 4096 -> 4096, 100 rows 10.7 / 10.7, from HBM 15.5 / 15.0, 128 rows from HBM 16.8 / 16.9; 8192 ->
// 4096, 100 rows 18.1 / 18.0, from HBM 26.4 / 25.5; eight adapters of 1 - 16 rows, 8896 -> 20480 218 / 214; one slab to a stage / two: 448 -> 4160, 64 rows 3.85 /
// 4.04; 1024 -> 4096, 100 rows from HBM 5.41 / 5.62; 3968 -> 5440, 64 rows 11.2 / 12.0; 4096 -> 4096, 128 rows 11.5 / 12.3; 3072 -> 2112, 128 rows from HBM 13.1 / 13.0.
// (5): two computing and two copying waves, over long contractions four of each (14336 to 4096 columns, 128 rows 41.8 / 40.6; 8192 to 8192, 64 rows 28.1 /
// 27.2; 1024 to 1024, 256 rows 4.70 / 4.78, 512 to 14336 3.79 / 3.94).
// Only where a row of W is a multiple of 512 bytes, which puts the rows of a slab into few of the memory channels, do whole tiles of (5) take
// stages of two slabs, from contractions of 1024 on and while all of them run at once.  One slab / two, weight cached and from HBM: to 4096 columns,
// contraction of 1024, 128 rows 5.05 / 4.92, 5.97 / 5.91, of 2048 7.2 / 6.8, 13.0 / 12.1, of 4096, 96 rows 13.7 / 13.6, 21.9 / 21.0; to 8192, 4096, 64 rows
// 15.4 / 14.1, 22.8 / 21.9; to 2560, 6144, 128 rows 21.0 / 20.2, 33.8 / 31.9; but to 4032, 4096, 96 rows 11.5 / 12.2, 17.5 / 17.8; to 2112, 8192, 128 rows 18.9 / 20.1,
// 29.7 / 30.7; to 4160, 14336, 60 rows 31.1 / 33.7, 51.7 / 53.4; to 1088, 4096, 240 rows 10.8 / 11.0, 13.2 / 14.0; to 8064, 8192, 64 rows level; to 4096, 576, 110 rows
// 4.20 / 4.27, 4.74 / 4.84; 2560 tiles to 20480, 8896, of eight adapters 291 / 296 (a whole backward; 384 tiles to 8192, 4096, of three 40.5 / 40.0).
using Ring64x64 = Ring<64, 64, 2, 2, 5, 2, 2>;       // of the launches that take the strips
using Ring32x64 = Ring<32, 64, 2, 2, 3, 1, 2, 2>;    // two slabs to a stage
using Narrow32x64 = Ring<32, 64, 1, 2, 6, 1, 1>;     // four waves
using Ring32x32 = Ring<32, 32, 2, 2, 4, 2, 2, 2>;    // half of such a tile
constexpr int kLongContraction = 4096;
constexpr bool deep_stages(int KC, int NC, int64_t tiles) { return KC >= 1024 && NC % 256 == 0 && tiles <= 2 * kComputeUnits; }

// Calls f(kernel, arguments) with what a launch of tiles of `kind` takes.
template <bool COL, class F>
static auto with_ring(int kind, const RingArgs& a, F&& f) {
    switch (kind) {
        case 0: return f(Ring<128, 256, 2, 4, 3, 0, 4>{}, a);
        case 1: return f(Ring<128, 128, 2, 2, 4, 2, 2>{}, a);
        case 2: return f(Ring<64, 128, 2, 4, 3, 1, 2>{}, a);
        case 3: return f(Ring<64, 64, 2, 2, COL ? 4 : 5, 2, 2>{}, a);
        case 4:
            if (ring_halves(a.tiles_m, a.tiles_n)) {
                RingArgs h = a;
                h.tiles_n *= 2;
                return f(Ring32x32{}, h);
            }
            if constexpr (COL) {
                if (deep_stages(a.KC, a.NC, (int64_t)a.tiles_m * a.tiles_n)) return f(Ring32x64{}, a);
                return a.KC < kLongContraction ? f(Narrow32x64{}, a) : f(Ring<32, 64, 2, 2, 6, 2, 2>{}, a);
            } else {
                return f(Ring<32, 64, 2, 2, 6, 1, 2>{}, a);
            }
        default: return f(Ring<128, 64, 2, 2, 6, 2, 1>{}, a);
    }
}

// ... with the strips beside them: f(kernel, r / 16, arguments).
template <class F>
static auto with_ring_strips(int kind, const RingStripsArgs& a, F&& f) {
    auto of_rank = [&](auto c, const RingStripsArgs& b) {
        return b.r == 16 ? f(c, std::integral_constant<int, 1>{}, b) : f(c, std::integral_constant<int, 2>{}, b);
    };
    if (kind == 3) return of_rank(Ring64x64{}, a);
    // halves beside the strips: with a compute unit for each, or where the longer contraction makes up for sharing one (us, whole / half tiles, backward:
    // 256 x 1024 x 1024 8.9 / 9.4, r = 32 8.8 / 10.5; 200 rows, 2048 -> 1024 10.9 / 10.8; 64 x 4096 x 4096, r = 32 20.7 / 20.4; 300 rows, 4096 -> 512 16.6 / 15.6).
    // kStripsBeside bounds the whole tiles and the strips: with halves there are up to 640 workgroups, the last strips of which start when
    // the first halves have ended, and which still are the faster way (560 workgroups, five adapters of 20 rows, 4096 -> 1024 17.7 / 15.0, r = 32 18.5 /
    // 15.7; 640, four of 8 rows, 4096 -> 2048 18.3 / 16.4, r = 32 18.4 / 16.8).
    const bool own = 2 * a.tiles_m * a.tiles_n + a.a.blocks + a.b.blocks <= kComputeUnits;
    if (ring_halves(a.tiles_m, a.tiles_n) && (own || a.KC >= 2048)) {
        RingStripsArgs h = a;
        h.tiles_n *= 2;
        return of_rank(Ring32x32{}, h);
    }
    // whole tiles that share compute units: four waves instead of seven (20 rows of three adapters, 10048 -> 4288, r = 32, 402 workgroups 25.4 us, 26.5
    // with seven); by themselves the seven are faster (256 x 1024 x 1024 backward 10.2, 10.5 with four)
    if (a.tiles_m * a.tiles_n + a.a.blocks + a.b.blocks > kComputeUnits) return of_rank(Narrow32x64{}, a);
    return of_rank(Ring32x64{}, a);
}

template <bool COL>
static hipError_t launch_ring_dir(int kind, const RingArgs& a, hipStream_t st) {
    return with_ring<COL>(kind, a, [&](auto c, const RingArgs& b) { return launch_ring_cfg<decltype(c), COL>(b, st); });
}

hipError_t launch_ring(int kind, bool col, const RingArgs& a, hipStream_t st) {
    return col ? launch_ring_dir<true>(kind, a, st) : launch_ring_dir<false>(kind, a, st);
}

hipError_t launch_ring_strips(int kind, const RingStripsArgs& a, hipStream_t st) {
    return with_ring_strips(kind, a, [&](auto c, auto cb, const RingStripsArgs& b) { return launch_ring_strips_t<decltype(c), cb()>(b, st); });
}

template <class C>
static GemmLaunch describe(C, int64_t workgroups) { return GemmLaunch{C::TM, C::TN, C::DEPTH, C::NS, C::NW + C::CW, 0, workgroups}; }

GemmLaunch ring_launch(int kind, bool col, const RingArgs& a) {
    auto f = [](auto c, const RingArgs& b) { return describe(c, (int64_t)b.tiles_m * b.tiles_n); };
    return col ? with_ring<true>(kind, a, f) : with_ring<false>(kind, a, f);
}

GemmLaunch ring_strips_launch(int kind, const RingStripsArgs& a) {
    return with_ring_strips(kind, a, [](auto c, auto, const RingStripsArgs& b) {
        return describe(c, (int64_t)b.tiles_m * b.tiles_n + b.a.blocks + b.b.blocks);
    });
}

}  // namespace lf
