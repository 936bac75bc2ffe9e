// Operations (2) and (5) of the fused LoRA linear layer (Section 5.1, FusedLoRA Design) on small output tiles:
// the launches whose 256- or 192-row tiles of lf_gemm.hip would leave most compute units without work.
//   (2)  Y  = X W + S' B                     out operand W [N,K], B [N,r]: contiguous along the contraction
//   (5)  dX = dY W^T + mask*q*(dS A^T)       out operand W [N,K], A [r,K]: contraction over the rows
// Every output element is formed by the same MFMAs in the same order as on the large tiles (contraction in steps of
// 32 from zero, then the LoRA term), so Y and dX are bit-identical whichever kernel a launch picks.
//
// What bounds them: with one small tile on a compute unit neither the matrix pipe nor memory is busy; a 64-deep slab
// costs its MFMAs plus about 0.1 us in which the waves meet, read their first fragments and issue copies (128 x 128:
// 0.33 us a slab against 0.21 us of MFMAs; without the copies 0.23 us, without the barrier 0.28 us), and with every
// compute unit loaded the copies out of L2 (0.47 us a slab).  Hence: a ring of three to six slabs in LDS, copied
// global -> LDS several slabs ahead (a slab then has about a microsecond to arrive), one barrier per slab, fragments
// read one sub-step ahead, eight waves where the tile has work for them, and two workgroups on a compute unit for the
// tiles whose ring leaves room.  Accumulators are vector registers, the MFMAs assembly (see ring_mfma): the compiler's
// own moved every accumulator block in every step (M = 1024, 4096 x 4096: 40 -> 35 us).
// Measured, one launch, against the 128-row tiles that served these sizes before: 256 x 1024 x 1024 16 -> 6.1 us
// forward, 22 -> 6.7 us backward; 1024 x 4096 x 4096 56 -> 35 and 66 -> 39 us; 77 rows, 4096 -> 14336 51 -> 24 and
// (backward) 174 -> 41 us; 64 rows, 15616 -> 320 176 -> 33 us.
#include <type_traits>

#include "lf_device.h"
#include "lf_gemm_parts.h"
#include "lf_gemm_ring.h"
#include "lf_internal.h"

namespace lf {

// One kernel of the family.  TM x TN output tile, WM x WN waves of (TM / WM) x (TN / WN) each, ring of NS LDS stages,
// one 64-deep slab pair per stage.
template <int TM_, int TN_, int WM_, int WN_, int NS_>
struct Ring {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, NS = NS_;
    static constexpr int NW = WM * WN, THREADS = 64 * NW;
    static constexpr int MI = TM / WM / 16, NI = TN / WN / 16;        // 16x16 blocks per wave
    static constexpr int PASS_TOK = TM / 8;                           // wave copies (1 KB) of a token slab
    static constexpr int PASSES = (TM + TN) / 8 / NW;                 // ... of a slab pair, per wave
    static constexpr int STAGE = (TM + TN) * BK * 2;
    static constexpr int LDS = NS * STAGE;
    static_assert((TM + TN) / 8 % NW == 0 && PASSES <= 8, "the copies of a slab pair divide evenly over the waves");
    static_assert(NS >= 2, "ring depth");
    static_assert(PASSES * (NS - 1) < 64, "the wait counter has six bits");
    static_assert(TM * TN * 2 <= LDS, "the way out goes through the ring");
};

// Column-operand slab of TN columns: 64 contraction rows of TN * 2 bytes, chunk index XOR-ed so that the 32 lanes of a
// transposing read ({a..a+3, a+8..a+11} x 32 bytes) cover 256 distinct bytes mod 256.  128 columns and more: as in the
// large tiles; 64 (32) columns: two (four) rows share 256 bytes, so only row bits 1 and 3 (bit 3) choose among a row's windows.
template <int TN>
__device__ __forceinline__ int ring_col_swz(int row) {
    return TN >= 128 ? col_slab_swz(row) : TN == 64 ? (row & 2) | ((row & 8) >> 1) : (row & 8) >> 2;
}

// Source offsets of a lane for the copies of one slab pair (bytes from the token or the out slab's first element).
// Copies are numbered token slab first; wave w issues numbers PASSES*w .. +PASSES-1.
template <class C> struct RingLanes { uint32_t off[C::PASSES]; };

// tok_chunks / out_chunks: valid 16-byte chunks along the contraction (8, or r / 8 for the LoRA slab);
// out_rows (COL): valid contraction rows (64, or r).
template <class C, bool COL>
__device__ __forceinline__ RingLanes<C> ring_lanes(int w, uint32_t tok_ld, uint32_t out_ld, int tok_rows, int out_cols,
                                                   int chunks, int out_rows) {
    const int l = threadIdx.x & 63;
    RingLanes<C> s;
#pragma unroll
    for (int i = 0; i < C::PASSES; ++i) {
        const int q = w * C::PASSES + i;
        uint32_t e;                                                   // < 2^30: at most 256 rows of 2^22 elements
        if (q < C::PASS_TOK) {
            const int row = 8 * q + (l >> 3);
            e = (uint32_t)min(row, tok_rows - 1) * tok_ld + min((l & 7) ^ row_slab_swz(row), chunks - 1) * 8;
        } else if (!COL) {
            const int row = 8 * (q - C::PASS_TOK) + (l >> 3);
            e = (uint32_t)min(row, out_cols - 1) * out_ld + min((l & 7) ^ row_slab_swz(row), chunks - 1) * 8;
        } else {
            constexpr int CPR = C::TN / 8;                            // chunks per slab row
            const int pos = (q - C::PASS_TOK) * 64 + l, row = pos / CPR;
            e = (uint32_t)min(row, out_rows - 1) * out_ld + min((pos % CPR) ^ ring_col_swz<C::TN>(row), (out_cols >> 3) - 1) * 8;
        }
        s.off[i] = e * 2 + kCopyBias - pass_imm(C::PASSES, i);
    }
    return s;
}

// Copies I .. END-1 of this wave.  tok / out: slab addresses - kCopyBias; m0: its destination (middle of its PASSES KB)
template <class C, int I = 0, int END = C::PASSES>
__device__ __forceinline__ void ring_issue(int w, const char* tok, const char* out, const RingLanes<C>& s, uint32_t m0) {
    if constexpr (I < END) {
        copy16_to_lds<pass_imm(C::PASSES, I), I == 0>(w * C::PASSES + I < C::PASS_TOK ? tok : out, s.off[I], m0);
        ring_issue<C, I + 1, END>(w, tok, out, s, m0);
    }
}

template <class C> struct RingFrags { bf16x8 ft[C::MI], fo[C::NI]; };

// Fragment number J of sub-step `sub` (32 contraction elements) of the slab pair at `st`, in the order of first use:
// token block 0, the out blocks, the other token blocks.
template <class C, bool COL, int J>
__device__ __forceinline__ void ring_read_one(RingFrags<C>& f, const char* st, int sub, int wm, int wn) {
    const int l = threadIdx.x & 63;
    const int off = row_slab_off(l & 15, 4 * sub + (l >> 4));
    if constexpr (J == 0 || J > C::NI) {
        constexpr int mi = J == 0 ? 0 : J - C::NI;
        f.ft[mi] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + off + (wm * C::MI + mi) * 2048));
    } else {
        constexpr int ni = J - 1;
        const char* so = st + C::TM * BK * 2;
        const int blk = wn * C::NI + ni;
        if constexpr (COL) {
            constexpr int PITCH = C::TN * 2;
            const int row = 8 * (l >> 4) + ((l & 15) >> 2), col = (l & 3) << 2;
            const int o = row * PITCH + (((col >> 3) ^ ring_col_swz<C::TN>(row)) << 4) + ((col & 7) << 1);
            const int a = (o ^ (blk << 5)) + sub * 32 * PITCH;
            f.fo[ni] = join_tr(lds_read_tr(so, a), lds_read_tr(so, a + 4 * PITCH));
        } else {
            f.fo[ni] = __builtin_bit_cast(bf16x8, *(const u32x4*)(so + off + blk * 2048));
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

// All MFMAs of a sub-step, from assembly with the accumulators tied in place: with the builtin the compiler moves
// accumulator blocks between registers in every step of the loop.  OPS_FROM_VALU: the operands may come straight from
// the vector ALU (zero_past_rank); the compiler keeps the wait states that needs only for its own MFMAs.
template <class C, bool OPS_FROM_VALU>
__device__ __forceinline__ void ring_mfma(f32x4 (&acc)[C::MI][C::NI], const RingFrags<C>& f) {
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < C::NI; ++ni) {
            if constexpr (OPS_FROM_VALU)
                asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(f.fo[ni]), "v"(f.ft[mi]));
            else
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(f.fo[ni]), "v"(f.ft[mi]));
        }
}
// ... and the distance to the vector ALU's first read of their results.
template <class C>
__device__ __forceinline__ void ring_mfma_done(f32x4 (&acc)[C::MI][C::NI]) {
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < C::NI; ++ni) asm volatile("" : "+v"(acc[mi][ni]));
}

template <class C>
__device__ __forceinline__ void ring_zero_past_rank(RingFrags<C>& f, int sub, int rank_chunks) {
    const int chunk = 4 * sub + ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int mi = 0; mi < C::MI; ++mi) f.ft[mi] = zero_past_rank(f.ft[mi], chunk, rank_chunks);
#pragma unroll
    for (int ni = 0; ni < C::NI; ++ni) f.fo[ni] = zero_past_rank(f.fo[ni], chunk, rank_chunks);
}

// Waits until all but the VM newest copies of the wave have landed and, with LGKM, all its LDS reads have returned.
// The builtin, not assembly: the compiler counts it, and does not wait again for reads it orders before.
template <int VM, bool LGKM>
__device__ __forceinline__ void ring_wait() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | ((LGKM ? 0 : 15) << 8) | ((VM >> 4) << 14));
    asm volatile("" ::: "memory");
}

// One sub-step of a slab: its MFMAs, and between them the reads of the fragments `nxt` (sub-step nxt_sub of the slab at
// `st`) and, in the second sub-step (HAND), the hand-over to the next slab and the copies of a slab.  A wave issues in
// order, so the three have to be mixed by hand.  With four or fewer MFMAs a sub-step the reads go out in its first half, so
// that the last one has returned when the hand-over (or the next sub-step) needs it, and the hand-over sits a quarter
// into the second sub-step; with more the reads spread evenly.
template <class C> struct RingSlots {
    static constexpr int SLOTS = C::MI * C::NI, READS = C::MI + C::NI, P = C::PASSES;
    static constexpr bool SHORT = SLOTS < 8;
    static constexpr int HAND_AT = SHORT ? SLOTS / 4 : 0;                       // hand-over before this slot's MFMA
    static constexpr int first(bool hand) { return hand ? HAND_AT : 0; }        // first slot that carries reads
    static constexpr int span(bool hand) { return SHORT ? (SLOTS - first(hand) + 1) / 2 : SLOTS; }   // ... and how many do
    static constexpr int reads_before(bool hand, int s) {
        const int k = s - first(hand);
        return k <= 0 ? 0 : k >= span(hand) ? READS : k * READS / span(hand);
    }
    static constexpr int copies_before(int s) {
        const int k = s - HAND_AT, n = SLOTS - HAND_AT;
        return k <= 0 ? 0 : k * P / n;
    }
};

template <class C, bool COL, bool HAND, bool COPY, int I, class F>
__device__ __forceinline__ void ring_half(f32x4 (&acc)[C::MI][C::NI], const RingFrags<C>& cur, RingFrags<C>& nxt, const char* st,
                                          int nxt_sub, int w, int wm, int wn, const char* tok, const char* out,
                                          const RingLanes<C>& lanes, uint32_t m0, F& hand_over) {
    using S = RingSlots<C>;
    if constexpr (I < S::SLOTS) {
        constexpr int mi = I / C::NI, ni = I % C::NI;
        if constexpr (HAND && I == S::HAND_AT) hand_over();
        ring_read<C, COL, S::reads_before(HAND, I), S::reads_before(HAND, I + 1)>(nxt, st, nxt_sub, wm, wn);
        if constexpr (COPY) ring_issue<C, S::copies_before(I), S::copies_before(I + 1)>(w, tok, out, lanes, m0);
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(cur.fo[ni]), "v"(cur.ft[mi]));
        __builtin_amdgcn_sched_barrier(0);
        ring_half<C, COL, HAND, COPY, I + 1>(acc, cur, nxt, st, nxt_sub, w, wm, wn, tok, out, lanes, m0, hand_over);
    }
}

template <class C, bool COL, class TB>
__global__ void __launch_bounds__(C::THREADS) ring_gemm_kernel(RingArgsOf<TB> p) {
    constexpr int NS = C::NS, MI = C::MI, NI = C::NI;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int tm, tn;
    tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm, tn);
    RowTile rt;
    if (!find_row_tile(p.tb, C::TM, tm, rt, p.row_lo, p.row_hi)) return;
    const int c0 = tn * C::TN, cols_valid = min(C::TN, p.NC - c0);
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w % C::WM, wn = w / C::WM;
    const bool has_lora = p.r > 0;
    const int nk = p.KC / BK, nkt = nk + (has_lora ? 1 : 0);

    const int out_ld = COL ? p.NC : p.KC;
    const char* tok_src = (const char*)(p.tok + (int64_t)rt.row_start * p.KC) - kCopyBias;
    const char* out_src = (const char*)(COL ? p.out + c0 : p.out + (int64_t)c0 * p.KC) - kCopyBias;
    const int64_t out_adv = COL ? (int64_t)BK * p.NC * 2 : BK * 2;
    const uint32_t m0 = lds_addr_of(smem) + w * (C::PASSES * 1024) + (C::PASSES / 2) * 1024;
    const RingLanes<C> base_lanes = ring_lanes<C, COL>(w, p.KC, out_ld, rt.rows, cols_valid, 8, BK);

    // Slab `kt` into stage `stage`: a base slab pair, the LoRA pair [S' | B] resp. [dS | A] (kt == nk), or nothing.
    auto issue_base = [&](int stage) {
        ring_issue<C>(w, tok_src, out_src, base_lanes, m0 + stage * C::STAGE);
        tok_src += BK * 2;
        out_src += out_adv;
    };
    auto issue = [&](int kt, int stage) {
        if (kt < nk) {
            issue_base(stage);
        } else if (kt < nkt) {
            const lora_bf16* lt = p.ltok + (int64_t)rt.row_start * p.r;
            const lora_bf16* lo = COL ? p.lout + (int64_t)rt.g * p.r * p.NC + c0 : p.lout + ((int64_t)rt.g * p.NC + c0) * p.r;
            const RingLanes<C> s = ring_lanes<C, COL>(w, p.r, COL ? p.NC : p.r, rt.rows, cols_valid, p.r >> 3, p.r);
            ring_issue<C>(w, (const char*)lt - kCopyBias, (const char*)lo - kCopyBias, s, m0 + stage * C::STAGE);
        }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s)
        issue(s, s);

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

    if (nkt >= NS) ring_wait<C::PASSES*(NS - 1), false>();
    else ring_wait<0, false>();
    asm volatile("s_barrier" ::: "memory");

    // Step kt computes slab kt.  The fragments of its second half are read while the first half's MFMAs run; then
    // every read of the stage is behind this wave, the copies of slab kt + 1 have landed, and one barrier makes both
    // true for the whole workgroup: the copies of slab kt + NS go into the stage just left.  (The last step reads
    // fragments of a stage that may hold nothing; without a LoRA term they are not used.)
    int stage = 0;
    RingFrags<C> f0, f1;
    ring_read<C, COL>(f0, smem, 0, wm, wn);
    auto step = [&](int kt, auto steady) {
        const int next = stage + 1 == NS ? 0 : stage + 1;
        auto hand_over = [&] {
            if (steady() || kt + NS <= nkt) ring_wait<C::PASSES*(NS - 2), true>();
            else ring_wait<0, true>();
            asm volatile("s_barrier" ::: "memory");
            if (!steady()) issue(kt + NS, stage);
        };
        ring_half<C, COL, false, false, 0>(acc, f0, f1, smem + stage * C::STAGE, 1, w, wm, wn, tok_src, out_src, base_lanes, 0u,
                                           hand_over);
        ring_half<C, COL, true, steady(), 0>(acc, f1, f0, smem + next * C::STAGE, 0, w, wm, wn, tok_src, out_src, base_lanes,
                                             m0 + stage * C::STAGE, hand_over);
        if (steady()) {
            tok_src += BK * 2;
            out_src += out_adv;
        }
        stage = next;
    };
    int kt = 0;
    for (; kt + NS < nk; ++kt) step(kt, std::true_type{});
    for (; kt < nk; ++kt) step(kt, std::false_type{});

    // LoRA term: (2) on the same accumulators; (5) by itself, masked and added
    const int rank_chunks = has_lora ? p.tb.a[rt.g].rank >> 3 : 0;
    if (has_lora) {
        f32x4 t[MI][NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) t[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto term = [&](f32x4 (&to)[MI][NI]) {
            ring_zero_past_rank<C>(f0, 0, rank_chunks);
            ring_mfma<C, true>(to, f0);
            if (rank_chunks > 4) {
                ring_read<C, COL>(f1, smem + stage * C::STAGE, 1, wm, wn);
                ring_mfma<C, false>(to, f1);
            }
            ring_mfma_done<C>(to);
        };
        if constexpr (!COL) {
            term(acc);
        } else {
            term(t);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int b = mi * NI + ni, bit = 2 * (b & 7) + (e >> 1) + (e & 1) * 16;
                        const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)keep[b >> 3], bit, 1);
                        const float te = t[mi][ni][e];            // (a copy: bit_cast of a vector element reads element 0)
                        acc[mi][ni][e] += __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, te) & m);
                    }
        }
    } else {
        ring_mfma_done<C>(acc);
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
    for (int i = 0; i < C::TM * CPR / C::THREADS; ++i) {
        const int pos = i * C::THREADS + (int)threadIdx.x, row = pos / CPR, ch = pos % CPR;
        const u32x4 v = *(const u32x4*)(smem + row * PITCH + ((ch ^ (swz(row) >> 1)) << 4));
        if (row < rt.rows && ch * 8 < cols_valid) __builtin_nontemporal_store(v, (u32x4*)(res + (int64_t)row * p.NC + ch * 8));
    }
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
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(C::THREADS), C::LDS, st, b);
        return hipGetLastError();
    });
}


// Which kernel of the family: see kRingTiles.  Two workgroups of kinds 2, 3 and 4 fit on a compute unit (their rings
// take 64 - 72 KB of LDS), one of the others.  Kind 5 is for launches of at most one workgroup per compute unit: the deeper
// ring and the single pass over the weight pay when that comes from HBM (77 rows, 4096 -> 14336, weight not cached: 64 x 128
// tiles 38 us, 128 x 64 tiles 32 us).
template <bool COL>
static hipError_t launch_ring_dir(int kind, const RingArgs& a, hipStream_t st) {
    switch (kind) {
        case 0: return launch_ring_cfg<Ring<128, 256, 2, 4, 3>, COL>(a, st);
        case 1: return launch_ring_cfg<Ring<128, 128, 2, 4, 4>, COL>(a, st);
        case 2: return launch_ring_cfg<Ring<64, 128, 2, 4, 3>, COL>(a, st);
        case 3: return launch_ring_cfg<Ring<64, 64, 2, 2, 4>, COL>(a, st);
        case 4: return launch_ring_cfg<Ring<32, 64, 2, 2, 6>, COL>(a, st);
        case 5: return launch_ring_cfg<Ring<128, 64, 4, 2, 6>, COL>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_ring(int kind, bool col, const RingArgs& a, hipStream_t st) {
    return col ? launch_ring_dir<true>(kind, a, st) : launch_ring_dir<false>(kind, a, st);
}

}  // namespace lf
