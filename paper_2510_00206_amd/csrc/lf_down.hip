// Operation (1) of the fused LoRA linear layer (Section 5.1, FusedLoRA Design): dropout and
// the down-projection in one pass over X,
//     S'[i,c] = s * q * sum_j keep(i,j) X[i,j] A[c,j],
// with the keep mask regenerated in registers from (seed, local row, column) and never stored.
// X is streamed once from HBM; A (r x K) stays cache resident.  Also the diagnostic mask writer.
//
// What bounds it: HBM once there are rows for every compute unit (8192 rows, K = 14336, r = 16: 37 us = 6.3 TB/s); below
// that the sweep of one workgroup over K, whose price is the number of vector memory instructions and of cache lines
// they touch (an instruction over 16 rows x 64 bytes costs the compute unit about 60 cycles, one over 8 rows x 128 bytes
// about 25), then the mask (12 vector instructions per column pair).  Hence X and A go global -> LDS in whole 128-byte
// lines, several stages of 256 columns ahead, by waves that do nothing else; A is fetched once per workgroup and stage, not
// once per wave; the masks of a stage are formed while its copies land, and not at all without dropout.
// Measured, us (cards differ by up to a tenth): fragments loaded straight into registers / copies by the computing waves / by waves of their
// own, 16 or 32 rows to a workgroup: K = 14336: 5003 rows r = 16 57 / 33.6 / 29.2, r = 64 128 / 39.5 / 35.0; K = 4096: 1024 rows r = 16 - / 7.9 / 7.2, r = 64 - /
// 11.2 / 8.7; 8192 rows r = 16 18 / 12.4 / 12.4, r = 64 - / 16.2 / 14.9; 19 rows, K = 24960, r = 16 - / 33.4 / 29.7, r = 64 - / 50.3 / 38.3.  In a kernel trace, those / as it
// is now, few rows in workgroups of eight and of a part of the rank: K = 4096, r = 16, 77 rows 7.5 / 6.8, 1024 rows 7.8 / 7.1, 2048 rows 8.2 / 7.6; r = 32, 500
// rows 8.0 / 7.1; r = 64, 1024 rows 9.5 / 8.4, 1531 rows 9.9 / 9.2; 19 rows, K = 24960, r = 16 29.3 / 23.7, r = 64 40.6 / 24.0.  Short contractions keep the registers
// (down_direct_kernel, rule in with_down).  The order of the sums is the same in both kernels and in every height, so S' has
// the same bits whichever is picked.
#include "lf_device.h"
#include "lf_gemm_parts.h"
#include "lf_internal.h"

namespace lf {

constexpr int DOWN_SLABS = 4;                       // 64-column slabs per stage
constexpr int DOWN_PARTS = 2 * DOWN_SLABS;          // a wave owns one half (32 columns) of one slab of every stage

// CB 16-column blocks of S' to a workgroup, PARTS workgroups to the call's rank; ROWS rows; ring of NS stages in LDS.  A wave computes for
// each column part or, with eight rows, for two of them: a lane then holds row l & 7 of part (l >> 3) & 1, and an MFMA for either
// part's columns of A has that part's sums in its half of the lanes.  Further waves copy, N KB of a stage each: XW of them rows of X,
// AW rows of A.
template <int CB_, int ROWS_, int NS_, int PARTS_ = 1>
struct Down {
    static constexpr int CB = CB_, ROWS = ROWS_, NS = NS_, PARTS = PARTS_;
    static constexpr bool PAIR = ROWS == 8;
    static constexpr int RB = PAIR ? 1 : ROWS / 16;                                        // fragments of rows
    static constexpr int WAVES = PAIR ? DOWN_PARTS / 2 : DOWN_PARTS, THREADS = 64 * WAVES; // that compute
    static constexpr int X_COPIES = DOWN_SLABS * ROWS / 8, A_COPIES = DOWN_SLABS * CB * 2; // 1 KB wave copies per stage
    static constexpr int XN = RB == 2 && CB < 4 ? 8 : 4, AN = CB == 4 || RB == 2 ? 8 : 4;    // ... per wave
    static constexpr int XW = X_COPIES / XN, AW = A_COPIES / AN;
    static constexpr int STAGE = (X_COPIES + A_COPIES) * 1024;
    static constexpr int LDS = NS * STAGE;
    static_assert(WAVES + XW + AW <= 16 && AN * (NS - 1) < 64, "a workgroup; the wait counter has six bits");
    static_assert(DOWN_PARTS * RB * CB * 1024 <= LDS, "the cross-wave sum goes through the ring");
};

template <int N, int I = 0>
__device__ __forceinline__ void down_copy(const char* src, const uint32_t (&off)[N], uint32_t m0) {
    if constexpr (I < N) {
        copy16_to_lds<pass_imm(N, I), I == 0>(src, off[I], m0);
        down_copy<N, I + 1>(src, off, m0);
    }
}

// A copying wave: copies N * w .. of every stage of one matrix, of which a slab has 8 * RP rows in RP copies; `last`: the last
// valid row (those past it repeat it), lds: the matrix's part of stage 0.  The barriers are those of the computing waves: one per
// stage, at which the stage has landed and the one before it is free.
template <class C, int N, int RP>
__device__ __forceinline__ void down_copier(int w, const lora_bf16* mat, int K, int last, int st, int nslabs, int nst, uint32_t lds) {
    const int l = threadIdx.x & 63;
    const char* base = (const char*)mat - kCopyBias;
    const uint32_t m0 = lds + w * (N * 1024) + (N / 2) * 1024;
    const int partial = nslabs % DOWN_SLABS;            // slabs of the last stage, if it is not full
    uint32_t off[N], off_last[N];                       // (slabs past K: copies of the last one, never used)
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int q = w * N + i, slab = q / RP, row = q % RP * 8 + (l >> 3);
        const uint32_t e = (uint32_t)min(row, last) * (uint32_t)K + (((l & 7) ^ row_slab_swz(row)) << 3);
        off[i] = (e + slab * BK) * 2 + kCopyBias - pass_imm(N, i);
        off_last[i] = (e + (partial ? min(slab, partial - 1) : slab) * BK) * 2 + kCopyBias - pass_imm(N, i);
    }
    auto issue = [&](int ring) {
        const char* src = base + (int64_t)st * (DOWN_SLABS * BK * 2);
        if (st == nst - 1) down_copy<N>(src, off_last, m0 + ring * C::STAGE);
        else down_copy<N>(src, off, m0 + ring * C::STAGE);
        st = st + 1 == nst ? 0 : st + 1;
    };
    constexpr int NS = C::NS;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nst) issue(s);
    int ring = NS - 1;
    for (int s = 0; s < nst; ++s) {
        if (s + NS - 2 < nst) wait_slab_loads_but<N*(NS - 2)>();
        else wait_slab_loads();
        asm volatile("s_barrier" ::: "memory");
        if (s + NS - 1 < nst) issue(ring);
        ring = ring + 1 == NS ? 0 : ring + 1;
    }
}

// Fixed-order sum over the column parts ([DOWN_PARTS][RB][CB][4 * RL] in LDS, RL rows to a block), scaled by s*q and rounded once to
// bf16, into columns c0 .. of S'.
template <int CB, int RB, int THREADS, int RL = 16, class TB>
__device__ __forceinline__ void down_store(const DownArgsOf<TB>& p, const RowTile& rt, const f32x4* red, int c0 = 0) {
    const float sq = p.tb.a[rt.g].s * p.tb.a[rt.g].q;
    constexpr int BLOCK = 4 * RL;
    for (int idx = threadIdx.x; idx < RB * CB * BLOCK; idx += THREADS) {
        const int lane = idx % BLOCK, cb = idx / BLOCK % CB, rb = idx / BLOCK / CB;
        f32x4 v = red[idx];
#pragma unroll
        for (int ww = 1; ww < DOWN_PARTS; ++ww) v += red[ww * (RB * CB * BLOCK) + idx];
        if (c0 + cb * 16 >= p.tb.a[rt.g].rank) v = f32x4{0.f, 0.f, 0.f, 0.f};
        const int row = rb * 16 + lane % RL;
        if (row < rt.rows) {
            u32x2 out;
            out.x = pack_bf16x2(v[0] * sq, v[1] * sq);
            out.y = pack_bf16x2(v[2] * sq, v[3] * sq);
            *(u32x2*)(p.S + (int64_t)(rt.row_start + row) * p.r + c0 + cb * 16 + 4 * (lane / RL)) = out;
        }
    }
}

template <class C, class TB>
__global__ void __launch_bounds__(C::THREADS + 64 * (C::XW + C::AW)) down_kernel(DownArgsOf<TB> p) {
    fetch_args<DownArgsOf<TB>>();
    constexpr int CB = C::CB, RB = C::RB, NS = C::NS;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    RowTile rt;
    if (!find_row_tile_by_lanes(p.tb, C::ROWS, blockIdx.x, rt)) return;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = rt.g, c0 = C::PARTS == 1 ? 0 : blockIdx.y * (CB * 16);          // this workgroup's first column of S'
    const int nslabs = p.K / BK, nst = (nslabs + DOWN_SLABS - 1) / DOWN_SLABS;
    // Every workgroup starts its sweep over K at a different stage (a function of its 32-row group within the segment,
    // so that single- and multi-adapter calls, and workgroups of every height, sum in the same order): workgroups sweeping
    // in lockstep would all hit the same few L2 channels, the row pitch being a multiple of the channel interleave.
    int st = (int)(((unsigned)(rt.local_row0 / 32) * 5u) % (unsigned)nst);
    if (w >= C::WAVES) {
        const int cw = w - C::WAVES;
        const uint32_t lds = lds_addr_of(smem);
        if (cw < C::XW)
            down_copier<C, C::XN, C::ROWS / 8>(cw, p.X + (int64_t)rt.row_start * p.K, p.K, rt.rows - 1, st, nslabs, nst, lds);
        else
            down_copier<C, C::AN, 2 * CB>(cw - C::XW, p.A + ((int64_t)g * p.r + c0) * p.K, p.K, max(p.tb.a[g].rank - c0, 1) - 1, st, nslabs, nst,
                                          lds + C::X_COPIES * 1024);
        return;
    }
    const int pos = C::PAIR ? w : w >> 1, sub = C::PAIR ? (l >> 3) & 1 : w & 1;  // this wave's slab and half of it (PAIR: this lane's half)
    const int lrow = C::PAIR ? l & 7 : l & 15;
    const uint32_t T = p.tb.a[g].T;
    const KeepThreshold th = keep_threshold(T);

    RowKey rk[RB];
    constexpr int H = C::PAIR ? 2 : 1;                  // halves that a wave forms
    f32x4 acc[H * RB][CB];
    u32x4 keep[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        rk[rb] = row_key(p.tb.a[g].k0, p.tb.a[g].k1, (uint32_t)(rt.local_row0 + rb * 16 + lrow));
        keep[rb] = u32x4{~0u, ~0u, ~0u, ~0u};
    }
#pragma unroll
    for (int i = 0; i < H * RB; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[i][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // keep masks of this lane's 8 columns in stage t
    auto form_masks = [&](int t) {
        const uint32_t x0 = (uint32_t)((t * DOWN_SLABS + pos) * (BK / 2) + 16 * sub + 4 * (l >> 4)) * kGold;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                keep[rb][i] = keep_pair_mask(hash_word_at(rk[rb], rk[rb].a + x0 + (uint32_t)i * kGold), th);
    };
    const char* xs = smem + pos * C::ROWS * 128 + row_slab_off(lrow, 4 * sub + (l >> 4));
    const char* as[H];
#pragma unroll
    for (int h = 0; h < H; ++h)
        as[h] = smem + C::X_COPIES * 1024 + pos * (CB * 2048) + row_slab_off(l & 15, 4 * (C::PAIR ? h : sub) + (l >> 4));

    int ring = 0;
    for (int s = 0; s < nst; ++s) {
        if (T) form_masks(st);                          // while the stage's copies land
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        u32x4 x[RB];
        bf16x8 a[H][CB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) x[rb] = *(const u32x4*)(xs + ring * C::STAGE + rb * 2048);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) a[h][cb] = __builtin_bit_cast(bf16x8, *(const u32x4*)(as[h] + ring * C::STAGE + cb * 2048));
        __builtin_amdgcn_sched_barrier(0);
        if (st * DOWN_SLABS + pos < nslabs) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                x[rb] &= keep[rb];
                const bf16x8 xf = __builtin_bit_cast(bf16x8, x[rb]);
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)            // (the call's rank: columns past the adapter's are zeroed on the way out)
                        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[h * RB + rb][cb]) : "v"(a[h][cb]), "v"(xf));
            }
        }
        st = st + 1 == nst ? 0 : st + 1;
        ring = ring + 1 == NS ? 0 : ring + 1;
    }

    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
    for (int i = 0; i < H * RB; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) asm volatile("" : "+v"(acc[i][cb]));
    __syncthreads();
    f32x4* red = (f32x4*)smem;                             // [DOWN_PARTS][RB][CB][64], PAIR: [DOWN_PARTS][CB][32]
    if constexpr (C::PAIR) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            f32x4 v = acc[0][cb];
            const f32x4 other = acc[H - 1][cb];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = v[e], y = other[e];
                v[e] = sub ? y : x;
            }
            red[((2 * w + sub) * CB + cb) * 32 + (l >> 4) * 8 + lrow] = v;
        }
    } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) red[((w * RB + rb) * CB + cb) * 64 + l] = acc[rb][cb];
    }
    __syncthreads();
    down_store<CB, RB, C::THREADS, C::PAIR ? 8 : 16>(p, rt, red, c0);
}

// The same sums without LDS: wave w loads the fragments of column part w of every stage straight into registers, D stages
// ahead.  No stage to fill and 64 KB of LDS at most, so several workgroups share a compute unit and cover for each other:
// the faster way where a workgroup's sweep is short against its start and its end (see with_down).
template <int CB, int RB, class TB>
__global__ void __launch_bounds__(64 * DOWN_PARTS) down_direct_kernel(DownArgsOf<TB> p) {
    fetch_args<DownArgsOf<TB>>();
    __shared__ f32x4 red[DOWN_PARTS * RB * CB * 64];
    RowTile rt;
    if (!find_row_tile(p.tb, 16 * RB, blockIdx.x, rt)) return;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = rt.g;
    const uint32_t T = p.tb.a[g].T;
    const KeepThreshold th = keep_threshold(T);
    const int cbn = p.tb.a[g].rank >> 4;                  // 16-column blocks this adapter uses (<= CB)
    const lora_bf16* Ag = p.A + (int64_t)g * p.r * p.K + (int64_t)(l & 15) * p.K;
    const lora_bf16* xrow[RB];
    RowKey rk[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = rb * 16 + (l & 15);
        xrow[rb] = p.X + (int64_t)(rt.row_start + min(row, rt.rows - 1)) * p.K;
        rk[rb] = row_key(p.tb.a[g].k0, p.tb.a[g].k1, (uint32_t)(rt.local_row0 + row));
    }
    f32x4 acc[RB][CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

    constexpr int D = CB == 1 ? 4 : 2;
    const int nchunks = p.K / 32, nst = (nchunks + DOWN_PARTS - 1) / DOWN_PARTS;
    struct Regs { u32x4 x[RB], a[CB]; } ring[D];
    int st = (int)(((unsigned)(rt.local_row0 / 32) * 5u) % (unsigned)nst), st_load = st;      // as in down_kernel
    auto advance = [&](int& t) { t = t + 1 == nst ? 0 : t + 1; };
    auto load = [&](Regs& c) {                            // (a part past K is never used)
        const int chunk = st_load * DOWN_PARTS + w, col = chunk * 32 + 8 * (l >> 4);
        advance(st_load);
        if (chunk >= nchunks) return;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) c.x[rb] = *(const u32x4*)(xrow[rb] + col);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            if (CB == 1 || cb < cbn) c.a[cb] = *(const u32x4*)(Ag + (int64_t)(cb * 16) * p.K + col);
    };
    auto consume = [&](const Regs& c) {
        const int chunk = st * DOWN_PARTS + w;
        advance(st);
        if (chunk >= nchunks) return;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const u32x4 x = T ? mask8(c.x[rb], rk[rb], (uint32_t)(chunk * 32 + 8 * (l >> 4)), th) : c.x[rb];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                if (CB == 1 || cb < cbn)
                    acc[rb][cb] = LF_MFMA(__builtin_bit_cast(bf16x8, c.a[cb]), __builtin_bit_cast(bf16x8, x), acc[rb][cb]);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < nst) load(ring[d]);
    for (int s = 0; s < nst; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (s + d < nst) {
                consume(ring[d]);
                if (s + d + D < nst) load(ring[d]);
            }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) red[((w * RB + rb) * CB + cb) * 64 + l] = acc[rb][cb];
    __syncthreads();
    down_store<CB, RB, 64 * DOWN_PARTS>(p, rt, red);
}

template <class C>
static hipError_t launch_down_cfg(const DownArgs& a, int tiles, hipStream_t st) {
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = down_kernel<C, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;                  // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3(tiles, C::PARTS), dim3(C::THREADS + 64 * (C::XW + C::AW)), C::LDS, st, b);
        return hipGetLastError();
    });
}

template <int CB, int RB>
static hipError_t launch_down_direct(const DownArgs& a, int tiles, hipStream_t st) {
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = down_direct_kernel<CB, RB, std::decay_t<decltype(b.tb)>>;
        hipLaunchKernelGGL(kernel, dim3(tiles), dim3(64 * DOWN_PARTS), 0, st, b);
        return hipGetLastError();
    });
}

template <int V> using IC = std::integral_constant<int, V>;

// Calls ring(kernel, row tiles) or direct(r / 16, 16-row blocks, row tiles) with what the launch takes.
template <class R, class D>
static auto with_down(const DownArgs& a, int forced, R&& ring, D&& direct) {
    int tiles32 = 0, tiles16 = 0, tiles8 = 0;
    for (int g = 0; g < a.tb.G; ++g) {
        const int len = a.tb.row0[g + 1] - a.tb.row0[g];
        tiles32 += (len + 31) / 32;
        tiles16 += (len + 15) / 16;
        tiles8 += (len + 7) / 8;
    }
    // A 16-row workgroup takes 0.65 - 0.8 of a 32-row one's time (its copies of A serve half as many rows), so it is the
    // faster one exactly while all of them run at once: K = 14336, r = 64: 4096 rows 29 against 36 us, 5003 rows 50
    // against 37 us; r = 16: 21 against 30 and 30 against 31 us.
    const bool one_round = tiles16 <= kComputeUnits, many = tiles32 > kComputeUnits;
    const bool small = forced ? forced == 128 : one_round;
    // Short contractions: a ring of one or two stages has nothing to run ahead of, and its LDS leaves room for one or two
    // workgroups on a compute unit, which tells when they come in several rounds (us, direct / ring): K = 64, r = 64: 5000
    // rows 3.8 / 4.7, 100000 rows 21 / 43; K = 256: r = 16 1000 rows 3.2 / 3.5, r = 64 16384 rows 6.9 / 9.4; K = 320, 1000 rows
    // r = 16 3.4 / 3.9, r = 64 4.6 / 4.5; K = 512: r = 64 5000 rows 6.4 / 5.6, 40000 rows 19 / 24, r = 16 16384 rows 6.6 / 5.9 (the line is
    // drawn for the larger ranks); K = 768: r = 32 40000 rows 18 / 20, r = 16 16384 rows 8.4 / 7.6.
    const int direct_up_to = !many ? 320 : a.r == 32 && tiles32 > 2 * kComputeUnits ? 768 : 512;
    if (a.K <= direct_up_to) {
        if (a.r == 16) return small ? direct(IC<1>{}, IC<1>{}, tiles16) : direct(IC<1>{}, IC<2>{}, tiles32);
        if (a.r == 32) return small ? direct(IC<2>{}, IC<1>{}, tiles16) : direct(IC<2>{}, IC<2>{}, tiles32);
        return small ? direct(IC<4>{}, IC<1>{}, tiles16) : direct(IC<4>{}, IC<2>{}, tiles32);
    }
    // r = 32: two of the 16-row workgroups fit on a compute unit, one of the 32-row ones (128 KB of LDS); in several rounds
    // that is worth more than the second reading of A up to K = 2048 (40000 rows: K = 1024 22 / 25 us, K = 2048 33 / 40, K = 4096 69 / 65).
    const bool small32 = forced ? forced == 128 : one_round || (many && a.K <= 2048);
    // A stage takes a workgroup the longer of its masks (16 rows 0.22 us: two waves of them to a SIMD) and its copies (X and A, 100 KB/us), so
    // while all workgroups run at once it is given eight rows, and as few of the rank's columns as that leaves room for; 16 rows by half the
    // columns at r = 64 (A is four fifths of its copies).  A forward over N = 256, operands from HBM, us, 16 rows by all columns / now: r = 16, K = 4096,
    // 77 rows without dropout 16.6 / 13.6, 1024 rows 18.7 / 15.4, 2048 rows 23.9 / 23.0; K = 2048, 1000 rows 12.6 / 11.0; r = 32, K = 4096, 500 rows 19.0 /
    // 15.2, 2000 rows 25.2 / 24.9; r = 64, 400 rows 20.3 / 15.7, 1531 rows 27.6 / 24.6; N = 64, operands cached and
    // from HBM: K = 384, r = 16, 1000 rows 6.6 / 6.4, 7.1 / 6.9, r = 64, 500 rows 7.3 / 6.6, 7.8 / 7.0; K = 1024, r = 16, 2048 rows 8.3 / 8.1, 8.7 / 8.8 (the least of 60
    // sizes), r = 64, 2048 rows 9.2 / 8.9, 9.7 / 9.3; K = 14336, r = 64, 1000 rows 46.6 / 42.3, 64.7 / 49.2.  Same bits.
    auto fits = [&](int tiles, int parts) { return !forced && tiles * parts <= kComputeUnits; };
    if (a.r == 16) {
        if (fits(tiles8, 1)) return ring(Down<1, 8, 6>{}, tiles8);
        return small ? ring(Down<1, 16, 5>{}, tiles16) : ring(Down<1, 32, 3>{}, tiles32);
    }
    if (a.r == 32) {
        if (fits(tiles8, 2)) return ring(Down<1, 8, 6, 2>{}, tiles8);
        if (fits(tiles8, 1)) return ring(Down<2, 8, 5>{}, tiles8);
        return small32 ? ring(Down<2, 16, 3>{}, tiles16) : ring(Down<2, 32, 4>{}, tiles32);
    }
    if (fits(tiles8, 4)) return ring(Down<1, 8, 6, 4>{}, tiles8);
    if (fits(tiles8, 2)) return ring(Down<2, 8, 5, 2>{}, tiles8);
    if (fits(tiles16, 2)) return ring(Down<2, 16, 4, 2>{}, tiles16);
    return small ? ring(Down<4, 16, 4>{}, tiles16) : ring(Down<4, 32, 3>{}, tiles32);
}

hipError_t launch_down(const DownArgs& a, int forced, hipStream_t st) {
    if (a.tb.row0[a.tb.G] == 0) return hipSuccess;
    if (a.r != 16 && a.r != 32 && a.r != 64) return hipErrorInvalidValue;
    return with_down(a, forced, [&](auto c, int tiles) { return launch_down_cfg<decltype(c)>(a, tiles, st); },
                     [&](auto cb, auto rb, int tiles) { return launch_down_direct<cb(), rb()>(a, tiles, st); });
}

DownLaunch down_launch(const DownArgs& a, int forced) {
    return with_down(a, forced, [](auto c, int tiles) { using C = decltype(c); return DownLaunch{C::ROWS, C::PARTS, 1, (int64_t)tiles * C::PARTS}; },
                     [](auto, auto rb, int tiles) { return DownLaunch{16 * rb(), 1, 0, tiles}; });
}

// keep[i,j] for one adapter, one thread per column pair
__global__ void debug_mask_kernel(int64_t M, int64_t K, uint32_t T, uint32_t k0, uint32_t k1, uint8_t* keep) {
    const int64_t pairs = (K + 1) >> 1;
    const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (idx >= M * pairs) return;
    const int64_t row = idx / pairs, cp = idx - row * pairs;
    const uint32_t wd = hash_word(row_key(k0, k1, (uint32_t)row), (uint32_t)cp);
    keep[row * K + 2 * cp] = (wd & 0xFFFFu) >= T;
    if (2 * cp + 1 < K) keep[row * K + 2 * cp + 1] = (wd >> 16) >= T;
}

hipError_t launch_debug_mask(int64_t M, int64_t K, uint32_t T, uint32_t k0, uint32_t k1, uint8_t* keep,
                             hipStream_t st) {
    const int64_t n = M * ((K + 1) >> 1);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(debug_mask_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, M, K, T, k0, k1, keep);
    return hipGetLastError();
}

}  // namespace lf
