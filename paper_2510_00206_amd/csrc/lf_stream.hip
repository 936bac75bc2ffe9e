// Operation (3) of the fused LoRA linear layer (Section 5.1, FusedLoRA Design), both results from a single read of dY:
//     dS[i,c] = s sum_n dY[i,n] B[n,c]   and   dB[n,c] = sum_i dY[i,n] S'[i,c]
// A workgroup owns a (row panel of 64 .. 1024 rows) x (512-column chunk) panel of dY and walks it in 32-row steps: the
// rows go global -> LDS in whole lines, NS - 1 steps ahead, and are read twice from there, with transposing reads for the
// row-contracted product dB and plainly for dS.  Results are partial sums (dB per row panel, dS per column
// chunk) that the finalize kernels add in a fixed order, so repeated runs agree bit for bit.  Also the finalize kernels.
#include "lf_device.h"
#include "lf_gemm_parts.h"
#include "lf_internal.h"

namespace lf {

constexpr int ST_THREADS = 512;
constexpr int ST_STEP = 32;                        // rows per step
constexpr int ST_BIG_BYTES = ST_STEP * kStreamChunk * 2;   // 32 KB

#define LF_MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a), (b), (c), 0, 0, 0)

__device__ __forceinline__ bf16x8 read_tr_frag(const char* lds, int r0, int c0, int nchunk) {
    const int l = threadIdx.x & 63;
    const s16x4 lo = lds_read_tr(lds, tr_off(r0, c0, l & 15, nchunk));
    const s16x4 hi = lds_read_tr(lds, tr_off(r0 + 4, c0, l & 15, nchunk));
    return join_tr(lo, hi);
}

__device__ __forceinline__ bf16x8 read_panel_tr_frag(const char* lds, int r0, int c0) {
    const int l = threadIdx.x & 63;
    const s16x4 lo = lds_read_tr(lds, panel_tr_off(r0, c0, l & 15));
    const s16x4 hi = lds_read_tr(lds, panel_tr_off(r0 + 4, c0, l & 15));
    return join_tr(lo, hi);
}

template <int CB_, int NS_>     // r / 16, ring depth in steps
struct Stream {
    static constexpr int CB = CB_, NS = NS_;
    static constexpr int STAGE = ST_BIG_BYTES + CB * 1024;              // rows of dY, rows of S'
    static constexpr int RED = 6 * CB * 1024;                           // dS of a step: quarters 1 .. 3 x two row blocks
    static constexpr int LDS = NS * STAGE + 2 * RED;
    // B (16 CB KB) passes through the ring's last stages at the start
    static constexpr int B_STAGES = (kStreamChunk * CB * 32 + STAGE - 1) / STAGE, FIRST = NS - B_STAGES;   // stages free for dY
    static_assert(FIRST >= 1, "the first step's rows and B are in flight together");
    static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
};

// Elements of a row-contracted fragment (lane: contraction rows 8 * (l >> 4) .. +7) at or past `rows` become zero.
__device__ __forceinline__ bf16x8 zero_past_rows(bf16x8 v, int rows) {
    u32x4 u = __builtin_bit_cast(u32x4, v);
    const int left = rows - 8 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] &= left >= 2 * i + 2 ? 0xFFFFFFFFu : left == 2 * i + 1 ? 0x0000FFFFu : 0u;
    return __builtin_bit_cast(bf16x8, u);
}

template <class C, class TB>
__global__ void __launch_bounds__(ST_THREADS, 2) stream_kernel(StreamArgsOf<TB> p) {
    fetch_args<StreamArgsOf<TB>>();
    constexpr int CB = C::CB, NS = C::NS, R = CB * 16, RCH = CB * 2;     // rank, 16-byte chunks per S' row
    extern __shared__ __attribute__((aligned(16))) char smem[];
    f32x4* red = (f32x4*)(smem + NS * C::STAGE);

    // Consecutive workgroup ids go to different XCDs (private L2s).  The column chunk is skewed by the
    // row tile so that one XCD does not end up reading a single column window of every row (which
    // would crowd a few of its L2 channels, the row pitch being a multiple of the channel interleave).
    const int tile = blockIdx.x / p.chunks;
    const int chunk_id = (int)((blockIdx.x - tile * p.chunks + tile) % p.chunks);
    RowTile rt;
    if (!find_panel(p.tb, p.panel_rows, tile, rt)) return;
    const int c0 = chunk_id * kStreamChunk;
    const int cols_valid = min(kStreamChunk, p.C - c0);       // multiple of 64
    const int t = threadIdx.x, l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int quarter = w & 3, rb = w >> 2;                   // this wave's part of dS: 128 columns, 16 of the 32 rows
    const int g = rt.g;
    const int rank_g = p.tb.a[g].rank, cbn = rank_g >> 4;       // columns / 16-column blocks this adapter uses
    // either output may be switched off (null pointer): the unfused baseline runs them as separate passes
    const bool do_red = p.part_out != nullptr, do_ds = p.part_ds != nullptr;
    const int nsteps = (rt.rows + ST_STEP - 1) / ST_STEP;

    // Copies of a step: wave w brings rows 4w .. 4w+3 of dY, and waves 0 .. CB-1 one KB of S' each.  Rows past the end of
    // the panel repeat its last row (the S' fragments are zero there), columns past the end the last valid chunk (never
    // stored).
    const char* big = (const char*)(p.big + (int64_t)rt.row_start * p.C + c0) - kCopyBias;
    const char* small_ = (const char*)(p.small_ + (int64_t)rt.row_start * R) - kCopyBias;
    uint32_t off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        off[i] = (uint32_t)(min(l ^ panel_swz(4 * w + i), (cols_valid >> 3) - 1) * 16 + kCopyBias - pass_imm(4, i));
    const uint32_t lds0 = lds_addr_of(smem);
    auto issue = [&](int step, int stage) {
        const uint32_t m0 = lds0 + stage * C::STAGE + w * 4096 + 2048;
        const int row = step * ST_STEP + 4 * w, last = rt.rows - 1;
        copy16_to_lds<pass_imm(4, 0), true>(big + (int64_t)min(row, last) * p.C * 2, off[0], m0);
        copy16_to_lds<pass_imm(4, 1), false>(big + (int64_t)min(row + 1, last) * p.C * 2, off[1], m0);
        copy16_to_lds<pass_imm(4, 2), false>(big + (int64_t)min(row + 2, last) * p.C * 2, off[2], m0);
        copy16_to_lds<pass_imm(4, 3), false>(big + (int64_t)min(row + 3, last) * p.C * 2, off[3], m0);
        if (w < CB) {
            const int pos = w * 64 + l, srow = pos / RCH, ch = (pos % RCH) ^ (swz(srow) & (RCH - 1));
            const uint32_t so = (uint32_t)(min(step * ST_STEP + srow, last) * R + ch * 8) * 2 + kCopyBias;
            copy16_to_lds<0, true>(small_, so, lds0 + stage * C::STAGE + ST_BIG_BYTES + w * 1024);
        }
    };
    // B fragments of this wave's quarter, kept in registers: [32-column block][16-column block of the rank].  The chunk's
    // rows come in first, then those of the first steps; blocks past the last column or the adapter's rank are zero.
    bf16x8 bf[4][CB];
    char* lds_b = smem + C::FIRST * C::STAGE;
    if (do_ds) {
        const char* Bg = (const char*)(p.Bmat + ((int64_t)g * p.C + c0) * R) - kCopyBias;
#pragma unroll
        for (int i = 0; i < 2 * CB; ++i) {
            const int q = w * 2 * CB + i, pos = q * 64 + l, row = pos / RCH, ch = (pos % RCH) ^ (swz(row) & (RCH - 1));
            copy16_to_lds<0, true>(Bg, (uint32_t)(min(row, cols_valid - 1) * R + ch * 8) * 2 + kCopyBias, lds_addr_of(lds_b) + q * 1024);
        }
    }
#pragma unroll
    for (int s = 0; s < C::FIRST && s < NS - 1; ++s)
        if (s < nsteps) issue(s, s);
    if (do_ds) {
        constexpr int after = C::FIRST < NS - 1 ? C::FIRST : NS - 1;         // steps asked for after B
        if (nsteps < after) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (w < CB) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(5 * after) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * after) : "memory");
        asm volatile("s_barrier" ::: "memory");
#pragma unroll
        for (int kq = 0; kq < 4; ++kq)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int col = quarter * 128 + kq * 32;
                bf[kq][cb] = read_tr_frag(lds_b, col + 8 * (l >> 4), cb * 16, RCH);
                if (col >= cols_valid || cb >= cbn) bf[kq][cb] = bf16x8{};
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");
    }
#pragma unroll
    for (int s = C::FIRST; s < NS - 1; ++s)
        if (s < nsteps) issue(s, s);

    f32x4 acc[4][CB], hold[CB];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[jb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) hold[cb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // dS of step s, one step late (its quarters meet at the next step's barrier): wave 0 for rows 0 .. 15, wave 4 for 16 .. 31
    auto store_ds = [&](int s) {
        const int row = s * ST_STEP + rb * 16 + (l & 15);
        const f32x4* rd = red + (s & 1) * (C::RED / 16) + rb * (CB * 64) + l;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const f32x4 v = ((hold[cb] + rd[cb * 64]) + rd[(2 * CB + cb) * 64]) + rd[(4 * CB + cb) * 64];
            if (row < rt.rows)
                *(f32x4*)(p.part_ds + ((int64_t)chunk_id * p.M + rt.row_start + row) * R + cb * 16 + 4 * (l >> 4)) = v;
        }
    };

    int stage = 0;
    for (int s = 0; s < nsteps; ++s) {
        // this step's copies have landed for every wave, and every wave has left the stage that the next copies overwrite
        if (s + NS - 2 >= nsteps) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        else if (w < CB) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(5 * (NS - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(4 * (NS - 2)) : "memory");
        asm volatile("s_barrier" ::: "memory");
        if (s + NS - 1 < nsteps) issue(s + NS - 1, stage == 0 ? NS - 1 : stage - 1);
        const char* lds_big = smem + stage * C::STAGE;
        const char* lds_small = lds_big + ST_BIG_BYTES;
        if (do_ds && quarter == 0 && s > 0) store_ds(s - 1);
        if (do_red) {
            // reduction over the step's 32 rows: this wave owns panel columns [64w, 64w+64)
            const int rows_left = rt.rows - s * ST_STEP;
            bf16x8 fs[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                fs[cb] = read_tr_frag(lds_small, 8 * (l >> 4), cb * 16, RCH);
                if (rows_left < ST_STEP) fs[cb] = zero_past_rows(fs[cb], rows_left);
            }
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                const bf16x8 fb = read_panel_tr_frag(lds_big, 8 * (l >> 4), w * 64 + jb * 16);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[jb][cb] = LF_MFMA16(fs[cb], fb, acc[jb][cb]);    // D[c][n]
            }
        }
        if (do_ds) {
            f32x4 ads[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) ads[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kq = 0; kq < 4; ++kq) {
                const u32x4 tv = *(const u32x4*)(lds_big + panel_off(rb * 16 + (l & 15), quarter * 16 + kq * 4 + (l >> 4)));
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    ads[cb] = LF_MFMA16(bf[kq][cb], __builtin_bit_cast(bf16x8, tv), ads[cb]);          // D[c][i]
            }
            if (quarter == 0) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) hold[cb] = ads[cb];
            } else {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    red[(s & 1) * (C::RED / 16) + (((quarter - 1) * 2 + rb) * CB + cb) * 64 + l] = ads[cb];
            }
        }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    if (do_ds) {
        __syncthreads();
        if (quarter == 0) store_ds(nsteps - 1);
    }

    // partial dB [tile][n][c] of this panel
    if (do_red)
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
        const int colb = w * 64 + jb * 16;
        if (colb >= cols_valid) continue;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int n = c0 + colb + (l & 15), c = cb * 16 + 4 * (l >> 4);
            // past the adapter's rank S' is zero, but zero times a non-finite dY is not: the padding of dB is set to zero here
            *(f32x4*)(p.part_out + ((int64_t)tile * p.C + n) * R + c) = cb < cbn ? acc[jb][cb] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
}

template <class C>
static hipError_t launch_stream_t(StreamArgs a, hipStream_t st) {
    if (a.panel_rows < ST_STEP) return hipErrorInvalidValue;
    a.tiles_m = count_panels(a.tb, a.panel_rows);
    a.chunks = (a.C + kStreamChunk - 1) / kStreamChunk;
    if (a.tiles_m == 0) return hipSuccess;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = stream_kernel<C, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;                  // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3(a.tiles_m * a.chunks), dim3(ST_THREADS), C::LDS, st, b);
        return hipGetLastError();
    });
}

hipError_t launch_stream_dsdb(StreamArgs a, hipStream_t st) {
    switch (a.r) {
        case 16: return launch_stream_t<Stream<1, 4>>(a, st);
        case 32: return launch_stream_t<Stream<2, 4>>(a, st);
        case 64: return launch_stream_t<Stream<4, 3>>(a, st);
    }
    return hipErrorInvalidValue;
}

// ---- finalize: fixed-order sums of the partials ---------------------------------------------------
// job 1: dS[i, c..c+3] = bf16(s_g * q_g * sum_chunks part_ds);  job 2: dB[g, n, c..c+3] (+)= sum over tiles of g
template <class TB>
__global__ void __launch_bounds__(256) finalize_ds_db_kernel(FinalizeArgsOf<TB> p, int blocks_ds) {
    fetch_args<FinalizeArgsOf<TB>>();
    const int r4 = p.r >> 2;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < p.n_zero; i += gridDim.x * 256) p.zero[i] = 0;
    if ((int)blockIdx.x < blocks_ds) {
        const int64_t idx = blockIdx.x * 256ll + threadIdx.x;
        if (idx >= (int64_t)p.M * r4) return;
        const int row = (int)(idx / r4);
        // dS leaves here scaled by s*q: the survivor scale q of the dropout that operations (4) and (5)
        // owe their LoRA terms is applied once, to the small matrix, instead of per element of dA and dX
        const int seg = segment_of_row(p.tb, row);
        const float s = p.tb.a[seg].s * p.tb.a[seg].q;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int ch = 0; ch < p.chunks; ++ch) v += *(const f32x4*)(p.part_ds + ((int64_t)ch * p.M * r4 + idx) * 4);
        u32x2 o;
        o.x = pack_bf16x2(v[0] * s, v[1] * s);
        o.y = pack_bf16x2(v[2] * s, v[3] * s);
        *(u32x2*)(p.dS + idx * 4) = o;
    } else {
        const int64_t per_g = (int64_t)p.N * r4;
        const int64_t idx = (blockIdx.x - blocks_ds) * 256ll + threadIdx.x;
        if (idx >= per_g * p.tb.G) return;
        const int g = (int)(idx / per_g);
        const int64_t e = idx - g * per_g;
        int reg0, nreg, extra;
        segment_planes(p.tb, p.panel_rows_db, g, reg0, nreg, extra);
        if (nreg == 0 && extra < 0 && p.accumulate) return;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int tl = reg0; tl < reg0 + nreg; ++tl) v += *(const f32x4*)(p.part_db + ((int64_t)tl * per_g + e) * 4);
        if (extra >= 0) v += *(const f32x4*)(p.part_db + ((int64_t)extra * per_g + e) * 4);
        f32x4* out = (f32x4*)(p.dB + idx * 4);
        *out = p.accumulate ? *out + v : v;
    }
}

// dA[g, c, j..j+3] (+)= sum over the row tiles of segment g (q_g is already in dS)
template <class TB>
__global__ void __launch_bounds__(256) finalize_da_kernel(FinalizeArgsOf<TB> p) {
    fetch_args<FinalizeArgsOf<TB>>();
    const int64_t per_g = (int64_t)p.r * (p.K >> 2);
    const int64_t idx = blockIdx.x * 256ll + threadIdx.x;
    if (idx >= per_g * p.tb.G) return;
    const int g = (int)(idx / per_g);
    const int64_t e = idx - g * per_g;
    int reg0, nreg, extra;
    segment_planes(p.tb, p.panel_rows_da, g, reg0, nreg, extra);
    if (nreg == 0 && extra < 0 && p.accumulate) return;
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int tl = reg0; tl < reg0 + nreg; ++tl) v += *(const f32x4*)(p.part_da + ((int64_t)tl * per_g + e) * 4);
    if (extra >= 0) v += *(const f32x4*)(p.part_da + ((int64_t)extra * per_g + e) * 4);
    f32x4* out = (f32x4*)(p.dA + idx * 4);
    *out = p.accumulate ? *out + v : v;
}

hipError_t launch_finalize_ds_db(const FinalizeArgs& a, hipStream_t st) {
    const int64_t n_ds = a.part_ds ? (int64_t)a.M * (a.r >> 2) : 0;
    const int64_t n_db = a.part_db ? (int64_t)a.tb.G * a.N * (a.r >> 2) : 0;
    if (n_ds + n_db == 0) return hipSuccess;
    const int blocks_ds = (int)((n_ds + 255) / 256), blocks_db = (int)((n_db + 255) / 256);
    if (n_db && a.panel_rows_db < 64) return hipErrorInvalidValue;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = finalize_ds_db_kernel<std::decay_t<decltype(b.tb)>>;
        hipLaunchKernelGGL(kernel, dim3(blocks_ds + blocks_db), dim3(256), 0, st, b, blocks_ds);
        return hipGetLastError();
    });
}

hipError_t launch_finalize_da(const FinalizeArgs& a, hipStream_t st) {
    const int64_t n = (int64_t)a.tb.G * a.r * (a.K >> 2);
    if (a.panel_rows_da < 64) return hipErrorInvalidValue;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = finalize_da_kernel<std::decay_t<decltype(b.tb)>>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, b);
        return hipGetLastError();
    });
}

}  // namespace lf
