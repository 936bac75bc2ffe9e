// dS of operation (3) by itself (Section 5.1, FusedLoRA Design), for the launches whose pass over dY is short:
//     dS[i,c] = s q sum_n dY[i,n] B[n,c]        (bf16, as operations (4) and (5) take it)
// A workgroup owns 16 rows (and of the rank's columns all, or a part: rule in launch_ds) and sweeps all of N, so that dS leaves
// it finished: no partial sums and no second launch.  The other half of the operation, dB, then runs beside operation (4)
// (lf_da.hip), whose strips read dY a second time.
#include "lf_device.h"
#include "lf_gemm_parts.h"
#include "lf_internal.h"

namespace lf {

constexpr int DS_ROWS = 16;

// CB * 16 of the call's RANK columns to a workgroup, PARTS workgroups to 16 rows; stages of SC columns of dY and as many rows of B, ring of NS stages in LDS.  A task is a quarter (128
// columns) of a 512-column chunk by 16 columns of the rank, four MFMAs; there is a wave for every task of a stage.  CW more
// waves do nothing but copy: a copy holds the wave that issues it up until the memory pipeline takes it, and forty of them a
// stage, shared among the waves with the tasks, took longer than the tasks.
template <int CB_, int SC_, int NS_, int CW_, int RANK_ = CB_ * 16>
struct Ds {
    static constexpr int CB = CB_, SC = SC_, NS = NS_, CW = CW_, RANK = RANK_, PARTS = RANK / (CB * 16);
    static constexpr int QUARTERS = SC / 128, TASKS = QUARTERS * CB;
    static constexpr int Y_COPIES = SC * DS_ROWS * 2 / 1024, B_COPIES = SC * CB * 32 / 1024;   // 1 KB wave copies per stage
    static constexpr int P = (Y_COPIES + B_COPIES) / CW;                                        // ... per copying wave
    static constexpr int THREADS = 64 * (TASKS + CW);
    static constexpr int STAGE = (Y_COPIES + B_COPIES) * 1024;
    static constexpr int RED = TASKS * 1024;                                                    // results of a stage's tasks
    static constexpr int LDS = NS * STAGE + 2 * RED;
    static_assert(SC == 512 || SC == 256, "a stage is a whole or half a chunk of the summation order");
    static_assert((Y_COPIES + B_COPIES) % CW == 0 && P <= 8 && P * (NS - 1) < 64, "copies per wave; the wait counter has six bits");
    static_assert(THREADS <= 1024 && LDS <= 160 * 1024, "a workgroup; LDS of a compute unit");
};

template <class C, int I = 0>
__device__ __forceinline__ void ds_copy(const char* const (&src)[C::P], const uint32_t (&off)[C::P], uint32_t m0) {
    if constexpr (I < C::P) {
        copy16_to_lds<pass_imm(C::P, I), I == 0>(src[I], off[I], m0);
        ds_copy<C, I + 1>(src, off, m0);
    }
}

// Every dS element is summed in the order of the two-launch form (stream_kernel, finalize_ds_db_kernel): four MFMAs from
// zero per quarter, ((q0 + q1) + q2) + q3 per chunk, then chunk by chunk; dS is the same bits either way.
template <class C, class TB>
__global__ void __launch_bounds__(C::THREADS) ds_kernel(DsArgsOf<TB> p) {
    fetch_args<DsArgsOf<TB>>();
    constexpr int CB = C::CB, SC = C::SC, NS = C::NS, P = C::P, R = C::RANK, RCH = CB * 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    if (C::PARTS == 1 || blockIdx.y == 0)
        for (int i = blockIdx.x * C::THREADS + threadIdx.x; i < p.n_zero; i += gridDim.x * C::THREADS) p.zero[i] = 0;
    RowTile rt;
    if (!find_row_tile_by_lanes(p.tb, DS_ROWS, blockIdx.x, rt)) return;
    f32x4* red = (f32x4*)(smem + NS * C::STAGE);
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = C::PARTS == 1 ? 0 : blockIdx.y * (CB * 16);                   // this workgroup's first column of dS
    const int g = rt.g, cbn = (p.tb.a[g].rank - c0) >> 4;  // 16-column blocks this adapter uses of them
    const int nst = (p.C + SC - 1) / SC;
    if (w >= C::TASKS) {                                  // a copying wave
        const int cw = w - C::TASKS;
        const char* dY = (const char*)(p.dY + (int64_t)rt.row_start * p.C) - kCopyBias;
        const char* Bg = (const char*)(p.Bmat + (int64_t)g * p.C * R + c0) - kCopyBias;
        const uint32_t m0 = lds_addr_of(smem) + cw * (P * 1024) + (P / 2) * 1024;
        // Its copies of a stage: dY first (rows past the tile repeat the last one), then B.  `cols`: the stage's columns;
        // copies past them repeat the last ones (never used).
        auto lanes = [&](uint32_t (&off)[P], int cols) {
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int q = cw * P + i;
                uint32_t e;
                if (q < C::Y_COPIES) {
                    constexpr int CPR = SC / 8;           // chunks per row
                    const int pos = q * 64 + l, row = pos / CPR;
                    e = (uint32_t)min(row, rt.rows - 1) * (uint32_t)p.C + min((pos % CPR) ^ panel_swz(row), (cols >> 3) - 1) * 8;
                } else {
                    const int pos = (q - C::Y_COPIES) * 64 + l, row = pos / RCH;
                    e = (uint32_t)(min(row, cols - 1) * R + ((pos % RCH) ^ (swz(row) & (RCH - 1))) * 8);
                }
                off[i] = e * 2 + kCopyBias - pass_imm(P, i);
            }
        };
        uint32_t off[P];
        lanes(off, SC);
        auto issue = [&](int st, int ring) {
            const char* src[P];
#pragma unroll
            for (int i = 0; i < P; ++i)
                src[i] = cw * P + i < C::Y_COPIES ? dY + (int64_t)st * (SC * 2) : Bg + (int64_t)st * (SC * R * 2);
            if (st == nst - 1 && p.C % SC) lanes(off, p.C % SC);
            ds_copy<C>(src, off, m0 + ring * C::STAGE);
        };
#pragma unroll
        for (int s = 0; s < NS - 1; ++s)
            if (s < nst) issue(s, s);
        int ring = NS - 1;
        for (int s = 0; s < nst; ++s) {
            // this wave's copies of stage s have landed; behind the barrier every wave's have, and the stage before is free
            if (s + NS - 2 < nst) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(P*(NS - 2)) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            asm volatile("s_barrier" ::: "memory");
            if (s + NS - 1 < nst) issue(s + NS - 1, ring);
            ring = ring + 1 == NS ? 0 : ring + 1;
        }
        asm volatile("s_barrier" ::: "memory");           // (the last one of the waves with tasks)
        return;
    }

    const int quarter = w % C::QUARTERS, cb = w / C::QUARTERS;                   // this wave's task
    const bool sums = quarter == 0;                                              // ... and it adds up the quarters of its 16 columns
    f32x4 total = f32x4{0.f, 0.f, 0.f, 0.f}, half = total;
    auto add_stage = [&](int s) {
        const f32x4* rd = red + (s & 1) * (C::RED / 16) + cb * (C::QUARTERS * 64) + l;
        if constexpr (SC == 512) {
            total += ((rd[0] + rd[64]) + rd[128]) + rd[192];
        } else if (s & 1) {
            total += (half + rd[0]) + rd[64];
        } else {
            half = rd[0] + rd[64];
            if (s == nst - 1) total += half;              // (the other half of the chunk is past N)
        }
    };

    const int y_off = (l & 15) * (SC * 2);
    int y_col[4], b_off[4][2];
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) {
        const int n0 = quarter * 128 + kq * 32 + 8 * (l >> 4);
        y_col[kq] = y_off + (((quarter * 16 + kq * 4 + (l >> 4)) ^ panel_swz(l & 15)) << 4);
        b_off[kq][0] = C::Y_COPIES * 1024 + tr_off(n0, cb * 16, l & 15, RCH);
        b_off[kq][1] = C::Y_COPIES * 1024 + tr_off(n0 + 4, cb * 16, l & 15, RCH);
    }
    int ring = 0;
    for (int s = 0; s < nst; ++s) {
        // the stage has landed; this wave is done with the stage before and with the results of the one before that
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // fragments first, all of them: read one by one between the MFMAs they cost their latency four times a stage
        const char* stage = smem + ring * C::STAGE;
        u32x4 y[4];
        bf16x8 b[4];
#pragma unroll
        for (int kq = 0; kq < 4; ++kq) {
            y[kq] = *(const u32x4*)(stage + y_col[kq]);
            b[kq] = join_tr(lds_read_tr(stage, b_off[kq][0]), lds_read_tr(stage, b_off[kq][1]));
        }
        __builtin_amdgcn_sched_barrier(0);
        const int left = p.C - s * SC - quarter * 128;    // valid columns from the quarter's first
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        if (cb < cbn) {
            if (left >= 128) {
#pragma unroll
                for (int kq = 0; kq < 4; ++kq) acc = LF_MFMA(b[kq], __builtin_bit_cast(bf16x8, y[kq]), acc);      // D[c][i]
            } else if (left > 0) {                        // (a multiple of 64)
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) acc = LF_MFMA(b[kq], __builtin_bit_cast(bf16x8, y[kq]), acc);
            }
        }
        red[(s & 1) * (C::RED / 16) + (cb * C::QUARTERS + quarter) * 64 + l] = acc;
        if (sums && s > 0) add_stage(s - 1);              // one stage late: its tasks have met at this barrier
        ring = ring + 1 == NS ? 0 : ring + 1;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (sums) {
        add_stage(nst - 1);
        const float sq = p.tb.a[g].s * p.tb.a[g].q;
        if ((l & 15) < rt.rows) {
            u32x2 o;
            o.x = pack_bf16x2(total[0] * sq, total[1] * sq);
            o.y = pack_bf16x2(total[2] * sq, total[3] * sq);
            *(u32x2*)(p.dS + (int64_t)(rt.row_start + (l & 15)) * R + c0 + cb * 16 + 4 * (l >> 4)) = o;
        }
    }
}

template <class C>
static hipError_t launch_ds_t(const DsArgs& a, int tiles, hipStream_t st) {
    if (tiles == 0 && a.n_zero == 0) return hipSuccess;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = ds_kernel<C, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;                  // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3(tiles ? tiles : 1, C::PARTS), dim3(C::THREADS), C::LDS, st, b);
        return hipGetLastError();
    });
}

hipError_t launch_ds(const DsArgs& a, hipStream_t st) {
    int tiles = 0;
    for (int g = 0; g < a.tb.G; ++g) tiles += (a.tb.row0[g + 1] - a.tb.row0[g] + DS_ROWS - 1) / DS_ROWS;
    // A workgroup is bound by its copies, four fifths of which are rows of B at r = 64 (0.6 us a stage of 256 columns): while
    // all of them run at once, several share 16 rows, each with columns of its own.  With the strips after it, us, one workgroup / two /
    // four: r = 64: 16 x 4096 x 4096 18.9 / 14.6 / 12.1 (one pass over dY 16.7), 1024 x 4096 x 4096 26.5 / 21.9 / 21.7, 2048 x 4096 x 4096
    // 37.2 / 32.7 / - (35.1); r = 32: 16 x 4096 x 4096 12.9 / 10.7 (12.4), 2048 x 4096 x 4096 22.7 / 21.9.  Same bits.
    switch (a.r) {
        case 16: return launch_ds_t<Ds<1, 512, 4, 8>>(a, tiles, st);
        case 32: return 2 * tiles <= kComputeUnits ? launch_ds_t<Ds<1, 512, 4, 8, 32>>(a, tiles, st) : launch_ds_t<Ds<2, 512, 3, 8>>(a, tiles, st);
        case 64:
            return 4 * tiles <= kComputeUnits   ? launch_ds_t<Ds<1, 512, 4, 8, 64>>(a, tiles, st)
                   : 2 * tiles <= kComputeUnits ? launch_ds_t<Ds<2, 512, 3, 8, 64>>(a, tiles, st)
                                                : launch_ds_t<Ds<4, 256, 3, 8>>(a, tiles, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace lf
