// Operation (4) of the fused LoRA linear layer (Section 5.1, FusedLoRA Design), one pass over X with the mask
// regenerated:
//     dA[c,j] = q sum_i keep(i,j) X[i,j] dS[i,c]          (dS arrives scaled by s*q)
// A workgroup owns a strip of 64 columns (one 128-byte line of every row) over a panel of rows; each of its eight waves
// walks the 32-row blocks w, w + 8, ... of the panel by itself: global -> registers two blocks ahead, mask, LDS of the
// wave's own, transposing reads, 16x16x32 bf16 MFMAs.  No barrier until the waves' sums are added, in a fixed order.
// A panel is a whole segment where that leaves the chip enough workgroups (the sum is then dA itself); otherwise the
// panels leave fp32 partial planes that finalize_da_kernel adds in a fixed order.  Repeated runs agree bit for bit.
#include "lf_device.h"
#include "lf_internal.h"

namespace lf {

constexpr int DA_WAVES = 8, DA_THREADS = 64 * DA_WAVES;
constexpr int DA_STRIP = 64;                       // columns per workgroup
constexpr int DA_BLOCK = 32;                       // rows per wave and block

#define LF_MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a), (b), (c), 0, 0, 0)

// X block of a wave: rows of 128 bytes, chunk index XOR-ed so that the 32 lanes of a transposing read ({a..a+3, a+8..a+11}
// x 32 bytes; two rows share 256 bytes) cover 256 distinct bytes.
__device__ __forceinline__ int da_x_off(int row, int chunk) {
    return row * 128 + ((chunk ^ ((row & 2) | ((row & 8) >> 1))) << 4);
}

template <int CB, class TB>                        // r / 16
__global__ void __launch_bounds__(DA_THREADS, CB == 4 ? 2 : 4) da_kernel(DaArgsOf<TB> p) {
    constexpr int R = CB * 16, RCH = CB * 2;       // rank, 16-byte chunks per dS row
    constexpr int WAVE_LDS = DA_BLOCK * (DA_STRIP + R) * 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int strips = p.K / DA_STRIP;
    const int tile = blockIdx.x / strips, c0 = (blockIdx.x - tile * strips) * DA_STRIP;
    RowTile rt;
    if (p.direct) {                                // panel = segment, empty ones too (their gradient is zero)
        rt.g = tile;
        rt.row_start = p.tb.row0[tile];
        rt.rows = p.tb.row0[tile + 1] - rt.row_start;
        rt.local_row0 = 0;
        if (rt.rows == 0 && p.accumulate) return;
    } else if (!find_panel(p.tb, p.panel_rows, tile, rt)) return;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = rt.g, cbn = p.tb.a[g].rank >> 4;
    const uint32_t T = p.tb.a[g].T, hk0 = p.tb.a[g].k0, hk1 = p.tb.a[g].k1;
    const KeepThreshold th = keep_threshold(T);
    char* lds_x = smem + w * WAVE_LDS;
    char* lds_s = lds_x + DA_BLOCK * DA_STRIP * 2;

    f32x4 acc[4][CB];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[jb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const lora_bf16* X = p.X + (int64_t)rt.row_start * p.K + c0 + (l & 7) * 8;
    const lora_bf16* dS = p.dS + (int64_t)rt.row_start * R;
    const int nblocks = (rt.rows + DA_BLOCK - 1) / DA_BLOCK;
    // lane l holds rows 8*i + (l >> 3), chunk l & 7 of a block; dS rows as they lie in memory, 1 KB per register
    struct Regs { u32x4 x[4], s[CB]; };
    auto load = [&](Regs& r, int blk) {            // (rows past the end read the last one: never used)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            r.x[i] = *(const u32x4*)(X + (int64_t)min(blk * DA_BLOCK + 8 * i + (l >> 3), rt.rows - 1) * p.K);
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int e = i * 64 + l;
            r.s[i] = *(const u32x4*)(dS + (int64_t)min(blk * DA_BLOCK + e / RCH, rt.rows - 1) * R + (e % RCH) * 8);
        }
    };
    auto consume = [&](const Regs& r, int blk) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * i + (l >> 3), prow = blk * DA_BLOCK + row;
            u32x4 v = r.x[i];
            if (T) v = mask8(v, row_key(hk0, hk1, (uint32_t)(rt.local_row0 + prow)), (uint32_t)(c0 + (l & 7) * 8), th);
            if (prow >= rt.rows) v = u32x4{0u, 0u, 0u, 0u};
            *(u32x4*)(lds_x + da_x_off(row, l & 7)) = v;
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const int e = i * 64 + l, row = e / RCH;
            const u32x4 v = blk * DA_BLOCK + row < rt.rows ? r.s[i] : u32x4{0u, 0u, 0u, 0u};
            *(u32x4*)(lds_s + tile_off(row, e % RCH, RCH)) = v;
        }
        // (LDS operations of one wave complete in order: no barrier between its writes and its reads)
        const int r0 = 8 * (l >> 4);
        bf16x8 fs[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            fs[cb] = join_tr(lds_read_tr(lds_s, tr_off(r0, cb * 16, l & 15, RCH)), lds_read_tr(lds_s, tr_off(r0 + 4, cb * 16, l & 15, RCH)));
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            const int row = r0 + ((l & 15) >> 2), col = jb * 16 + ((l & 3) << 2);
            const int o = da_x_off(row, col >> 3) + ((col & 7) << 1);
            const bf16x8 fb = join_tr(lds_read_tr(lds_x, o), lds_read_tr(lds_x, o + 4 * 128));   // (row + 4: same swizzle)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                if (CB == 1 || cb < cbn) acc[jb][cb] = LF_MFMA16(fb, fs[cb], acc[jb][cb]);       // D[j][c]
        }
    };
    if (w < nblocks) {
        Regs a, b;
        load(a, w);
        load(b, w + DA_WAVES);
        __builtin_amdgcn_sched_barrier(0);
        for (int blk = w;; blk += 2 * DA_WAVES) {
            consume(a, blk);
            load(a, blk + 2 * DA_WAVES);
            __builtin_amdgcn_sched_barrier(0);
            if (blk + DA_WAVES >= nblocks) break;
            consume(b, blk + DA_WAVES);
            load(b, blk + 3 * DA_WAVES);
            __builtin_amdgcn_sched_barrier(0);
            if (blk + 2 * DA_WAVES >= nblocks) break;
        }
    }

    // fixed-order sum over the waves, one 16-row block of dA at a time; plane layout [c][j]
    f32x4* red = (f32x4*)smem;                     // [DA_WAVES][4][64]
    float* out = p.direct ? p.dA + (int64_t)g * R * p.K : p.part + (int64_t)tile * R * p.K;
    for (int cb = 0; cb < CB; ++cb) {
        __syncthreads();
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            f32x4 v = acc[jb][0];
#pragma unroll
            for (int k = 1; k < CB; ++k)
                if (cb == k) v = acc[jb][k];
            red[(w * 4 + jb) * 64 + l] = v;
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            const int jb = threadIdx.x >> 6;
            f32x4 v = red[threadIdx.x];
#pragma unroll
            for (int ww = 1; ww < DA_WAVES; ++ww) v += red[ww * 256 + threadIdx.x];
            f32x4* o = (f32x4*)(out + (int64_t)(cb * 16 + (l & 15)) * p.K + c0 + jb * 16 + 4 * (l >> 4));
            *o = p.direct && p.accumulate ? *o + v : v;
        }
    }
}

template <int CB>
static hipError_t launch_da_t(const DaArgs& a, hipStream_t st) {
    const int lds = DA_WAVES * DA_BLOCK * (DA_STRIP + CB * 16) * 2;
    const int panels = a.direct ? a.tb.G : count_panels(a.tb, a.panel_rows);
    if (panels == 0) return hipSuccess;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = da_kernel<CB, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;              // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)((int64_t)panels * (a.K / DA_STRIP))), dim3(DA_THREADS), lds, st, b);
        return hipGetLastError();
    });
}

hipError_t launch_da(const DaArgs& a, hipStream_t st) {
    if (!a.direct && a.panel_rows < DA_BLOCK) return hipErrorInvalidValue;
    switch (a.r) {
        case 16: return launch_da_t<1>(a, st);
        case 32: return launch_da_t<2>(a, st);
        case 64: return launch_da_t<4>(a, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace lf
