// One workgroup of the strip sums (see lf_da.hip), for the launches that have such workgroups.
#pragma once
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

// Partial sums of a strip meet in the last of its workgroups: every workgroup leaves an fp32 piece of R x 64, counts itself in,
// and the one that finds all others there adds the pieces in the order of the panels (segment_planes).  The pieces are
// written and read past the XCDs' own L2s (sc1, as agent-scope atomic stores and loads are, sixteen bytes at a time); a store has
// arrived when the wave's vmcnt counts it, so that no cache has to be written back or invalidated around the counter (a
// release and an acquire fence instead, which do that, cost 2048 x 4096, r = 16, 256 workgroups 40 us).
constexpr int kPastL2 = 16;                        // cache policy bits of a buffer access: sc1
typedef __attribute__((__vector_size__(16))) uint32_t buffer_u32x4;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t piece_of(float* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x27000);
}
__device__ __forceinline__ void store_piece(__amdgpu_buffer_rsrc_t piece, int i, f32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(buffer_u32x4, v), piece, i * 16, 0, kPastL2);
}
__device__ __forceinline__ f32x4 load_piece(__amdgpu_buffer_rsrc_t piece, int i) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(piece, i * 16, 0, kPastL2));
}
__device__ __forceinline__ bool last_of_strip(uint32_t* counter, uint32_t panels, uint32_t* flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's piece has arrived ...
    __syncthreads();                                      // ... and every wave's
    if (threadIdx.x == 0) *flag = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == panels;
    __syncthreads();
    return *flag != 0;
}

// One workgroup of a strip job.  MASKED: dA [r, C] of operation (4); otherwise dB [C, r] of operation (3).
template <int CB, bool MASKED, class Args>
__device__ __forceinline__ void strip_body(const Args& p, const StripJob& job, int block, char* smem) {
    constexpr int R = CB * 16, RCH = CB * 2;       // rank, 16-byte chunks per dS (S') row
    constexpr int WAVE_LDS = DA_BLOCK * (DA_STRIP + R) * 2;
    const int strips = job.C / DA_STRIP;
    const int tile = block / strips, strip = block - tile * strips, c0 = strip * DA_STRIP;
    RowTile rt;
    if (job.panel_rows == 0) {                     // panel = segment, empty ones too (their gradient is zero)
        rt.g = tile;
        rt.row_start = p.tb.row0[tile];
        rt.rows = p.tb.row0[tile + 1] - rt.row_start;
        rt.local_row0 = 0;
    } else if (tile < job.panels) {
        find_panel(p.tb, job.panel_rows, tile, rt);
    } else {                                       // no panel cuts an empty segment: one workgroup each writes its zeros
        int n = tile - job.panels;
        rt.g = 0;
        while (p.tb.row0[rt.g] != p.tb.row0[rt.g + 1] || n-- > 0) ++rt.g;
        rt.row_start = p.tb.row0[rt.g];
        rt.rows = rt.local_row0 = 0;
    }
    if (rt.rows == 0 && p.accumulate) return;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = rt.g, cbn = p.tb.a[g].rank >> 4;
    const uint32_t T = MASKED ? p.tb.a[g].T : 0u, hk0 = p.tb.a[g].k0, hk1 = p.tb.a[g].k1;
    const KeepThreshold th = keep_threshold(T);
    char* lds_x = smem + w * WAVE_LDS;
    char* lds_s = lds_x + DA_BLOCK * DA_STRIP * 2;

    f32x4 acc[4][CB];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[jb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const lora_bf16* X = job.big + (int64_t)rt.row_start * job.C + c0 + (l & 7) * 8;
    const lora_bf16* dS = job.small_ + (int64_t)rt.row_start * R;
    const int nblocks = (rt.rows + DA_BLOCK - 1) / DA_BLOCK;
    // lane l holds rows 8*i + (l >> 3), chunk l & 7 of a block; dS rows as they lie in memory, 1 KB per register
    struct Regs { u32x4 x[4], s[CB]; };
    auto load = [&](Regs& r, int blk) {            // (rows past the end read the last one: never used)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            r.x[i] = *(const u32x4*)(X + (int64_t)min(blk * DA_BLOCK + 8 * i + (l >> 3), rt.rows - 1) * job.C);
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
            if (MASKED && T) v = mask8(v, row_key(hk0, hk1, (uint32_t)(rt.local_row0 + prow)), (uint32_t)(c0 + (l & 7) * 8), th);
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
        // (all of the call's rank: the padding past the adapter's is zeroed on the way out; a test per MFMA would wait for every
        // fragment by itself)
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
            for (int cb = 0; cb < CB; ++cb)        // D[j][c], resp. D[c][n]: four consecutive elements of the output to a lane
                acc[jb][cb] = MASKED ? LF_MFMA16(fb, fs[cb], acc[jb][cb]) : LF_MFMA16(fs[cb], fb, acc[jb][cb]);
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

    // Where the sum goes: the gradient itself if this workgroup has the whole segment, else a piece for the last workgroup of
    // the strip (counters), or a plane for finalize_da_kernel.
    int panels = 1;
    if (job.panel_rows) {
        const SegmentPanels sp = segment_panels(p.tb, job.panel_rows, g);
        panels = sp.nreg + sp.has_long + sp.has_short;
    }
    const bool whole = job.panel_rows == 0 || (job.counters && panels <= 1);
    constexpr int PIECE = R * DA_STRIP;
    auto piece = [&](int t) { return piece_of(job.part + ((int64_t)t * strips + strip) * PIECE, PIECE * 4); };
    float* grad = job.out + (int64_t)g * R * job.C;
    auto grad_at = [&](int cb, int jb) {
        return (f32x4*)(MASKED ? grad + (int64_t)(cb * 16 + (l & 15)) * job.C + c0 + jb * 16 + 4 * (l >> 4)
                               : grad + (int64_t)(c0 + jb * 16 + (l & 15)) * R + cb * 16 + 4 * (l >> 4));
    };

    // fixed-order sum over the waves, one 16-column block of the rank at a time
    f32x4* red = (f32x4*)smem;                     // [DA_WAVES][4][64]
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
            f32x4 v[DA_WAVES];
#pragma unroll
            for (int ww = 0; ww < DA_WAVES; ++ww) v[ww] = red[ww * 256 + threadIdx.x];
#pragma unroll
            for (int d = 1; d < DA_WAVES; d *= 2)  // pairwise: the smaller rounding error
#pragma unroll
                for (int ww = 0; ww < DA_WAVES; ww += 2 * d) v[ww] += v[ww + d];
            // zero times a non-finite element is not zero.  (Here and not on every wave's sum before it is written, where each block of
            // the rank waited for it: backward without dX of 213 rows in 53 segments, 11840 -> 4480, r = 64 352 -> 338 us.)
            if (cb >= cbn) v[0] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (whole) {
                f32x4* o = grad_at(cb, threadIdx.x >> 6);
                *o = p.accumulate ? *o + v[0] : v[0];
            } else if (job.counters) {
                store_piece(piece(tile), cb * 256 + threadIdx.x, v[0]);
            } else {
                *(f32x4*)(job.part + (int64_t)tile * R * job.C + (grad_at(cb, threadIdx.x >> 6) - (f32x4*)grad) * 4) = v[0];
            }
        }
    }
    if (whole || !job.counters) return;
    __syncthreads();                               // (the flag lies where the waves' sums were)
    if (!last_of_strip(job.counters + g * strips + strip, panels, (uint32_t*)smem)) return;
    int reg0, nreg, extra;
    segment_planes(p.tb, job.panel_rows, g, reg0, nreg, extra);
    for (int i = threadIdx.x; i < CB * 256; i += DA_THREADS) {
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int t = reg0; t < reg0 + nreg; ++t) v += load_piece(piece(t), i);
        if (extra >= 0) v += load_piece(piece(extra), i);
        f32x4* o = grad_at(i >> 8, (i >> 6) & 3);
        *o = p.accumulate ? *o + v : v;
    }
}

// Workgroup `block` of both jobs.
template <int CB, class Args>
__device__ __forceinline__ void strip_of(const Args& p, int block, char* smem) {
    const int first = p.b_first ? p.b.blocks : p.a.blocks;
    if ((block < first) != (p.b_first != 0)) strip_body<CB, true>(p, p.a, p.b_first ? block - first : block, smem);
    else strip_body<CB, false>(p, p.b, p.b_first ? block : block - first, smem);
}

constexpr int strip_lds(int cb) { return DA_WAVES * DA_BLOCK * (DA_STRIP + cb * 16) * 2; }

}  // namespace lf
