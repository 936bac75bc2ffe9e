// Device-side pieces that the GEMM kernels of operations (2) and (5) share (lf_gemm.hip: the large tiles;
// lf_gemm_ring.hip: the small ones): workgroup -> tile map, global -> LDS slab copies, waits.
#pragma once
#include "lf_device.h"

namespace lf {

constexpr int BK = 64;                      // contraction depth of a slab

// Workgroup id -> output tile.  Consecutive workgroup ids go round-robin over the 8 XCDs, each
// with a private L2, so ids are first regrouped per XCD (XCD x gets a run of total/8 tiles, the first total%8 XCDs
// one more) and then walked in bands of 8 row tiles so that the tiles resident on one XCD share operand slabs.
__device__ __forceinline__ void tile_of_block(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int total = tiles_m * tiles_n;
    const int xcd = bid & 7;
    const int lid = xcd * (total >> 3) + min(xcd, total & 7) + (bid >> 3);
    constexpr int GROUP = 8;
    const int per_group = GROUP * tiles_n;
    const int group = lid / per_group;
    const int first_m = group * GROUP;
    const int gsz = min(tiles_m - first_m, GROUP);
    const int in_group = lid - group * per_group;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
}

// ---- slab movement ------------------------------------------------------------------------------
// Slabs go from global memory straight into LDS (16 bytes per lane, no register staging): one wave
// instruction fills 1024 contiguous LDS bytes, lane l writing bytes [16 l, 16 l + 16), so the
// swizzle is applied by choosing which global chunk each lane fetches.  The load is issued from
// inline assembly: the LDS destination (M0) and the completion wait are managed by hand, so that
// the copy of the next slab stays in flight while the current one is consumed.
__device__ __forceinline__ uint32_t lds_addr_of(const char* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// The LDS destination of a copy is M0 + the instruction's immediate offset + 16 * lane, and the same
// immediate also moves the memory address.  A wave's passes of one slab are therefore laid out 1024 bytes
// apart (pass i of an NP-pass slab at immediate (i - NP/2) * 1024, M0 pointing at the middle), so that M0 is
// written once per slab instead of once per copy - a copy is then a single instruction, which matters between
// MFMAs of 16 cycles; the lane offsets are pre-biased by the opposite amount.  kCopyBias keeps those offsets
// non-negative: every source address handed to a copy is the slab's first element MINUS kCopyBias bytes (an
// address that is never dereferenced by itself).
constexpr int kCopyBias = 4096;
constexpr int pass_imm(int np, int i) { return (i - np / 2) * 1024; }

// M0 is named as clobbered so that the compiler never keeps a value of its own in it across a copy (it
// defines M0 itself before indirect register indexing, lane selects and its own LDS-DMA builtins; none of
// these occur in the kernels below, whose later passes rely on the M0 of pass 0).  Clang warns about every
// reserved register on a clobber list; the clobber is still recorded, hence the pragma.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int IMM, bool SET_M0>
__device__ __forceinline__ void copy16_to_lds(const char* biased_base, uint32_t lane_byte_off, uint32_t m0_value) {
    if constexpr (SET_M0)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                     :: "s"(m0_value), "v"(lane_byte_off), "s"(biased_base), "n"(IMM) : "memory", "m0");
    else
        asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2"
                     :: "v"(lane_byte_off), "s"(biased_base), "n"(IMM) : "memory");
}
#pragma clang diagnostic pop

__device__ __forceinline__ void wait_slab_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// all copies but the N issued last have landed (loads of a wave complete in order; only valid while no stores
// of the wave are outstanding)
template <int N> __device__ __forceinline__ void wait_slab_loads_but() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// ---- the MFMA ------------------------------------------------------------------------------------
#define LF_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a), (b), (c), 0, 0, 0)

// Lanes whose contraction elements lie at or past `valid_chunks` 16-byte chunks (8 elements each) of a rank-wide
// slab get a zero fragment: the slab's LDS rows hold duplicates there (the copies clamp), and a 32-deep MFMA
// sub-step reaches past a rank of 16 (or 48).
__device__ __forceinline__ bf16x8 zero_past_rank(bf16x8 v, int chunk, int valid_chunks) {
    u32x4 u = __builtin_bit_cast(u32x4, v);
    if (chunk >= valid_chunks) u = u32x4{0u, 0u, 0u, 0u};
    return __builtin_bit_cast(bf16x8, u);
}

}  // namespace lf
