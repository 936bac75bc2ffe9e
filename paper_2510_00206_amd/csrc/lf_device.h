// Device-side helpers shared by the gfx950 kernels: vector types, the dropout hash, LDS swizzles,
// and the per-adapter table that routes row tiles to adapters (Section 5.1, FusedMultiLoRA:
// every M-tile carries an adapter id that indexes a small lookup table).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lf {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kMaxAdapters = 64;

// Lookup table passed by value in the kernel arguments.  Every workgroup walks the segments to find its tile and then reads
// the fields of one adapter: the row offsets lie side by side (16 of them to a cache line of the arguments), the fields of an
// adapter in one or two lines.  These reads are a latency at the start of every launch.  Against one array per field, two
// backward passes of four launches each over 2048 x 4096 x 4096: 46.0 -> 44.8 us; against offsets that lie in the adapters'
// entries, 28 bytes apart, (1) over 64 adapters x 4 rows, K = 1024: 16.5 -> 11.9 us, (2) 4096 -> 1024 over 64 x 100 rows:
// 66 -> 60 us.
struct Adapter {
    // rank of the adapter (16, 32 or 64), at most the call's r: the arrays are laid out with r columns
    // (rows of A) per adapter and the adapter uses the first `rank`; the padding of A and B is never used
    // and the padding of S', dS, dA and dB is written as zeros
    int rank;                         // (32 bits: a kernel reads it with a scalar load, a byte would take a vector load and its wait)
    uint32_t T;                       // dropout threshold: keep iff bits16 >= T
    uint32_t k0, k1;                  // seed-derived hash keys
    float s;                          // the paper's alpha
    float q;                          // survivor scale 65536/(65536-T)
};

template <int MAX>
struct AdapterTableOf {
    int G;
    int row0[MAX + 1];                // segment g owns rows [row0[g], row0[g + 1])
    Adapter a[MAX];
};
using AdapterTable = AdapterTableOf<kMaxAdapters>;

// What a launch of few adapters takes of it.  The table is nearly all of a kernel's arguments (1.8 KB of 1.9), which are
// copied several times on the way to the device and written there over the bus; the kernels that small launches use are
// instantiated for both sizes (a step of six launches over 256 x 1024 x 1024 33.9 -> 30.7 us, 1000 rows and more level).
constexpr int kFewAdapters = 4;
using FewAdapters = AdapterTableOf<kFewAdapters>;

// First statement of a kernel whose arguments are of type Args: asks for every cache line of them at once.  A launch finds them in
// memory, not in a cache, and the compiler loads a field where it is first needed: the number of adapters, behind that the walk over
// the segments, behind that the adapter's entry, 0.35 us each.  us, without / with: two accumulating backward passes over 2048 x 4096 x 4096 37.2 / 36.6, a step of
// 1531 packed rows 63.2 / 62.6; backward without dX, of launches of many workgroups too, 256 x 1024 x 1024 7.89 / 7.84, ten adapters of 300 rows, 256 -> 512
// 8.21 / 8.12, 8192 rows, 4096 -> 4096 38.0 / 37.6, -> 14336 75.2 / 74.5, 5003 rows, 14336 -> 4096 49.7 / 49.0; level for (1) straight into registers (16384 rows, K =
// 256 7.8).  Not in the GEMMs of small tiles, whose entry code needs most of the lines at once and waits for the last (471 workgroups, a step of
// 66.5 -> 67.9 us); those of few workgroups have not been told apart.
template <class Args>
__device__ __forceinline__ void fetch_args() {
    constexpr int LINES = ((int)sizeof(Args) + 63) / 64, N = LINES < 8 ? LINES : 3;     // (of a full table its first offsets)
    const auto* w = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = w[i < N ? i * 16 : 0];
    const uint32_t end = w[N == LINES ? sizeof(Args) / 4 - 1 : 0];
    asm volatile("" :: "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]), "s"(end));
}

// A row tile: `rows` valid rows starting at global row `row_start`, owned by adapter g.
struct RowTile {
    int g, row_start, rows, local_row0;   // local_row0 = row_start - row0[g] (mask row index base)
};

// Tiles never straddle a segment: segment g contributes ceil(len/gran) tiles, len counting its rows in
// [row_lo, row_hi).
template <class TB>
__device__ __forceinline__ bool find_row_tile(const TB& tb, int gran, int tile, RowTile& rt, int row_lo = 0,
                                              int row_hi = 0x7FFFFFFF) {
    int t = tile;
    for (int g = 0; g < tb.G; ++g) {
        const int lo = max(tb.row0[g], row_lo), hi = min(tb.row0[g + 1], row_hi);
        const int nt = max(hi - lo + gran - 1, 0) / gran;
        if (t < nt) {
            rt.g = g;
            rt.row_start = lo + t * gran;
            rt.rows = min(gran, hi - rt.row_start);
            rt.local_row0 = rt.row_start - tb.row0[g];
            return true;
        }
        t -= nt;
    }
    return false;
}

// The same, for a whole wave and from the full table: a lane for every adapter, a sum over the lanes.  Every wave of a workgroup walks the
// table for itself, and the loop above is some ten scalar instructions an adapter on the one scalar unit of the compute
// unit: with waves that only copy beside those that compute it cost 64 adapters more than their copying saves.
template <class TB>
__device__ __forceinline__ bool find_row_tile_by_lanes(const TB& tb, int gran, int tile, RowTile& rt, int row_lo = 0,
                                                       int row_hi = 0x7FFFFFFF) {
    if constexpr (sizeof(tb.a) / sizeof(tb.a[0]) <= kFewAdapters) {
        return find_row_tile(tb, gran, tile, rt, row_lo, row_hi);
    } else {
        static_assert(sizeof(tb.a) / sizeof(tb.a[0]) <= 64, "a lane for every adapter");
        const int l = threadIdx.x & 63, g0 = min(l, tb.G - 1);
        const int first = tb.row0[g0], lo = max(first, row_lo), hi = min(tb.row0[g0 + 1], row_hi);
        const int nt = l < tb.G ? max(hi - lo + gran - 1, 0) / gran : 0;
        int sum = nt;                                        // of lanes 0 .. l: within rows of 16 lanes, then row 0 into 1 and 2 into 3, 1 into 2 and 3
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x111, 0xF, 0xF, false);
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x112, 0xF, 0xF, false);
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x114, 0xF, 0xF, false);
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x118, 0xF, 0xF, false);
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x142, 0xA, 0xF, false);
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x143, 0xC, 0xF, false);
        const uint64_t past = __ballot(sum > tile);
        if (past == 0) return false;
        const int g = __builtin_ctzll(past);
        auto of_g = [&](int v) { return __builtin_amdgcn_readlane(v, g); };
        const int in_g = (tile - of_g(sum - nt)) * gran;
        rt.g = g;
        rt.row_start = of_g(lo) + in_g;
        rt.rows = min(gran, of_g(hi) - rt.row_start);
        rt.local_row0 = rt.row_start - of_g(first);
        return true;
    }
}

// Row panels of the streaming reductions (operations (3) and (4)).  A segment of length len holds
// nf = len / gran full panels; a remainder is merged into the segment's last panel (a "long" panel of
// fewer than 2*gran rows) or, when the segment is shorter than gran, forms one "short" panel.  Cutting
// the remainder off as a panel of its own would add a workgroup per column chunk for a few rows and,
// with the panel count just past a multiple of the CU count, a whole extra round of workgroups.
// Panels are numbered long ones first (they run longest, so they start first), then the regular
// ones, then the short ones; the number is also the plane index of the panel's partial sums.
struct SegmentPanels { int nreg; bool has_long, has_short; int rem; };

template <class TB>
__host__ __device__ __forceinline__ SegmentPanels segment_panels(const TB& tb, int gran, int g) {
    const int len = tb.row0[g + 1] - tb.row0[g];
    const int nf = len >> __builtin_ctz((unsigned)gran);      // (every panel height is a power of two)
    SegmentPanels sp;
    sp.rem = len - nf * gran;
    sp.has_short = nf == 0 && sp.rem > 0;
    sp.has_long = nf > 0 && sp.rem > 0;
    sp.nreg = nf - (sp.has_long ? 1 : 0);
    return sp;
}

template <class TB>
__host__ __device__ __forceinline__ int count_panels(const TB& tb, int gran) {
    int n = 0;
    for (int g = 0; g < tb.G; ++g) {
        const SegmentPanels sp = segment_panels(tb, gran, g);
        n += sp.nreg + (sp.has_long ? 1 : 0) + (sp.has_short ? 1 : 0);
    }
    return n;
}

template <class TB>
__device__ __forceinline__ bool find_panel(const TB& tb, int gran, int panel, RowTile& rt) {
    int idx = panel;
    for (int g = 0; g < tb.G; ++g) {                     // long panels
        const SegmentPanels sp = segment_panels(tb, gran, g);
        if (!sp.has_long) continue;
        if (idx == 0) {
            rt.g = g;
            rt.local_row0 = sp.nreg * gran;
            rt.row_start = tb.row0[g] + rt.local_row0;
            rt.rows = gran + sp.rem;
            return true;
        }
        --idx;
    }
    for (int g = 0; g < tb.G; ++g) {                     // regular panels
        const SegmentPanels sp = segment_panels(tb, gran, g);
        if (idx < sp.nreg) {
            rt.g = g;
            rt.local_row0 = idx * gran;
            rt.row_start = tb.row0[g] + rt.local_row0;
            rt.rows = gran;
            return true;
        }
        idx -= sp.nreg;
    }
    for (int g = 0; g < tb.G; ++g) {                     // short panels
        const SegmentPanels sp = segment_panels(tb, gran, g);
        if (!sp.has_short) continue;
        if (idx == 0) {
            rt.g = g;
            rt.local_row0 = 0;
            rt.row_start = tb.row0[g];
            rt.rows = sp.rem;
            return true;
        }
        --idx;
    }
    return false;
}

// Plane indices of segment g's panels: regular planes [reg0, reg0 + nreg), then `extra` (its long or
// short panel, -1 if none).  The finalize kernels add them in exactly this order.
template <class TB>
__device__ __forceinline__ void segment_planes(const TB& tb, int gran, int g, int& reg0, int& nreg, int& extra) {
    int n_long = 0, n_reg = 0, long_before = 0, reg_before = 0, short_before = 0;
    for (int gg = 0; gg < tb.G; ++gg) {
        const SegmentPanels sp = segment_panels(tb, gran, gg);
        if (gg < g) { long_before += sp.has_long; reg_before += sp.nreg; short_before += sp.has_short; }
        n_long += sp.has_long; n_reg += sp.nreg;
    }
    const SegmentPanels me = segment_panels(tb, gran, g);
    reg0 = n_long + reg_before;
    nreg = me.nreg;
    extra = me.has_long ? long_before : me.has_short ? n_long + n_reg + short_before : -1;
}

template <class TB>
__device__ __forceinline__ int segment_of_row(const TB& tb, int row, int g = 0) {
    while (g + 1 < tb.G && row >= tb.row0[g + 1]) ++g;
    return g;
}

// Packed tiling for the GEMMs: when every segment boundary is a multiple of 64 rows, the packed
// batch is cut into uniform tiles of 256 (or 192) rows and a tile may hold up to four (three) adapters, one per 64-row
// group; only such mixed tiles take the slower per-group LoRA path.  `g`: one byte per group.
struct GroupMap {
    uint32_t g;
    bool mixed;
    __device__ __forceinline__ int adapter(int q) const { return (int)(g >> (8 * q) & 0xFFu); }
};
static_assert(kMaxAdapters <= 256, "a group's adapter is one byte");

__device__ __forceinline__ GroupMap one_group(int g) { return GroupMap{(uint32_t)g * 0x01010101u, false}; }

__device__ __forceinline__ void find_uniform_tile(const AdapterTable& tb, int M, int gran, int tile, RowTile& rt,
                                                  GroupMap& gm) {
    rt.row_start = tile * gran;
    rt.rows = min(gran, M - rt.row_start);
    gm.g = 0;
    int g = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = rt.row_start + 64 * q;
        if (q == 0 || (64 * q < gran && row < M))
            g = segment_of_row(tb, row, g);
        if (q == 0) rt.g = g;
        gm.g |= (uint32_t)g << (8 * q);
    }
    gm.mixed = gm.g != (uint32_t)rt.g * 0x01010101u;
    rt.local_row0 = rt.row_start - tb.row0[rt.g];
}

// ---- dropout hash (unsigned 32-bit arithmetic) ------------------------------------------------
constexpr uint32_t kGold = 0x9E3779B9u, kM1 = 0x6A09E667u, kM2 = 0xBB67AE85u, kC5 = 0x3C6EF373u,
                   kC7 = 0xA54FF53Bu;

__host__ __device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16; x *= kM1; x ^= x >> 15; x *= kM2; x ^= x >> 16;
    return x;
}

struct RowKey { uint32_t a, b; };

__device__ __forceinline__ RowKey row_key(uint32_t k0, uint32_t k1, uint32_t local_row) {
    RowKey rk;
    rk.a = mix32(k1 ^ (local_row * kGold));
    rk.b = mix32(rk.a + k0 + kC7);
    return rk;
}

// One word decides columns 2*cp (low half) and 2*cp+1 (high half).
__device__ __forceinline__ uint32_t hash_word(RowKey rk, uint32_t cp) {
    uint32_t x = rk.a + cp * kGold;
    x ^= x >> 16; x *= kM1; x += rk.b; x ^= x >> 15; x *= kM2; x ^= x >> 16;
    return x;
}

// Same word from x = rk.a + cp * kGold already formed (consecutive pairs differ by kGold).
__device__ __forceinline__ uint32_t hash_word_at(RowKey rk, uint32_t x) {
    x ^= x >> 16; x *= kM1; x += rk.b; x ^= x >> 15; x *= kM2; x ^= x >> 16;
    return x;
}

// AND-mask for a packed pair of bf16 (even column in the low half): 0xFFFF in a half iff its
// 16 hash bits are >= T.  Packed 16-bit arithmetic: saturating (bits - (T-1)) is non-zero iff
// bits >= T (for T >= 1); min(.,1) * 0xFFFF spreads it over the half.  T == 0 keeps everything.
struct KeepThreshold { uint32_t tm1_packed; uint32_t keep_all; };

__host__ __device__ __forceinline__ KeepThreshold keep_threshold(uint32_t T) {
    KeepThreshold k;
    const uint32_t tm1 = T ? T - 1 : 0xFFFFu;          // T == 0: nothing passes the test, keep_all covers it
    k.tm1_packed = tm1 | (tm1 << 16);
    k.keep_all = T ? 0u : 0xFFFFFFFFu;
    return k;
}

__device__ __forceinline__ uint32_t keep_pair_mask(uint32_t w, KeepThreshold kt) {
    // Three packed 16-bit instructions, written as such: from the generic form the compiler makes two
    // compares, two selects and a byte permute per word.
    uint32_t d, m;
    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(d) : "v"(w), "v"(kt.tm1_packed));
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(m) : "v"(d), "v"(0x00010001u));
    asm("v_pk_mul_lo_u16 %0, %1, %2" : "=v"(d) : "v"(m), "v"(0xFFFFFFFFu));
    return d | kt.keep_all;
}

// Mask 8 consecutive bf16 (columns col..col+7, col % 8 == 0) held in a 16-byte vector.
__device__ __forceinline__ u32x4 mask8(u32x4 v, RowKey rk, uint32_t col, KeepThreshold kt) {
    const uint32_t x = rk.a + (col >> 1) * kGold;      // consecutive column pairs differ by kGold
    v.x &= keep_pair_mask(hash_word_at(rk, x), kt);
    v.y &= keep_pair_mask(hash_word_at(rk, x + kGold), kt);
    v.z &= keep_pair_mask(hash_word_at(rk, x + 2u * kGold), kt);
    v.w &= keep_pair_mask(hash_word_at(rk, x + 3u * kGold), kt);
    return v;
}

// ---- bf16 helpers -----------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    bf16x2 v;
    v.x = (__bf16)lo;
    v.y = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// ---- LDS layouts --------------------------------------------------------------------------------
// Tiles are stored as rows of 16-byte chunks whose index is XOR-ed with a function of the row.
// Measured on gfx950: the LDS has 64 banks of 4 bytes (256 bytes per cycle); a 16-byte-per-lane read
// is served 16 consecutive lanes per cycle and an 8-byte-per-lane (transposing) read 32 consecutive
// lanes per cycle, so an access is conflict-free when each such lane group covers 256 bytes that are
// distinct modulo 256.

// Generic small tiles (rank-wide operands: S', dS, B chunk), nchunk a power of two.
__device__ __forceinline__ int swz(int row) { return ((row & 3) << 1) | ((row >> 2) & 1); }
__device__ __forceinline__ int tile_off(int row, int chunk, int nchunk) {
    return (row * nchunk + (chunk ^ (swz(row) & (nchunk - 1)))) * 16;
}

// GEMM row-operand slab: rows of 128 bytes (8 chunks), read 16 consecutive rows at one chunk index.
// Two rows share a 256-byte line, so rows of equal parity must differ in the chunk position.
__device__ __forceinline__ int row_slab_swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int row_slab_off(int row, int chunk) {
    return row * 128 + ((chunk ^ row_slab_swz(row)) << 4);
}

// GEMM column-operand slab: rows of 512 bytes (32 chunks), read with transposing loads for the 16x16x32 MFMA: the
// 32 lanes served in one cycle address rows {a..a+3, a+8..a+11} x 32 bytes, which must fall into eight different
// 32-byte windows: row bits (0, 1, 3) go to chunk bits (1, 2, 3).
__device__ __forceinline__ int col_slab_swz(int row) { return ((row & 3) << 1) | (row & 8); }
__device__ __forceinline__ int col_slab_off(int row, int chunk) {
    return row * 512 + ((chunk ^ col_slab_swz(row)) << 4);
}

// Streaming panel tile: rows of 1024 bytes (64 chunks), read both ways: 16 consecutive rows at one
// chunk index (needs 16 distinct chunk positions) and transposing loads over rows {a..a+3, a+8..a+11}
// x 32 bytes (needs 8 distinct 32-byte windows): row bits (r0, r1, r3) go to chunk bits (1, 2, 3), r2 to bit 0.
__device__ __forceinline__ int panel_swz(int row) {
    return ((row & 1) << 1) | ((row & 2) << 1) | (row & 8) | ((row >> 2) & 1);
}
__device__ __forceinline__ int panel_off(int row, int chunk) {
    return row * 1024 + ((chunk ^ panel_swz(row)) << 4);
}

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Transposing LDS read: the 16 lanes of a group address a 4-row x 16-column block of 16-bit
// elements (lane i: row i/4, columns 4*(i%4)..+3); lane i receives column i of the four rows.
__device__ __forceinline__ s16x4 lds_read_tr(const char* lds_base, int byte_off) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4*)(__attribute__((address_space(3))) char*)(lds_base + byte_off));
}

// Byte offset for the transposing read of rows r0..r0+3 (r0 % 4 == 0), columns c0..c0+15
// (c0 % 16 == 0), for lane-in-group i16, in a generic small tile with nchunk chunks per row ...
__device__ __forceinline__ int tr_off(int r0, int c0, int i16, int nchunk) {
    const int row = r0 + (i16 >> 2);
    const int col = c0 + ((i16 & 3) << 2);           // element column, multiple of 4
    return tile_off(row, col >> 3, nchunk) + ((col & 7) << 1);
}
// ... in a GEMM column-operand slab ...
__device__ __forceinline__ int col_slab_tr_off(int r0, int c0, int i16) {
    const int row = r0 + (i16 >> 2);
    const int col = c0 + ((i16 & 3) << 2);
    return col_slab_off(row, col >> 3) + ((col & 7) << 1);
}
// ... and in a streaming panel tile.
__device__ __forceinline__ int panel_tr_off(int r0, int c0, int i16) {
    const int row = r0 + (i16 >> 2);
    const int col = c0 + ((i16 & 3) << 2);
    return panel_off(row, col >> 3) + ((col & 7) << 1);
}

__device__ __forceinline__ bf16x8 join_tr(s16x4 lo, s16x4 hi) {
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

}  // namespace lf
