// Internal C++ interface between the C ABI (lf_api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <type_traits>
#include <string.h>

#include "lf_device.h"

typedef uint16_t lora_bf16;

namespace lf {

// Operation (1): S' = s*q*(mask.X) A^T.
template <class TB>
struct DownArgsOf {
    const lora_bf16* X; const lora_bf16* A; lora_bf16* S;
    int M, K, r;
    TB tb;
};
using DownArgs = DownArgsOf<AdapterTable>;

// Operation (2).
struct FwdGemmArgs {
    const lora_bf16* X; const lora_bf16* W; const lora_bf16* S; const lora_bf16* B; lora_bf16* Y;
    int M, K, N, r, tiles_m, tiles_n;
    int uniform_tiles;         // set by the launcher: uniform tiles over the packed batch (boundaries % 64 == 0)
    AdapterTable tb;
};

// Operation (3) (lf_stream.hip).
template <class TB>
struct StreamArgsOf {
    const lora_bf16* big;      // dY [M,N]
    const lora_bf16* small_;   // S' [M,r]
    const lora_bf16* Bmat;     // B [G,N,r]
    float* part_out;           // per-row-panel partials of dB ([panels,N,r])
    float* part_ds;            // per-column-chunk partials of dS [chunks,M,r]
    int M, C, r;               // C = N
    int tiles_m, chunks;
    int panel_rows;            // rows per panel (stream_panel_rows), chosen once per entry-point call
    TB tb;
};
using StreamArgs = StreamArgsOf<AdapterTable>;

// dS by itself (lf_ds.hip); the launch also clears `n_zero` words for the counters of the strips that follow.
template <class TB>
struct DsArgsOf {
    const lora_bf16* dY; const lora_bf16* Bmat; lora_bf16* dS;
    uint32_t* zero;
    int n_zero;
    int M, C, r;               // C = N
    TB tb;
};
using DsArgs = DsArgsOf<AdapterTable>;

// Operation (4), and dB by itself (lf_da.hip): sums over the rows of a [M, C] activation in strips of 64 columns.
struct StripJob {
    const lora_bf16* big;      // X for dA, dY for dB
    const lora_bf16* small_;   // dS, resp. S'
    float* out;                // dA [G, r, C], resp. dB [G, C, r]; NULL: no such job
    float* part;               // fp32 partial sums of the panels (not whole segments)
    uint32_t* counters;        // [G, C / 64], zero, for the sum over the panels; NULL: `part` holds planes [panels] for finalize_da
    int C;
    int panel_rows;            // 0: one panel per segment
    int panels, blocks;        // set by the launcher
};
template <class TB>
struct StripArgsOf {
    StripJob a, b;             // dA, dB
    int b_first;               // set by the launcher: the job whose workgroups run longest starts first
    int r, accumulate;
    TB tb;
};
using StripArgs = StripArgsOf<AdapterTable>;

// Reductions of the partials.
template <class TB>
struct FinalizeArgsOf {
    const float* part_ds; lora_bf16* dS;        // dS[i,c] = s_g * sum over chunks
    const float* part_db; float* dB;            // dB[g,n,c] (+)= sum over the row tiles of segment g
    const float* part_da; float* dA;            // dA[g,c,j] (+)= q_g * sum over the row tiles of segment g
    int M, K, N, r, chunks, accumulate;
    int panel_rows_db, panel_rows_da;           // the panel heights operations (3) / (4) ran with (same call, same values)
    uint32_t* zero; int n_zero;                 // words that finalize_ds_db clears for the strips that follow
    TB tb;
};
using FinalizeArgs = FinalizeArgsOf<AdapterTable>;

// Operation (5).
struct DxGemmArgs {
    const lora_bf16* dY; const lora_bf16* W; const lora_bf16* dS; const lora_bf16* A; lora_bf16* dX;
    int M, K, N, r, tiles_m, tiles_n;
    int uniform_tiles;
    AdapterTable tb;
};

constexpr int kRowTile = 256;        // row-tile granularity of the dA/dB partials (and the GEMMs' larger tile)
constexpr int kComputeUnits = 256;   // of the one chip this library is written for
constexpr int kStreamChunk = 512;    // column-chunk width of operation (3)

// Calls launch(arguments) with a table no larger than the batch needs.
template <template <class> class Args, class F>
hipError_t with_few(const Args<AdapterTable>& a, F&& launch) {
    if (a.tb.G > kFewAdapters) return launch(a);
    Args<FewAdapters> few;
    static_assert(offsetof(Args<FewAdapters>, tb) == offsetof(Args<AdapterTable>, tb), "the table is the last member");
    memcpy((void*)&few, (const void*)&a, offsetof(Args<FewAdapters>, tb));
    few.tb.G = a.tb.G;
    memcpy(few.tb.row0, a.tb.row0, sizeof(few.tb.row0));
    memcpy(few.tb.a, a.tb.a, sizeof(few.tb.a));
    return launch(few);
}

void force_row_tile(int rows);        // 0 (automatic), or the small (128) / large (256) height of every kernel that has two
int forced_row_tile();                // an entry point reads this ONCE and hands the value to everything it launches
void force_slab_lookahead(int slabs); // 0 (automatic), or how many slabs ahead the GEMMs' copies run (1 or 2); read per GEMM launch,
                                      // results do not depend on it

// Longest row panel of a panel height.
inline int longest_panel(const AdapterTable& tb, int rows) {
    int n = 0;
    for (int g = 0; g < tb.G; ++g) {
        const SegmentPanels sp = segment_panels(tb, rows, g);
        const int len = sp.has_long ? rows + sp.rem : sp.has_short ? sp.rem : sp.nreg ? rows : 0;
        if (len > n) n = len;
    }
    return n;
}

// Row panels of a reduction over a [M, C] activation.  Every panel leaves an fp32 partial of C x r values, so taller
// panels mean less partial traffic, while a launch with fewer workgroups than compute units is bound by the latency of
// one workgroup's sweep: the largest of 1024 .. 64 rows that still gives about one workgroup of 512 columns per compute
// unit (256 rows at least when the large kernel heights are forced).  No launch takes more panels than this gives.
constexpr int kStreamFill = 224;     // workgroups that count as "about one per compute unit"
inline int fill_panel_rows(const AdapterTable& tb, int C, int forced) {
    const int chunks = (C + kStreamChunk - 1) / kStreamChunk, lowest = forced == 256 ? kRowTile : 64;
    int rows = 4 * kRowTile;
    while (rows > lowest && count_panels(tb, rows) * chunks < kStreamFill) rows >>= 1;
    return rows;
}

// Rows per panel of operation (3): that height, or a taller one where its rounds of workgroups and its fewer planes make
// up for it: a workgroup takes about 6 us + 2 us per 64 rows, a plane 64 ns per 1000 columns (at rank 32; the rule knows
// no rank, so that adapters of any rank are summed alike).  With the finalize launch, r = 32: 2999 rows, C = 4096: 64-row
// panels in two rounds 31 us, 128-row panels in one 26 us; 2048 rows: 32 planes 20.5 us, 16 planes 17.8 us.
// Evaluated once per entry-point call; the streaming launch and
// the finalize launch that adds its partial planes both receive the result.
inline int stream_panel_rows(const AdapterTable& tb, int C, int forced) {
    const int chunks = (C + kStreamChunk - 1) / kStreamChunk;
    auto cost = [&](int h) {
        const int64_t planes = count_panels(tb, h), steps = (longest_panel(tb, h) + 63) / 64;
        return (double)((planes * chunks + kComputeUnits - 1) / kComputeUnits) * (6.0 + 2.0 * (double)steps) + 6.4e-5 * (double)(planes * C);
    };
    int best = fill_panel_rows(tb, C, forced);
    for (int h = best * 2; h <= 4 * kRowTile; h <<= 1)
        if (cost(h) < cost(best)) best = h;
    return best;
}

// How operation (4) cuts its rows in a launch of its own.  A workgroup owns 64 columns of a panel and takes about 4 us + 1.3 us
// per 256 rows, a few of them on every compute unit; panels shorter than a segment cost the sum over them (finalize launch:
// 5 us) and an fp32 piece of r x K each.  Height 0: whole segments, no pieces.  (8192 x 4096, r = 16: 2048-row panels 16.7 us, 512-row
// panels 18.6 us, whole 43 us, as 64 workgroups; 5003 x 14336: whole 31 us, 512-row panels 34 us.)  The rule counts whole rounds of
// workgroups: one that prices their mean load instead makes taller panels, which chain more MFMAs on a sum (8192 x 26496, r = 16,
// fp32 error against 64 bits: 1024-row panels 0.99e-7, whole segments 1.90e-7; 4096 x 20480 0.92e-7 / 1.34e-7) and run longer than
// the rounds they save (6888 + 5702 rows x 4160, r = 16 29.7 -> 32.9 us).  It knows no rank, so that adapters of any rank are summed
// alike.  The panels are never more than fill_panel_rows gives for the same sizes, which is what the workspace provides for.
inline int plan_da(const AdapterTable& tb, int K, int forced) {
    if (forced == 256) return fill_panel_rows(tb, K, forced);
    const int64_t strips = K / 64;
    const int longest = longest_panel(tb, 1 << 30);
    auto cost = [&](int rows) {
        const int64_t panels = rows ? count_panels(tb, rows) : tb.G;
        const double rounds = (double)((panels * strips + kComputeUnits - 1) / kComputeUnits);
        return 4.0 + rounds * 1.3 * (double)((longest_panel(tb, rows ? rows : 1 << 30) + 255) / 256) +
               (rows ? 5.0 + 3.2e-5 * (double)(panels * K) : 0.0);
    };
    int best = 0, least = stream_panel_rows(tb, K, forced);
    if (least < kRowTile) least = kRowTile;
    for (int64_t h = least; h < longest; h <<= 1)
        if (cost((int)h) < cost(best)) best = (int)h;
    return best;
}

// Who adds the pieces of (4) in a launch of its own: the last workgroup of every strip, which saves the finalize launch (0.7 - 1.4 us of a
// backward pass) but reads all its pieces alone, where that launch spreads them over the chip.  us that the finalize launch
// takes longer, r = 16 and 32: 2 - 4 panels 0.7 - 1.1, 9 - 12 panels -0.1 - 1.1, 16 panels (4096 x 1024) -1.0, 32 panels (8192 x 512) -1.1; r = 64:
// 2 panels 0.7, 4 panels -0.1, 9 panels -0.3, 16 panels -2.4, 32 panels -4.1.  The order of the sum is the same either way.
inline bool strips_add_pieces(const AdapterTable& tb, int rows, int r) {
    int most = 0;
    for (int g = 0; rows && g < tb.G; ++g) {
        const SegmentPanels sp = segment_panels(tb, rows, g);
        if (sp.nreg + sp.has_long + sp.has_short > most) most = sp.nreg + sp.has_long + sp.has_short;
    }
    return most <= (r == 64 ? 3 : 12);
}

// ... and with the strips of dB beside it (split_ds_db): the two share the chip, two workgroups on a compute unit (at r = 64 one, which the
// rule does not know) as long as one after the other, at about 1.3 us (dA: the mask) or 0.6 us (dB) per 256 rows; the last workgroup of a
// strip adds its pieces: 2 us, and 40 ns per panel and 1000 columns.
constexpr int kLowestStripPanel = 512;               // (two rounds of a workgroup's eight 32-row blocks)
constexpr double kDaBlock = 1.3, kDbBlock = 0.6;     // us per 256 rows
struct StripLoad { double path, work; };           // us: the longest workgroup; all of them, per compute unit
inline StripLoad strip_load(const AdapterTable& tb, int C, int rows, double us_per_block) {
    const int64_t panels = rows ? count_panels(tb, rows) : tb.G;
    const double t = us_per_block * (double)((longest_panel(tb, rows ? rows : 1 << 30) + 255) / 256);
    return StripLoad{t, t * (double)(panels * (C / 64)) / kComputeUnits};
}
inline int plan_strips(const AdapterTable& tb, int C, double us_per_block, StripLoad beside, int highest = 1 << 30) {
    const int longest = longest_panel(tb, 1 << 30);
    auto cost = [&](int rows) {
        const StripLoad l = strip_load(tb, C, rows, us_per_block);
        const double path = l.path > beside.path ? l.path : beside.path, work = l.work + beside.work;
        return (path > work ? path : work) + (rows ? 2.0 + 4e-5 * (double)count_panels(tb, rows) * C : 0.0);
    };
    int best = 0, least = fill_panel_rows(tb, C, 0);
    if (least < kLowestStripPanel) least = kLowestStripPanel;
    for (int64_t h = least; h < longest && (h <= highest || best == 0); h <<= 1)
        if (cost((int)h) < cost(best) || (best == 0 && longest > highest)) best = (int)h;
    return best;
}
// dB: panels of at most 1024 rows, 1792 with a remainder where that is the whole segment (a remainder joins the last panel), that no
// wave chains more MFMAs on one sum than costs precision: fp32 error against 64 bits, 4096 columns, in panels of 512 rows and more / one panel /
// the one-pass form: 1800 rows 0.75e-7 / 0.93e-7 / 0.94e-7, 2047 rows 0.77e-7 / 0.98e-7 / 0.96e-7; 2999 rows, 1024 + 1975 0.94e-7, whole 1.21e-7,
// one pass 1.09e-7.  (2047 x 4096 x 4096 without dX, r = 16 19.0 -> 19.9 us, r = 64 27.4 -> 30.5; one pass 29.2, 44.5.)
inline int plan_db(const AdapterTable& tb, int N, int K, int rows_da) {
    const int h = plan_strips(tb, N, kDbBlock, strip_load(tb, K, rows_da, kDaBlock), 1024);
    bool whole_too_long = false;
    for (int g = 0; h == 1024 && g < tb.G; ++g) {
        const int len = tb.row0[g + 1] - tb.row0[g];
        whole_too_long |= len > 1792 && len < 2048;
    }
    return whole_too_long && fill_panel_rows(tb, N, 0) <= kLowestStripPanel ? kLowestStripPanel : h;
}
// Operation (3) as one pass over dY whose partial sums a second launch adds (lf_stream.hip), or as dS in one launch without
// partial sums (lf_ds.hip) and dB as further strips beside (4), reading dY twice: the latter while the pass is bound by the
// latency of its launches rather than by memory, and dS's workgroups, one to 16 rows and a compute unit, run at once or sweep
// short rows.  Backward without dX, times that the split is faster, r = 16 / 32 / 64, K = 1024: 1024 x 4096 1.26 / 1.49 / 1.54; 4096 x 3072
// 1.13 / 1.21 / 0.98, 4096 x 4096 1.06 / 1.17 / 0.99; in two rounds: 5003 x 1024 1.42 / 1.39 / 1.28, 6144 x 1024 1.07 / 1.12 / 0.98,
// 5003 x 2048 1.13 / 1.13 / 0.99, 6144 x 2048 1.04 / 1.04 / 0.89, 6144 x 4096 0.85 / 0.90 / 0.72.  K = 2048: 64 x 8192 0.82 (r = 16), 64 x 6144
// 0.81 (r = 64).
inline bool split_ds_db(const AdapterTable& tb, int M, int N, int K, int forced) {
    if (forced == 256 || N > 4096 || M > 6144 || (int64_t)M * K > (24ll << 20)) return false;
    int groups = 0;
    for (int g = 0; g < tb.G; ++g) groups += (tb.row0[g + 1] - tb.row0[g] + 15) / 16;
    return groups <= kComputeUnits || (int64_t)M * N <= (7ll << 20);
}

// Upper bound on the number of panels (planes of dA / dB partials) of any launch over M rows in G
// segments.  Height h gives at most M/h + G panels.  A height h < 256 is only chosen when height 2h
// gives fewer than kStreamFill panels, which needs M/(2h) < kStreamFill + G, i.e. M/h + G < 2 kStreamFill + 3 G.
inline int64_t max_stream_panels(int64_t M, int G) {
    const int64_t tall = M / kRowTile + G;
    int64_t low = M / 64 + G;
    if (low > 2 * kStreamFill + 3 * G) low = 2 * kStreamFill + 3 * G;
    return tall > low ? tall : low;
}

// `forced`: the row-tile knob as read by the entry point (0, 128 or 256).  The streaming launchers need
// StreamArgs::panel_rows, the finalize launchers FinalizeArgs::panel_rows_db / _da, filled in by the caller (strips that have
// counters, or whole segments, need no finalize launch).
hipError_t launch_down(const DownArgs& a, int forced, hipStream_t st);
hipError_t launch_fwd_gemm(const FwdGemmArgs& a, int forced, hipStream_t st);
hipError_t launch_stream_dsdb(StreamArgs a, hipStream_t st);
hipError_t launch_ds(const DsArgs& a, hipStream_t st);
hipError_t launch_strips(StripArgs a, hipStream_t st);
hipError_t launch_finalize_ds_db(const FinalizeArgs& a, hipStream_t st);
hipError_t launch_finalize_da(const FinalizeArgs& a, hipStream_t st);
hipError_t plan_strip_jobs(StripArgs& a);           // the members that the launcher sets
// `strips`: what the call will launch next; *took: it went into the GEMM's launch
hipError_t launch_bwd_dx(const DxGemmArgs& a, int forced, hipStream_t st, const StripArgs* strips = nullptr, bool* took = nullptr);
bool dx_takes_strips(const AdapterTable& tb, int M, int N, int K, int r, int forced, StripArgs strips);   // ... whether it would

// The output tiles of a GEMM's one or two launches (returns how many), as launch_fwd_gemm and launch_bwd_dx choose them.
struct GemmTile { int rows, columns, first_row; };
int gemm_tiles(const AdapterTable& tb, int M, int contraction, int columns, int r, int forced, GemmTile (&out)[2]);

// The kernels that launch_down, launch_fwd_gemm and launch_bwd_dx would launch for the same arguments (the GEMMs: returns how many).
struct DownLaunch { int rows, parts, ring; int64_t workgroups; };
struct GemmLaunch { int rows, columns, depth, stages, waves, asks_ahead; int64_t workgroups; };
DownLaunch down_launch(const DownArgs& a, int forced);
int fwd_gemm_launches(const FwdGemmArgs& a, int forced, GemmLaunch (&out)[2]);
int bwd_dx_launches(const DxGemmArgs& a, int forced, const StripArgs* strips, GemmLaunch (&out)[2]);

hipError_t launch_debug_mask(int64_t M, int64_t K, uint32_t T, uint32_t k0, uint32_t k1, uint8_t* keep,
                             hipStream_t st);

}  // namespace lf
