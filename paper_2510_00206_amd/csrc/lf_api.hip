// C ABI of the fused LoRA linear layer: argument validation, the per-adapter lookup table,
// workspace carving and the launch sequences of the five fused operations (Section 5.1).
// Nothing here allocates device memory or synchronises; every kernel goes to the caller's stream.
#include <math.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "../../include/lorafusion.h"
#include "lf_internal.h"

using namespace lf;

namespace {

inline bool misaligned(const void* p, size_t a = 16) { return ((uintptr_t)p & (a - 1)) != 0; }
inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

lora_status check_shape(int64_t M, int64_t K, int64_t N, int32_t r, int32_t G) {
    if (M < 0 || K <= 0 || N <= 0 || M >= (1ll << 31) || K >= (1ll << 31) || N >= (1ll << 31)) return LORA_ERR_SHAPE;
    if (G < 1) return LORA_ERR_SHAPE;
    if ((K & 63) || (N & 63) || !(r == 16 || r == 32 || r == 64) || G > kMaxAdapters) return LORA_ERR_UNSUPPORTED;
    if (K > (1 << 22) || N > (1 << 22)) return LORA_ERR_UNSUPPORTED;   // per-lane slab offsets are 32-bit
    return LORA_OK;
}

// Threshold and keys exactly as the written specification of the hash: p is an IEEE float
// widened to double, T = min(65535, floor(p * 65536)); k0 = mix(seed_lo ^ C5), k1 = mix(seed_hi + k0).
lora_status fill_adapter(AdapterTable& tb, int g, float s, float p, uint64_t seed) {
    if (!(p >= 0.0f && p < 1.0f) || !isfinite(s)) return LORA_ERR_PARAM;
    double t = floor((double)p * 65536.0);
    uint32_t T = t > 65535.0 ? 65535u : (uint32_t)t;
    tb.a[g].T = T;
    tb.a[g].q = (float)(65536.0 / (65536.0 - (double)T));
    tb.a[g].s = s;
    tb.a[g].k0 = mix32((uint32_t)(seed & 0xFFFFFFFFull) ^ kC5);
    tb.a[g].k1 = mix32((uint32_t)(seed >> 32) + tb.a[g].k0);
    return LORA_OK;
}

// ranks == NULL: every adapter has the call's rank r
lora_status build_table(AdapterTable& tb, int64_t M, int32_t r, int32_t G, const int64_t* off, const float* s,
                        const float* p, const uint64_t* seeds, const int32_t* ranks) {
    memset(&tb, 0, sizeof(tb));
    tb.G = G;
    for (int g = 0; g < G; ++g) {
        const int32_t rg = ranks ? ranks[g] : r;
        if (!(rg == 16 || rg == 32 || rg == 64) || rg > r) return LORA_ERR_UNSUPPORTED;
        tb.a[g].rank = rg;
    }
    if (off[0] != 0 || off[G] != M) return LORA_ERR_SEGMENTS;
    for (int g = 0; g < G; ++g)
        if (off[g + 1] < off[g]) return LORA_ERR_SEGMENTS;
    for (int g = 0; g <= G; ++g) tb.row0[g] = (int)off[g];
    for (int g = 0; g < G; ++g) {
        lora_status st = fill_adapter(tb, g, s[g], p[g], seeds[g]);
        if (st != LORA_OK) return st;
    }
    return LORA_OK;
}

// A table that knows the segments only, for the diagnostics of what a launch would choose over C columns.
lora_status segments_only(AdapterTable& tb, int64_t M, int64_t C, int32_t G, const int64_t* off) {
    if (M < 0 || C <= 0 || M >= (1ll << 31) || C >= (1ll << 31) || G < 1) return LORA_ERR_SHAPE;
    if (G > kMaxAdapters) return LORA_ERR_UNSUPPORTED;
    memset(&tb, 0, sizeof(tb));
    tb.G = G;
    if (off[0] != 0 || off[G] != M) return LORA_ERR_SEGMENTS;
    for (int g = 0; g < G; ++g)
        if (off[g + 1] < off[g]) return LORA_ERR_SEGMENTS;
    for (int g = 0; g <= G; ++g) tb.row0[g] = (int)off[g];
    return LORA_OK;
}

// Optional per-kernel timing (diagnostic): HIP events bracket every launch on the caller's stream.
struct ProfRec { hipEvent_t beg, end; int id; };
bool g_prof_on = false;
std::vector<ProfRec> g_prof;

template <typename F>
hipError_t timed(int id, hipStream_t st, F&& launch) {
    if (!g_prof_on) return launch();
    ProfRec r{nullptr, nullptr, id};
    if (hipEventCreate(&r.beg) != hipSuccess) return hipErrorUnknown;
    if (hipEventCreate(&r.end) != hipSuccess) { (void)hipEventDestroy(r.beg); return hipErrorUnknown; }
    hipError_t e = hipEventRecord(r.beg, st);
    if (e == hipSuccess) e = launch();
    const hipError_t e2 = hipEventRecord(r.end, st);
    g_prof.push_back(r);
    return e != hipSuccess ? e : e2;
}

// What one backward call launches with: the knob is read once and the panel heights are chosen here, for the launches that
// leave partial sums and for those that add them, so that a change of the knob by another thread in the middle of a call
// cannot make the two disagree.
struct BwdPlan {
    int forced;
    bool split;                // dS by itself, dB beside (4)
    int rows_db, rows_da;      // panel heights (0: whole segments, no partial sums)
};

BwdPlan plan_bwd(const AdapterTable& tb, int64_t M, int64_t K, int64_t N) {
    BwdPlan pl;
    pl.forced = forced_row_tile();
    pl.split = split_ds_db(tb, (int)M, (int)N, (int)K, pl.forced);
    pl.rows_da = pl.split ? plan_strips(tb, (int)K, kDaBlock, StripLoad{0, 0}) : plan_da(tb, (int)K, pl.forced);
    pl.rows_db = pl.split ? plan_db(tb, (int)N, (int)K, pl.rows_da) : stream_panel_rows(tb, (int)N, pl.forced);
    return pl;
}

struct Workspace {
    lora_bf16* dS; float* part_ds; float* part_db; float* part_da; size_t bytes;
    uint32_t* counters;        // NULL: finalize_da adds the planes
    int n_counters;
};

// planes_db / planes_da: fp32 planes of dB / dA partials to provide for (one per row panel)
Workspace carve(void* base, int64_t M, int64_t K, int64_t N, int32_t r, int64_t planes_db, int64_t planes_da, int64_t chunks) {
    size_t off = 0;
    Workspace w{};
    char* b = (char*)base;
    w.dS = (lora_bf16*)(b + off);      off += align_up((size_t)M * r * 2);
    w.part_ds = (float*)(b + off);     off += align_up((size_t)chunks * M * r * 4);
    w.part_db = (float*)(b + off);     off += align_up((size_t)planes_db * N * r * 4);
    w.part_da = (float*)(b + off);     off += align_up((size_t)planes_da * r * K * 4);
    w.bytes = off;
    return w;
}

int64_t stream_chunks(int64_t N) { return (N + kStreamChunk - 1) / kStreamChunk; }

// The caller-provided workspace is sized before the call's panel heights are known: for the most panels
// any launch over M rows in G segments can choose.
size_t workspace_bytes_of(int64_t M, int64_t K, int64_t N, int32_t r, int32_t G) {
    const int64_t tiles = max_stream_panels(M, G);
    return carve(nullptr, M, K, N, r, tiles, tiles, stream_chunks(N)).bytes;
}

// What a call lays out in `bytes` of it: the planes that its launches write, and behind them the counters of the strips where
// those add their pieces themselves.
Workspace lay_out(void* base, size_t bytes, int64_t M, int64_t K, int64_t N, int32_t r, const AdapterTable& tb, BwdPlan& pl) {
    Workspace w = carve(base, M, K, N, r, pl.rows_db ? count_panels(tb, pl.rows_db) : 0,
                        pl.rows_da ? count_panels(tb, pl.rows_da) : 0, pl.split ? 0 : stream_chunks(N));
    const int64_t n = tb.G * ((pl.rows_da ? K / 64 : 0) + (pl.split && pl.rows_db ? N / 64 : 0));
    if (n && w.bytes + (size_t)n * 4 <= bytes && (pl.split || strips_add_pieces(tb, pl.rows_da, r))) {
        w.counters = (uint32_t*)((char*)base + w.bytes);
        w.n_counters = (int)n;
    } else if (pl.split) {
        pl.rows_db = 0;        // (nothing else would add the pieces of dB)
    }
    return w;
}

// Operation (4), and dB beside it where (3) forms dS by itself.
StripArgs strip_args(const lora_bf16* X, const lora_bf16* S, const lora_bf16* dY, int64_t K, int64_t N, int32_t r, const AdapterTable& tb,
                     float* dA, float* dB, int accumulate, const Workspace& ws, const BwdPlan& pl) {
    StripArgs s{{X, ws.dS, dA, ws.part_da, pl.rows_da ? ws.counters : nullptr, (int)K, pl.rows_da, 0, 0}, {}, 0, r, accumulate, tb};
    if (pl.split)
        s.b = StripJob{dY, S, dB, ws.part_db, pl.rows_db ? ws.counters + (pl.rows_da ? tb.G * (K / 64) : 0) : nullptr, (int)N, pl.rows_db, 0, 0};
    return s;
}

lora_status fwd_impl(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                     int64_t M, int64_t K, int64_t N, int32_t r, const AdapterTable& tb,
                     lora_bf16* Y, lora_bf16* S, hipStream_t st) {
    const int forced = forced_row_tile();              // the knob is read once per call
    DownArgs d{X, A, S, (int)M, (int)K, r, tb};
    if (timed(LORA_PROF_DOWN, st, [&] { return launch_down(d, forced, st); }) != hipSuccess) return LORA_ERR_HIP;
    FwdGemmArgs f{X, W, S, B, Y, (int)M, (int)K, (int)N, r, 0, 0, 0, tb};
    if (timed(LORA_PROF_FWD_GEMM, st, [&] { return launch_fwd_gemm(f, forced, st); }) != hipSuccess) return LORA_ERR_HIP;
    return LORA_OK;
}

lora_status bwd_impl(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                     const lora_bf16* S, const lora_bf16* dY, int64_t M, int64_t K, int64_t N, int32_t r,
                     const AdapterTable& tb, lora_bf16* dX, float* dA, float* dB, int accumulate,
                     const Workspace& ws, const BwdPlan& pl, hipStream_t st) {
    const int chunks = (int)stream_chunks(N);
    FinalizeArgs fin{ws.part_ds, ws.dS, ws.part_db, dB, ws.part_da, dA,
                     (int)M, (int)K, (int)N, r, chunks, accumulate, pl.rows_db, pl.rows_da, ws.counters, ws.n_counters, tb};
    if (pl.split) {
        DsArgs s3{dY, B, ws.dS, ws.counters, ws.n_counters, (int)M, (int)N, r, tb};
        if (timed(LORA_PROF_DS_DB, st, [&] { return launch_ds(s3, st); }) != hipSuccess) return LORA_ERR_HIP;
    } else {
        StreamArgs s3{dY, S, B, ws.part_db, ws.part_ds, (int)M, (int)N, r, 0, 0, pl.rows_db, tb};
        if (timed(LORA_PROF_DS_DB, st, [&] { return launch_stream_dsdb(s3, st); }) != hipSuccess) return LORA_ERR_HIP;
        if (timed(LORA_PROF_FIN_DS_DB, st, [&] { return launch_finalize_ds_db(fin, st); }) != hipSuccess) return LORA_ERR_HIP;
    }
    const StripArgs s4 = strip_args(X, S, dY, K, N, r, tb, dA, dB, accumulate, ws, pl);
    // (5) right after (3): it re-reads dY while that pass's copy still sits in the memory-side cache
    bool took_s4 = false;
    if (dX) {
        DxGemmArgs g5{dY, W, ws.dS, A, dX, (int)M, (int)K, (int)N, r, 0, 0, 0, tb};
        if (timed(LORA_PROF_DX_GEMM, st, [&] { return launch_bwd_dx(g5, pl.forced, st, &s4, &took_s4); }) != hipSuccess) return LORA_ERR_HIP;
    }
    if (!took_s4 && timed(LORA_PROF_DA, st, [&] { return launch_strips(s4, st); }) != hipSuccess) return LORA_ERR_HIP;
    if (pl.rows_da && !ws.counters &&
        timed(LORA_PROF_FIN_DA, st, [&] { return launch_finalize_da(fin, st); }) != hipSuccess) return LORA_ERR_HIP;
    return LORA_OK;
}

// ---- scratch of the allocation-free backward ------------------------------------------------------
// One array per GPU, part of the library's device image: it exists from the moment the image is loaded
// on a device until the process ends.  In host code `scratch` is only a handle for the symbol, never a
// device address: the address of each device's copy is asked for once (with that device current) and
// only that pointer is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[LORA_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];        // per device, filled on the first call on that device

lora_status scratch_of_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LORA_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LORA_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return LORA_OK;
}

}  // namespace

extern "C" {

size_t lora_bwd_workspace_bytes(int64_t M, int64_t K, int64_t N, int32_t r, int32_t G) {
    if (check_shape(M, K, N, r, G) != LORA_OK) return 0;
    return workspace_bytes_of(M, K, N, r, G);
}

lora_status multi_lora_fwd_ranked(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                                  int64_t M, int64_t K, int64_t N, int32_t r, int32_t G,
                                  const int64_t* seg_offsets, const int32_t* ranks, const float* s, const float* p,
                                  const uint64_t* seeds, lora_bf16* Y, lora_bf16* S_saved, lora_stream stream) {
    // with M == 0 the token-sized arrays are empty and may be NULL
    if (!W || !A || !B || !seg_offsets || !s || !p || !seeds) return LORA_ERR_NULL;
    if (M != 0 && (!X || !Y || !S_saved)) return LORA_ERR_NULL;
    lora_status st = check_shape(M, K, N, r, G);
    if (st != LORA_OK) return st;
    if (misaligned(X) || misaligned(W) || misaligned(A) || misaligned(B) || misaligned(Y) || misaligned(S_saved))
        return LORA_ERR_ALIGN;
    AdapterTable tb;
    st = build_table(tb, M, r, G, seg_offsets, s, p, seeds, ranks);
    if (st != LORA_OK) return st;
    if (M == 0) return LORA_OK;
    return fwd_impl(X, W, A, B, M, K, N, r, tb, Y, S_saved, (hipStream_t)stream);
}

lora_status multi_lora_fwd(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                           int64_t M, int64_t K, int64_t N, int32_t r, int32_t G,
                           const int64_t* seg_offsets, const float* s, const float* p, const uint64_t* seeds,
                           lora_bf16* Y, lora_bf16* S_saved, lora_stream stream) {
    return multi_lora_fwd_ranked(X, W, A, B, M, K, N, r, G, seg_offsets, nullptr, s, p, seeds, Y, S_saved, stream);
}

lora_status lora_fwd(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                     int64_t M, int64_t K, int64_t N, int32_t r, float s, float p, uint64_t seed,
                     lora_bf16* Y, lora_bf16* S_saved, lora_stream stream) {
    const int64_t off[2] = {0, M};
    return multi_lora_fwd(X, W, A, B, M, K, N, r, 1, off, &s, &p, &seed, Y, S_saved, stream);
}

lora_status multi_lora_bwd_ranked(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                                  const lora_bf16* S_saved, const lora_bf16* dY,
                                  int64_t M, int64_t K, int64_t N, int32_t r, int32_t G,
                                  const int64_t* seg_offsets, const int32_t* ranks, const float* s, const float* p,
                                  const uint64_t* seeds, lora_bf16* dX, float* dA, float* dB, int accumulate,
                                  void* workspace, size_t workspace_bytes, lora_stream stream) {
    if (!W || !A || !B || !dA || !dB || !workspace || !seg_offsets || !s || !p || !seeds) return LORA_ERR_NULL;
    if (M != 0 && (!X || !S_saved || !dY)) return LORA_ERR_NULL;
    lora_status st = check_shape(M, K, N, r, G);
    if (st != LORA_OK) return st;
    if (misaligned(X) || misaligned(W) || misaligned(A) || misaligned(B) || misaligned(S_saved) ||
        misaligned(dY) || misaligned(dA) || misaligned(dB) || (dX && misaligned(dX)) || misaligned(workspace, 256))
        return LORA_ERR_ALIGN;
    AdapterTable tb;
    st = build_table(tb, M, r, G, seg_offsets, s, p, seeds, ranks);
    if (st != LORA_OK) return st;
    const size_t need = workspace_bytes_of(M, K, N, r, G);
    if (workspace_bytes < need) return LORA_ERR_WORKSPACE;
    BwdPlan pl = plan_bwd(tb, M, K, N);
    const Workspace ws = lay_out(workspace, need, M, K, N, r, tb, pl);
    return bwd_impl(X, W, A, B, S_saved, dY, M, K, N, r, tb, dX, dA, dB, accumulate,
                    ws, pl, (hipStream_t)stream);
}

lora_status multi_lora_bwd(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                           const lora_bf16* S_saved, const lora_bf16* dY,
                           int64_t M, int64_t K, int64_t N, int32_t r, int32_t G,
                           const int64_t* seg_offsets, const float* s, const float* p, const uint64_t* seeds,
                           lora_bf16* dX, float* dA, float* dB, int accumulate,
                           void* workspace, size_t workspace_bytes, lora_stream stream) {
    return multi_lora_bwd_ranked(X, W, A, B, S_saved, dY, M, K, N, r, G, seg_offsets, nullptr, s, p, seeds, dX, dA, dB,
                                 accumulate, workspace, workspace_bytes, stream);
}

lora_status lora_bwd(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                     const lora_bf16* S_saved, const lora_bf16* dY,
                     int64_t M, int64_t K, int64_t N, int32_t r, float s, float p, uint64_t seed,
                     lora_bf16* dX, float* dA, float* dB, int accumulate,
                     void* workspace, size_t workspace_bytes, lora_stream stream) {
    const int64_t off[2] = {0, M};
    return multi_lora_bwd(X, W, A, B, S_saved, dY, M, K, N, r, 1, off, &s, &p, &seed, dX, dA, dB, accumulate,
                          workspace, workspace_bytes, stream);
}

lora_status lora_bwd_noalloc(const lora_bf16* X, const lora_bf16* W, const lora_bf16* A, const lora_bf16* B,
                             const lora_bf16* S_saved, const lora_bf16* dY,
                             int64_t M, int64_t K, int64_t N, int32_t r, float s, float p, uint64_t seed,
                             lora_bf16* dX, float* dA, float* dB, int accumulate, lora_stream stream) {
    if (!W || !A || !B || !dA || !dB) return LORA_ERR_NULL;
    if (M != 0 && (!X || !S_saved || !dY)) return LORA_ERR_NULL;
    lora_status st = check_shape(M, K, N, r, 1);
    if (st != LORA_OK) return st;
    if (misaligned(X) || misaligned(W) || misaligned(A) || misaligned(B) || misaligned(S_saved) ||
        misaligned(dY) || misaligned(dA) || misaligned(dB) || (dX && misaligned(dX)))
        return LORA_ERR_ALIGN;
    const int64_t off[2] = {0, M};
    AdapterTable tb;
    st = build_table(tb, M, r, 1, off, &s, &p, &seed, nullptr);
    if (st != LORA_OK) return st;
    // The limit goes by the most panels of these sizes (fill_panel_rows), so that it does not move with the launches'
    // choice of taller ones; the planes laid out are exactly those that this call's launches will write.
    BwdPlan pl = plan_bwd(tb, M, K, N);
    if (carve(nullptr, M, K, N, r, count_panels(tb, fill_panel_rows(tb, (int)N, pl.forced)),
              count_panels(tb, fill_panel_rows(tb, (int)K, pl.forced)), stream_chunks(N)).bytes > (size_t)LORA_NOALLOC_SCRATCH_BYTES)
        return LORA_ERR_WORKSPACE;
    void* base = nullptr;
    st = scratch_of_current_device(&base);
    if (st != LORA_OK) return st;
    // Nothing in the scratch has to start at zero: every partial plane and every dS element that a
    // later kernel of this call reads is written by an earlier kernel of this call.
    const Workspace ws = lay_out(base, (size_t)LORA_NOALLOC_SCRATCH_BYTES, M, K, N, r, tb, pl);
    return bwd_impl(X, W, A, B, S_saved, dY, M, K, N, r, tb, dX, dA, dB, accumulate, ws, pl, (hipStream_t)stream);
}

lora_status lora_debug_mask(int64_t M, int64_t K, float p, uint64_t seed, uint8_t* keep, lora_stream stream) {
    if (M < 0 || K < 0 || M >= (1ll << 31) || K >= (1ll << 31)) return LORA_ERR_SHAPE;
    AdapterTable tb;
    lora_status st = fill_adapter(tb, 0, 1.0f, p, seed);
    if (st != LORA_OK) return st;
    if (M == 0 || K == 0) return LORA_OK;
    if (!keep) return LORA_ERR_NULL;
    if (launch_debug_mask(M, K, tb.a[0].T, tb.a[0].k0, tb.a[0].k1, keep, (hipStream_t)stream) != hipSuccess)
        return LORA_ERR_HIP;
    return LORA_OK;
}

lora_status lora_debug_stream_panels(int64_t M, int64_t C, int32_t G, const int64_t* seg_offsets,
                                     int32_t* panel_rows, int64_t* panels, int64_t* panels_bound) {
    if (!seg_offsets || !panel_rows || !panels || !panels_bound) return LORA_ERR_NULL;
    AdapterTable tb;
    const lora_status st = segments_only(tb, M, C, G, seg_offsets);
    if (st != LORA_OK) return st;
    *panel_rows = stream_panel_rows(tb, (int)C, forced_row_tile());
    *panels = count_panels(tb, *panel_rows);
    *panels_bound = max_stream_panels(M, G);
    return LORA_OK;
}

lora_status lora_debug_da_panels(int64_t M, int64_t K, int32_t G, const int64_t* seg_offsets,
                                 int32_t* panel_rows, int64_t* panels, int64_t* panels_bound) {
    if (!seg_offsets || !panel_rows || !panels || !panels_bound) return LORA_ERR_NULL;
    AdapterTable tb;
    const lora_status st = segments_only(tb, M, K, G, seg_offsets);
    if (st != LORA_OK) return st;
    *panel_rows = plan_da(tb, (int)K, forced_row_tile());
    *panels = *panel_rows ? count_panels(tb, *panel_rows) : 0;
    *panels_bound = max_stream_panels(M, G);
    return LORA_OK;
}

lora_status lora_debug_bwd_plan(int64_t M, int64_t K, int64_t N, int32_t r, int32_t G, const int64_t* seg_offsets, int32_t need_dx,
                                size_t scratch, lora_bwd_plan* plan) {
    if (!seg_offsets || !plan) return LORA_ERR_NULL;
    lora_status st = check_shape(M, K, N, r, G);
    if (st != LORA_OK) return st;
    AdapterTable tb;
    st = segments_only(tb, M, K, G, seg_offsets);
    if (st != LORA_OK) return st;
    BwdPlan pl = plan_bwd(tb, M, K, N);
    alignas(256) char base[256];                       // (addresses only: nothing is read or written through them)
    const lora_bf16* any = (const lora_bf16*)base;
    const Workspace ws = lay_out(base, scratch ? scratch : workspace_bytes_of(M, K, N, r, G), M, K, N, r, tb, pl);
    *plan = lora_bwd_plan{pl.split, pl.rows_db, pl.rows_da, ws.counters != nullptr,
                          need_dx && dx_takes_strips(tb, (int)M, (int)N, (int)K, r, pl.forced,
                                                     strip_args(any, any, any, K, N, r, tb, (float*)base, (float*)base, 0, ws, pl)),
                          (int64_t)(ws.bytes + (size_t)ws.n_counters * 4)};
    return LORA_OK;
}

lora_status lora_debug_gemm_tiles(int64_t M, int64_t contraction, int64_t columns, int32_t r, int32_t G,
                                  const int64_t* seg_offsets, int32_t* parts, int32_t* tile_rows, int32_t* tile_columns,
                                  int64_t* first_row) {
    if (!seg_offsets || !parts || !tile_rows || !tile_columns || !first_row) return LORA_ERR_NULL;
    lora_status st = check_shape(M, contraction, columns, r ? r : 16, G);
    if (st != LORA_OK) return st;
    AdapterTable tb;
    st = segments_only(tb, M, contraction, G, seg_offsets);
    if (st != LORA_OK) return st;
    GemmTile t[2];
    *parts = gemm_tiles(tb, (int)M, (int)contraction, (int)columns, r, forced_row_tile(), t);
    for (int i = 0; i < *parts; ++i) {
        tile_rows[i] = t[i].rows;
        tile_columns[i] = t[i].columns;
        first_row[i] = t[i].first_row;
    }
    return LORA_OK;
}

static lora_gemm_launch as_abi(const GemmLaunch& g) {
    return lora_gemm_launch{g.rows, g.columns, g.depth, g.stages, g.waves, g.asks_ahead, g.workgroups};
}

lora_status lora_debug_launches(int64_t M, int64_t K, int64_t N, int32_t r, int32_t G, const int64_t* seg_offsets,
                                lora_launches* out) {
    if (!seg_offsets || !out) return LORA_ERR_NULL;
    lora_status st = check_shape(M, K, N, r, G);
    if (st != LORA_OK) return st;
    AdapterTable tb;
    st = segments_only(tb, M, K, G, seg_offsets);
    if (st != LORA_OK) return st;
    *out = lora_launches{};
    if (M == 0) return LORA_OK;
    BwdPlan pl = plan_bwd(tb, M, K, N);
    alignas(256) char base[256];                       // (addresses only, as in lora_debug_bwd_plan)
    lora_bf16* any = (lora_bf16*)base;
    const Workspace ws = lay_out(base, workspace_bytes_of(M, K, N, r, G), M, K, N, r, tb, pl);
    const StripArgs strips = strip_args(any, any, any, K, N, r, tb, (float*)base, (float*)base, 0, ws, pl);
    const DownLaunch d = down_launch(DownArgs{any, any, any, (int)M, (int)K, r, tb}, pl.forced);
    out->down_rows = d.rows;
    out->down_parts = d.parts;
    out->down_ring = d.ring;
    out->down_workgroups = d.workgroups;
    GemmLaunch g[2];
    int n = fwd_gemm_launches(FwdGemmArgs{any, any, any, any, any, (int)M, (int)K, (int)N, r, 0, 0, 0, tb}, pl.forced, g);
    for (int i = 0; i < n; ++i) out->fwd[i] = as_abi(g[i]);
    n = bwd_dx_launches(DxGemmArgs{any, any, any, any, any, (int)M, (int)K, (int)N, r, 0, 0, 0, tb}, pl.forced, &strips, g);
    for (int i = 0; i < n; ++i) out->dx[i] = as_abi(g[i]);
    return LORA_OK;
}

const char* lora_status_string(lora_status st) {
    switch (st) {
        case LORA_OK: return "ok";
        case LORA_ERR_NULL: return "a required pointer is NULL";
        case LORA_ERR_SHAPE: return "invalid shape";
        case LORA_ERR_ALIGN: return "pointer not sufficiently aligned";
        case LORA_ERR_PARAM: return "dropout probability outside [0,1) or non-finite scale";
        case LORA_ERR_SEGMENTS: return "segment offsets must rise from 0 to M";
        case LORA_ERR_WORKSPACE: return "workspace too small (lora_bwd_noalloc: problem beyond the built-in scratch)";
        case LORA_ERR_UNSUPPORTED: return "unsupported size (K, N multiples of 64; r in {16,32,64}; G <= 64)";
        case LORA_ERR_HIP: return "kernel launch failed";
    }
    return "unknown status";
}

int lora_version(void) { return 100; }

lora_status lora_set_row_tile(int32_t rows) {
    if (rows != 0 && rows != 128 && rows != 256) return LORA_ERR_PARAM;
    force_row_tile(rows);
    return LORA_OK;
}

lora_status lora_set_slab_lookahead(int32_t slabs) {
    if (slabs < 0 || slabs > 2) return LORA_ERR_PARAM;
    force_slab_lookahead(slabs);
    return LORA_OK;
}

lora_status lora_profile_begin(void) {
    for (ProfRec& r : g_prof) { (void)hipEventDestroy(r.beg); (void)hipEventDestroy(r.end); }
    g_prof.clear();
    g_prof_on = true;
    return LORA_OK;
}

lora_status lora_profile_end(float* ms_total, int32_t* launches) {
    g_prof_on = false;
    if (!ms_total || !launches) return LORA_ERR_NULL;
    for (int i = 0; i < LORA_PROF_KERNELS; ++i) { ms_total[i] = 0.f; launches[i] = 0; }
    lora_status st = LORA_OK;
    for (ProfRec& r : g_prof) {
        float ms = 0.f;
        if (hipEventSynchronize(r.end) != hipSuccess || hipEventElapsedTime(&ms, r.beg, r.end) != hipSuccess)
            st = LORA_ERR_HIP;
        else if (r.id >= 0 && r.id < LORA_PROF_KERNELS) { ms_total[r.id] += ms; launches[r.id] += 1; }
        (void)hipEventDestroy(r.beg);
        (void)hipEventDestroy(r.end);
    }
    g_prof.clear();
    return st;
}

}  // extern "C"
