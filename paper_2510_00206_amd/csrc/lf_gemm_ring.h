// Arguments of the small-tile GEMM kernels (lf_gemm_ring.hip).
#pragma once
#include "lf_internal.h"

namespace lf {

// Operation (2): tok X [M,KC], out W [NC,KC], ltok S' [M,r], lout B [G,NC,r], res Y [M,NC].
// Operation (5): tok dY [M,KC], out W [KC,NC], ltok dS [M,r], lout A [G,r,NC], res dX [M,NC].
// r == 0: no LoRA term.
template <class TB>
struct RingArgsOf {
    const lora_bf16* tok; const lora_bf16* out; const lora_bf16* ltok; const lora_bf16* lout; lora_bf16* res;
    int M, KC, NC, r, tiles_m, tiles_n;
    int row_lo, row_hi;                              // the launch covers rows [row_lo, row_hi) of the packed batch
    TB tb;
};
using RingArgs = RingArgsOf<AdapterTable>;

// Operation (5) with (4), and dB if there is such a job, as further workgroups of the launch: the members of both.
template <class TB>
struct RingStripsArgsOf {
    const lora_bf16* tok; const lora_bf16* out; const lora_bf16* ltok; const lora_bf16* lout; lora_bf16* res;
    int M, KC, NC, r, tiles_m, tiles_n;
    int row_lo, row_hi;
    StripJob a, b;
    int b_first, accumulate;
    TB tb;
};
using RingStripsArgs = RingStripsArgsOf<AdapterTable>;

constexpr int kRingKinds = 6;
constexpr int kRingTiles[kRingKinds][2] = {{128, 256}, {128, 128}, {64, 128}, {64, 64}, {32, 64}, {128, 64}};   // rows x columns

// A 32 x 64 tile is shared by two workgroups, 32 columns each, while there is a compute unit for every one of them (beside strips: with_ring_strips).
constexpr bool ring_halves(int tiles_m, int tiles_n) { return 2 * (int64_t)tiles_m * tiles_n <= kComputeUnits; }

hipError_t launch_ring(int kind, bool col, const RingArgs& a, hipStream_t st);
GemmLaunch ring_launch(int kind, bool col, const RingArgs& a);                    // ... what it would launch

constexpr bool ring_takes_strips(int kind, int r) { return (kind == 3 || kind == 4) && (r == 16 || r == 32); }
hipError_t launch_ring_strips(int kind, const RingStripsArgs& a, hipStream_t st);
GemmLaunch ring_strips_launch(int kind, const RingStripsArgs& a);

}  // namespace lf
