// Sums over the rows of an activation, in strips of 64 columns.  Operation (4) of the fused LoRA linear layer (Section 5.1,
// FusedLoRA Design), one pass over X with the mask regenerated:
//     dA[c,j] = q sum_i keep(i,j) X[i,j] dS[i,c]          (dS arrives scaled by s*q)
// and, beside it in the same launch, the dB half of operation (3) where dS has been formed by itself (lf_ds.hip):
//     dB[n,c] = sum_i dY[i,n] S'[i,c]
// A workgroup owns a strip of 64 columns (one 128-byte line of every row) over a panel of rows; each of its eight waves
// walks the 32-row blocks w, w + 8, ... of the panel by itself: global -> registers two blocks ahead, mask, LDS of the
// wave's own, transposing reads, 16x16x32 bf16 MFMAs.  No barrier until the waves' sums are added, pairwise.
// A panel is a whole segment where that leaves the chip enough workgroups (the sum is then the gradient itself); otherwise the
// panels (plan_da, with dB beside it plan_strips) leave fp32 pieces that the last workgroup of the strip adds in a fixed order or,
// where there are many (strips_add_pieces), a finalize launch in the same one.  Repeated runs agree bit for bit.
// What bounds it: the mask of dA (about 0.85 us of a compute unit per 256 rows x 64 columns; 13 vector instructions a
// column pair), then memory.  (3) and (4) in two launches instead of four, us: 256 x 1024 x 1024, r = 16 12.2 -> 7.6; 1531 x 4096 ->
// 1024 in three segments, r = 64 29 -> 16.4; 2999 x 4096 x 4096, r = 32 37 -> 29; 2048 x 4096 x 4096, r = 16 22 -> 18.6.
#include "lf_device.h"
#include "lf_internal.h"
#include "lf_strips.h"

namespace lf {

template <int CB, class TB>                        // r / 16
__global__ void __launch_bounds__(DA_THREADS, CB == 4 ? 2 : 4) strip_kernel(StripArgsOf<TB> p) {
    fetch_args<StripArgsOf<TB>>();
    extern __shared__ __attribute__((aligned(16))) char smem[];
    strip_of<CB>(p, blockIdx.x, smem);
}

// Workgroups of a job: strips x (panels, and with counters the empty segments).
static void plan_job(const AdapterTable& tb, StripJob& job) {
    job.blocks = 0;
    if (!job.big && !job.out) return;
    int tiles = tb.G;
    if (job.panel_rows) {
        tiles = job.panels = count_panels(tb, job.panel_rows);
        if (job.counters)
            for (int g = 0; g < tb.G; ++g) tiles += tb.row0[g] == tb.row0[g + 1];
    }
    job.blocks = tiles * (job.C / DA_STRIP);
}

template <int CB>
static hipError_t launch_strips_t(const StripArgs& a, hipStream_t st) {
    constexpr int lds = strip_lds(CB);
    if (a.a.blocks + a.b.blocks == 0) return hipSuccess;
    return with_few(a, [&](const auto& b) {
        constexpr auto kernel = strip_kernel<CB, std::decay_t<decltype(b.tb)>>;
        static bool attr_set = false;              // one flag per instantiation
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)(b.a.blocks + b.b.blocks)), dim3(DA_THREADS), lds, st, b);
        return hipGetLastError();
    });
}

hipError_t plan_strip_jobs(StripArgs& a) {
    if ((a.a.panel_rows && a.a.panel_rows < DA_BLOCK) || (a.b.panel_rows && a.b.panel_rows < DA_BLOCK)) return hipErrorInvalidValue;
    plan_job(a.tb, a.a);
    plan_job(a.tb, a.b);
    a.b_first = a.b.blocks && kDbBlock * longest_panel(a.tb, a.b.panel_rows ? a.b.panel_rows : 1 << 30) >
                                  kDaBlock * longest_panel(a.tb, a.a.panel_rows ? a.a.panel_rows : 1 << 30);
    return hipSuccess;
}

hipError_t launch_strips(StripArgs a, hipStream_t st) {
    const hipError_t e = plan_strip_jobs(a);
    if (e != hipSuccess) return e;
    switch (a.r) {
        case 16: return launch_strips_t<1>(a, st);
        case 32: return launch_strips_t<2>(a, st);
        case 64: return launch_strips_t<4>(a, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace lf
