"""The small-tile GEMM kernels, the 192-row large tiles and the split of a launch between two kernels, at sizes on the
edges of their tiles: every output against the oracle, and Y, S' and dX bit for bit against the 256 x 256 tiles (the
contraction is walked in the same order by every kernel, so the tolerance between them is zero)."""
import pytest
import torch

from paper_2510_00206_amd import binding, workloads
from gpu_util import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# (K, N, r, segments).  Which tiles the two GEMMs take follows from the sizes: 32 x 64 and 64 x 64 (few rows), 128 x 64,
# 64 x 128 and 128 x 128 (some hundred rows by some thousand columns), 128 x 256 and 192 x 256 (more), and two launches
# for one GEMM where the last round of tiles would be nearly empty.
CASES = [
    (64, 64, 16, (1,)),                      # one row, one slab, one column block
    (128, 192, 64, (31, 1, 33)),             # around the 32-row tile, contraction shorter than the ring
    (320, 1024, 32, (63, 65)),               # around the 64-row tile
    (576, 448, 16, (70, 5)),
    (704, 2112, 16, (500, 131)),             # 128 x 64 forward, columns past the last full tile
    (2112, 320, 64, (129, 511)),             # 128 x 64 backward
    (576, 3072, 32, (150, 49)),              # 64 x 64 forward
    (3072, 576, 16, (199,)),                 # 64 x 64 backward
    (2112, 2112, 64, (127, 129, 521)),       # 64 x 128
    (320, 8192, 32, (385, 127)),             # 128 x 128 forward
    (320, 4160, 16, (1000,)),                # 128 x 256
    (1024, 4096, 16, (4396,)),               # 256 x 256 for 4096 rows, small tiles for the rest
    (832, 4160, 32, (3000, 1500)),           # the cut falls inside the second segment
    (2112, 4096, 16, (1088, 3072, 256, 64)), # uniform 256-row tiles (boundaries on 64 rows), then small tiles
    (320, 448, 32, (33, 0, 70, 1)),          # four adapters: the last count with the small adapter table
    (320, 448, 32, (33, 0, 70, 1, 64)),      # five: the full one
    (4096, 4096, 16, (2113,)),               # 192 x 256, last row tile of one row
    (2048, 4096, 16, (64, 1152, 832, 640, 256)),   # 192 x 256 forward, several adapters in a tile
]


@pytest.mark.parametrize("K,N,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_small_tiles(K, N, r, lens):
    print(f"small tiles K={K} N={N} r={r} lens={lens}", flush=True)
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.25, seg_lens=lens, cfg=61)
    inp = workloads.make_inputs(L)
    auto = run_gpu(L, *inp)
    binding.lora_set_row_tile(256)
    try:
        large = run_gpu(L, *inp)
    finally:
        binding.lora_set_row_tile(0)
    for name in ("Y", "S", "dX"):
        assert torch.equal(auto[name], large[name]), name
    compare(auto, run_oracle(L, *inp), label=f"small tiles {K} {N} {r} {lens}")
