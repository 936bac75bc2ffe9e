"""32 x 64 tiles shared by two workgroups, and 128-deep stages: contractions that end in half a stage or fill less than the ring, row and
column remainders, both sides of the lines between the forms (asked of the library), with the strips of (4) in the launch and without; Y and dX bit for bit
against the 256 x 256 tiles, and every output against the oracle."""
import pytest
import torch

from gpu_util import compare, launch_names, run_gpu, run_oracle
from paper_2510_00206_amd import binding, workloads

pytestmark = pytest.mark.gpu

HALVES, ONE_SLAB = "32x32x128:8", "32x64x64:7"                          # (2) and (5); whole tiles of (2)
DEEP, NARROW, WIDE = "32x64x128:7", "32x64x64:4", "32x64x64:8"          # whole tiles of (5)

# (K, N, r, segments): what (2) and (5) run as, workgroups of (5) with the strips beside it
CASES = {
    (64, 128, 16, (1,)): (HALVES, HALVES, 5),                           # half a stage and a whole one
    (192, 64, 64, (33,)): (HALVES, HALVES, 12),                         # three slabs and one; no strips in the launch
    (576, 704, 32, (31, 0, 34, 1)): (HALVES, HALVES, 152),
    (1024, 1024, 16, (256,)): (HALVES, DEEP, 160),                      # 128 tiles: shared, but not beside the strips
    (1024, 1088, 16, (250,)): (ONE_SLAB, DEEP, 161),                    # 136 tiles (2)
    (2048, 1984, 32, (127,)): (HALVES, DEEP, 191),                      # 124 and 128 tiles; beside the strips, contraction just below 2048
    (1984, 2048, 32, (127,)): (HALVES, HALVES, 311),                    # ... and from there on
    (4032, 4096, 16, (50,)): (HALVES, HALVES, 379),                     # 128 tiles (2) of a contraction of 63 slabs
    (4160, 4160, 16, (50,)): (ONE_SLAB, DEEP, 195),                     # 130: whole tiles of (2) over a long contraction
    (4096, 4096, 16, (5, 91)): (ONE_SLAB, NARROW, 512),                 # ... and of (5) that share compute units with the strips
    (320, 64, 32, (40, 7, 64, 1, 33)): (HALVES, HALVES, 110),           # the full adapter table
    (2048, 4096, 32, (8, 8, 8, 8)): (ONE_SLAB, HALVES, 640),            # as many halves and strips as there can be
    (1024, 4096, 16, (20, 20, 20, 20, 20)): ("64x128x64:11", HALVES, 560),   # ... with the full adapter table
    # whole tiles of (5) by themselves: rows of W of a multiple of 512 bytes and others, contractions below and from 1024 and 4096 on
    (4096, 1024, 64, (97,)): (HALVES, DEEP, 256),
    (4096, 1088, 64, (70,)): (HALVES, DEEP, 192),                       # ... that end in half a stage
    (4096, 960, 64, (97,)): (HALVES, NARROW, 256),
    (4160, 1024, 64, (70,)): (HALVES, NARROW, 195),
    (4160, 4096, 64, (33, 8)): (ONE_SLAB, WIDE, 195),
    (4864, 576, 64, (3, 1, 5, 2, 4, 16, 15, 16)): (HALVES, NARROW, 608),   # in several rounds, hardly more slabs than stages
    (4096, 1024, 64, (1, 5, 7, 16, 3, 5, 2, 29, 9)): (ONE_SLAB, NARROW, 576),   # ... of a multiple, but more than run at once
    (320, 4160, 64, (70,)): (ONE_SLAB, HALVES, 30),                     # (2): fewer slabs than stages
    (384, 4160, 64, (70,)): (ONE_SLAB, HALVES, 36),                     # ... as many
    (512, 4160, 16, (70,)): (ONE_SLAB, HALVES, 56),
}


@pytest.mark.parametrize("K,N,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_half_tiles(K, N, r, lens):
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.1, seg_lens=lens, cfg=71)
    print(f"half tiles {L}", flush=True)
    assert launch_names(K, N, r, lens)[1:] == CASES[K, N, r, lens]
    inp = workloads.make_inputs(L)
    got = run_gpu(L, *inp)
    binding.lora_set_row_tile(256)
    try:
        want = run_gpu(L, *inp)
    finally:
        binding.lora_set_row_tile(0)
    for name in ("Y", "dX"):
        assert torch.equal(got[name].view(torch.int16), want[name].view(torch.int16)), name
    compare(got, run_oracle(L, *inp), label=f"half tiles {K} {N} {r} {lens}")
