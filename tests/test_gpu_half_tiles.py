"""32 x 64 tiles shared by two workgroups, and 128-deep stages: contractions that end in half a stage or fill less than the ring, row and
column remainders, both sides of the line from which a tile is not shared, with the strips of (4) in the launch and without; Y and dX bit for bit
against the 256 x 256 tiles, and every output against the oracle."""
import pytest
import torch

from gpu_util import compare, run_gpu, run_oracle
from paper_2510_00206_amd import binding, workloads

pytestmark = pytest.mark.gpu

# K, N, r, segments
CASES = [
    (64, 128, 16, (1,)),                    # half a stage and a whole one
    (192, 64, 64, (33,)),                   # three slabs and one; no strips in the launch
    (576, 704, 32, (31, 0, 34, 1)),
    (1024, 1024, 16, (256,)),               # 128 tiles: all shared, but not beside the strips
    (1024, 1088, 16, (250,)),               # 136 tiles (2): none shared
    (2048, 1984, 32, (127,)),               # 124 and 128 tiles; beside the strips, contraction just below 2048
    (1984, 2048, 32, (127,)),               # ... and from there on
    (4032, 4096, 16, (50,)),                # 128 tiles (2) of a contraction of 63 slabs
    (4160, 4160, 16, (50,)),                # 130: whole tiles of (2) over a long contraction
    (320, 64, 32, (40, 7, 64, 1, 33)),      # the full adapter table
]


@pytest.mark.parametrize("K,N,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_half_tiles(K, N, r, lens):
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.1, seg_lens=lens, cfg=71)
    print(f"half tiles {L}", flush=True)
    assert binding.lora_debug_gemm_tiles(K, N, r, L.seg_offsets)[0][:2] == (32, 64)
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
