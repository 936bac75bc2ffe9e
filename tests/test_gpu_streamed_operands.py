"""(2) and (5) where both operands together outgrow the memory-side cache (256 MiB): the large tiles that ask for lines ahead of
their copies, bit for bit against 128 x 256 tiles, which do not.  Ragged rows and columns, 256- and 192-row tiles, tiles of several
adapters, remainders in a second launch, and contractions of hardly more slabs than are in flight."""
import pytest
import torch

from gpu_util import launch_names
from paper_2510_00206_amd import binding

pytestmark = pytest.mark.gpu

# (K, N, r, segments): what (2) and (5) run as; +: lines are asked for ahead
CASES = {
    (28672, 4096, 16, (2999,)): ("192x256x64:4+", "192x256x64:4"),                      # 192-row tiles
    (4096, 28672, 32, (2999,)): ("192x256x64:4", "192x256x64:4+"),
    (14336, 12352, 16, (4001,)): ("256x256x64:4+ and 128x128x64:8", "192x256x64:4+"),   # (2): a second launch; a last column tile of 64
    (8192, 16384, 64, (1088, 1984, 1024)): ("256x256x64:4+", "256x256x64:4+"),          # tiles of two adapters
    (20480, 4160, 16, (6900, 13)): ("256x256x64:4+", "256x256x64:4"),                   # boundaries off every grid
    (256, 192, 16, (700037,)): ("256x256x64:4", "256x256x64:4+"),                       # three slabs, two of them in flight before the loop
    (320, 64, 16, (1100037,)): ("128x64x64:7", "256x256x64:4"),                         # (5): one slab
}


@pytest.mark.parametrize("K,N,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_same_bits_as_small_tiles(K, N, r, lens):
    M, G = sum(lens), len(lens)
    print(f"streamed operands {K} {N} {r} {lens}", flush=True)
    assert launch_names(K, N, r, lens)[1:3] == CASES[K, N, r, lens]
    o = [sum(lens[:g]) for g in range(G + 1)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    draw = lambda *shape, std=1.0: torch.randn(shape, generator=gen, device="cuda").mul_(std).to(torch.bfloat16)
    X, W, A, B, dY = draw(M, K), draw(N, K, std=K ** -0.5), draw(G, r, K, std=K ** -0.5), draw(G, N, r, std=0.02), draw(M, N)
    s, p, seeds = [1.5] * G, [0.1] * G, list(range(5, 5 + G))

    def run():
        Y, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, seeds)
        dX, _, _ = binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, seeds)
        return Y, S, dX

    got = run()
    binding.lora_set_row_tile(128)
    try:
        want = run()
    finally:
        binding.lora_set_row_tile(0)
    for name, a, b in zip(("Y", "S", "dX"), got, want):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), name
