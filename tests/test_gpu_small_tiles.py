"""The small-tile GEMM kernels, the 192-row large tiles and the split of a launch between two kernels, at sizes on the
edges of their tiles: every output against the oracle, and Y, S' and dX bit for bit against the 256 x 256 tiles (the
contraction is walked in the same order by every kernel, so the tolerance between them is zero)."""
import pytest
import torch

from paper_2510_00206_amd import binding, workloads
from gpu_util import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# (K, N, r, segments): tiles of operation (2), tiles of operation (5).  Which tiles a GEMM takes follows from the sizes alone
# (tests/test_launch_plan.py holds the library to what stands here): "128x64" one launch, "256x256+64x64@4096" two, the second
# from row 4096 on.
PLANS = {
    (64, 64, 16, (1,)): ("32x64", "32x64"),                       # one row, one slab, one column block
    (128, 192, 64, (31, 1, 33)): ("32x64", "32x64"),              # around the 32-row tile, contraction shorter than the ring
    (320, 1024, 32, (63, 65)): ("32x64", "32x64"),
    (576, 448, 16, (70, 5)): ("32x64", "32x64"),
    (704, 2112, 16, (500, 131)): ("128x64", "32x64"),             # columns past the last full tile
    (2112, 320, 64, (129, 511)): ("32x64", "128x64"),
    (576, 3072, 32, (150, 49)): ("64x64", "32x64"),
    (3072, 576, 16, (199,)): ("32x64", "64x64"),
    (2112, 2112, 64, (127, 129, 521)): ("64x128", "64x128"),
    (2112, 2112, 64, (1000,)): ("128x128", "128x128"),
    (320, 4160, 32, (134, 286)): ("128x128", "32x64"),            # ragged segments around two tiles, contraction of five slabs
    (4160, 320, 16, (466,)): ("32x64", "128x128"),
    (320, 8192, 32, (385, 127)): ("128x256", "32x64"),
    (320, 4160, 16, (1000,)): ("128x256", "32x64"),
    (2112, 320, 64, (1948,)): ("64x64", "128x256"),
    (1024, 4096, 16, (4396,)): ("256x256+128x64@4096", "128x128+32x64@4096"),
    (1024, 4096, 64, (4700,)): ("192x256", "128x128+64x64@4096"),
    (1280, 2112, 16, (8208,)): ("256x256+128x128@7168", "192x256"),
    (2368, 2048, 32, (7238,)): ("256x256", "256x256+128x128@6400"),
    (832, 4160, 32, (3000, 1500)): ("192x256", "128x128"),        # ragged boundary between 192-row tiles
    (704, 4160, 32, (1983, 108, 289, 1427)): ("256x256+64x128@3404", "128x128"),   # the cut falls inside the last segment, off the 64-row grid
    (2112, 704, 64, (2253, 1382, 1029, 921, 639, 1208)): ("128x256", "256x256+64x128@6480"),   # ... the same backward
    (2112, 4096, 16, (1088, 3072, 256, 64)): ("256x256+128x64@4096", "192x256"),   # boundaries on 64 rows: uniform large tiles
    (320, 448, 32, (33, 0, 70, 1)): ("32x64", "32x64"),           # four adapters: the last count with the small adapter table
    (320, 448, 32, (33, 0, 70, 1, 64)): ("32x64", "32x64"),       # five: the full one
    (4096, 4096, 16, (2113,)): ("192x256", "192x256"),            # last row tile of one row
    (2048, 4096, 16, (64, 1152, 832, 640, 256)): ("192x256", "128x256"),          # several adapters in a 192-row tile
    (576, 320, 32, (2112, 2112, 1920, 1152, 1664, 2048)): ("128x64", "192x256"),  # ... backward
}
CASES = list(PLANS)


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


# The same, for one diverged adapter (index) in a packed batch and padding of A and B that holds NaN; ranks per adapter.
POISON_PLANS = {
    (320, 320, 32, (320, 128, 1216), (32, 16, 16), 1): ("64x64", "64x64"),
    (320, 832, 64, (128, 640, 512), (16, 64, 32), 1): ("128x64", "32x64"),
    (832, 320, 64, (640, 640), (32, 64), 0): ("32x64", "128x64"),
    (320, 1024, 64, (64, 576, 64, 1216), (32, 16, 64, 16), 2): ("64x128", "64x64"),
    (2112, 320, 32, (34, 828), (16, 32), 0): ("32x64", "64x128"),
    (320, 576, 32, (640, 832, 2176), (16, 32, 16), 2): ("128x128", "128x64"),
    (704, 320, 64, (459, 2258, 131), (64, 32, 16), 0): ("64x64", "128x128"),
    (320, 1088, 32, (1536, 1728, 1728, 896, 64, 448), (16, 32, 16, 16, 32, 16), 4): ("192x256", "64x64"),
    (576, 320, 64, (2112, 2112, 1920, 1152, 1664, 2048), (16, 32, 64, 16, 32, 64), 3): ("128x64", "192x256"),
    (704, 4160, 32, (1983, 108, 289, 1427), (16, 32, 32, 16), 1): ("256x256+64x128@3404", "128x128"),
    (2112, 704, 64, (2253, 1382, 1029, 921, 639, 1208), (16, 64, 32, 16, 64, 32), 4): ("128x256", "256x256+64x128@6480"),
}


@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("case", list(POISON_PLANS), ids=lambda c: "x".join(map(str, c[:3])))
def test_diverged_adapter_and_padding_stay_where_they_are(case, value):
    """Every other segment has the bits of the call in which the adapter is sound and the padding zero (same packing, so the
    same launches), and the diverged one's own padding of S', dA and dB is zero."""
    K, N, r, lens, ranks, bad = case
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.25, seg_lens=lens, cfg=62)
    print(f"poison {L} ranks={ranks} adapter={bad} value={value}", flush=True)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    s, p, o = [0.5 + g for g in range(L.G)], [0.05 * (g + 1) for g in range(L.G)], L.seg_offsets

    def run(A, B):
        Y, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds, ranks=ranks)
        return (Y, S) + tuple(binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, ranks=ranks))

    for g, rg in enumerate(ranks):
        A[g, rg:], B[g, :, rg:] = 0, 0
    clean = run(A, B)
    for g, rg in enumerate(ranks):
        A[g, rg:], B[g, :, rg:] = float("nan"), float("nan")
    A[bad, ::2], A[bad, 1::2], B[bad, ::2], B[bad, 1::2] = value, -value, -value, value
    Y, S, dX, dA, dB = got = run(A, B)
    torch.cuda.synchronize()
    assert not torch.isfinite(Y[o[bad]:o[bad + 1]]).all() and not torch.isfinite(dX[o[bad]:o[bad + 1]]).all()
    for g, rg in enumerate(ranks):
        sl = slice(o[g], o[g + 1])
        assert not S[sl, rg:].any() and not dA[g, rg:].any() and not dB[g, :, rg:].any(), g
        if g != bad:
            for name, a, b in zip(("Y", "S", "dX"), got, clean):
                assert torch.equal(a[sl], b[sl]) and torch.isfinite(a[sl]).all(), (g, name)
            assert torch.equal(dA[g], clean[3][g]) and torch.equal(dB[g], clean[4][g]), g


@pytest.mark.parametrize("N", [4032, 4096, 4160])
@pytest.mark.parametrize("lens", [(1,), (33, 0, 31, 65)], ids=str)
def test_wave_splits_of_32_row_tiles(N, lens):
    """(5) over contractions on both sides of the one from which more waves share a 32 x 64 tile, with no strips in its launch (rank 64);
    (2) the other way round; the frozen products."""
    K = 320
    print(f"wave splits {K} {N} {lens}", flush=True)
    for k, n in ((K, N), (N, K)):
        L = workloads.custom_layer(sum(lens), k, n, 64, 1.5, 0.25, seg_lens=lens, cfg=63)
        inp = workloads.make_inputs(L)
        X, W, dY = inp[0].cuda(), inp[1].cuda(), inp[4].cuda()
        out = []
        try:
            for rows in (0, 256):
                binding.lora_set_row_tile(rows)
                out.append(dict(run_gpu(L, *inp), F=binding.frozen_fwd(X, W), D=binding.frozen_bwd(dY, W)))
        finally:
            binding.lora_set_row_tile(0)
        assert binding.lora_debug_gemm_tiles(N, K, 64, L.seg_offsets) == [(32, 64, 0)]
        for name in ("Y", "S", "dX", "F", "D"):
            assert torch.equal(out[0][name], out[1][name]), (k, n, name)
        compare({k: v for k, v in out[0].items() if k not in "FD"}, run_oracle(L, *inp), label=f"wave splits {k} {n} {lens}")
