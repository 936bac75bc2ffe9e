"""(5) on 32 x 64 and 64 x 64 tiles with the strips of (4) and dB in its launch, against the same sums in launches of their own (a call
without dX, and the large heights fixed): at one tile, at remainders of tiles and strips, with empty segments, several panels, and on
both sides of what one launch takes."""
import pytest
import torch

from paper_2510_00206_amd import binding, workloads

pytestmark = pytest.mark.gpu

# K, N, r, segments (ranks: alternating where there are several)
CASES = [
    (64, 64, 16, (1,)),
    (1024, 1024, 16, (256,)),
    (320, 512, 32, (2500,)),                       # two panels and a remainder, counters
    (192, 4160, 16, (200,)),                       # (3) in one pass: no dB job
    (256, 320, 32, (33, 0, 31, 64)),
    (1024, 192, 16, (700, 0, 500)),                # (5) on 128 x 64 tiles: launches of their own
    (320, 512, 32, (2000, 0, 600)),                # panels of several segments, an empty one
    (320, 512, 16, (1300, 0, 90, 1200)),
    (256, 512, 32, (1100, 40, 0, 600, 33, 513)),   # ... and the full adapter table
    (8192, 64, 16, (64,)),                         # 256 tiles and 129 strips
    (16384, 64, 16, (64,)),                        # more than two workgroups to a compute unit: launches of their own
]
OWN_LAUNCHES = [(1024, 192, 16, (700, 0, 500)), (16384, 64, 16, (64,))]


@pytest.mark.parametrize("K,N,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_same_bits(K, N, r, lens):
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.1, seg_lens=lens, cfg=93)
    print(f"dX with strips {L}", flush=True)
    plan = binding.lora_debug_bwd_plan(K, N, r, L.seg_offsets)
    assert plan.with_dx == ((K, N, r, lens) not in OWN_LAUNCHES)
    assert sum(lens) < 2000 or (plan.panel_rows_db >= 512, plan.panel_rows_da, plan.added_in_strips) == (True, 512, 1)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    s, p, o = [L.s] * L.G, [L.p] * L.G, L.seg_offsets
    ranks = [(r, 16)[g % 2] for g in range(L.G)]
    if L.G == 1:
        A, B = A.reshape(1, L.r, K), B.reshape(1, N, L.r)
    fwd = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds, ranks=ranks)
    bwd = lambda **kw: binding.multi_lora_bwd(X, W, A, B, fwd[1], dY, o, s, p, L.seeds, ranks=ranks, **kw)
    binding.profile_begin()
    dX, dA, dB = bwd()
    assert binding.profile_end()["da"][1] == int(not plan.with_dx)
    _, dA2, dB2 = bwd(need_dx=False)
    base = [torch.randn_like(dA), torch.randn_like(dB)]
    got = [t.clone() for t in base]
    dX3 = bwd(dA=got[0], dB=got[1], accumulate=True)[0]
    binding.lora_set_row_tile(256)
    try:
        dX4 = bwd()[0]
    finally:
        binding.lora_set_row_tile(0)
    torch.cuda.synchronize()
    assert torch.equal(dA, dA2) and torch.equal(dB, dB2)
    assert torch.equal(dX, dX3) and torch.equal(dX, dX4)
    assert torch.equal(got[0], base[0] + dA) and torch.equal(got[1], base[1] + dB)
