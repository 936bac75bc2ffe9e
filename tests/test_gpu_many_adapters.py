"""Tables of more than four adapters, whose tiles a wave finds with a lane for every adapter: every segment's Y, S', dX are the bits of a
call with that adapter alone, with empty segments first, last and in rows, segments that end around the tile heights, and rows past
what one launch takes (two launches that share the rows)."""
import random

import pytest
import torch

from paper_2510_00206_amd import binding, workloads

pytestmark = pytest.mark.gpu

# K, N, r, adapters, longest segment (0: lengths around the tile heights)
CASES = [(64, 64, 16, 5, 40), (192, 320, 32, 16, 0), (384, 128, 64, 17, 90), (512, 1088, 16, 33, 0), (320, 64, 64, 64, 33), (1024, 192, 32, 64, 0),
         (4096, 1024, 16, 64, 30), (128, 4096, 16, 63, 300)]


@pytest.mark.parametrize("K,N,r,G,longest", CASES, ids=str)
def test_segments_as_single_calls(K, N, r, G, longest):
    rnd = random.Random(G * K)
    lens = [rnd.choice((0, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129)) if longest == 0 else rnd.randrange(longest) for _ in range(G)]
    lens[0] = lens[-1] = lens[G // 2] = lens[G // 2 - 1] = 0
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.1, seg_lens=lens, cfg=96)
    print(f"many adapters G={G} M={L.M} K={K} N={N} r={r}", flush=True)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    s, p, o = [L.s] * G, [rnd.choice((0.0, 0.1)) for _ in lens], L.seg_offsets
    Y, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds)
    dX, dA, dB = binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds)
    for g in range(G):
        a, b = o[g], o[g + 1]
        if a == b:
            assert not dA[g].any() and not dB[g].any()
            continue
        one = (X[a:b], W, A[g], B[g])
        Y1, S1 = binding.lora_fwd(*one, s[g], p[g], L.seeds[g])
        dX1, dA1, dB1 = binding.lora_bwd(*one, S1, dY[a:b], s[g], p[g], L.seeds[g])
        assert torch.equal(Y1, Y[a:b]) and torch.equal(S1, S[a:b]) and torch.equal(dX1, dX[a:b]), g
        for got, want in ((dA[g], dA1), (dB[g], dB1)):       # fp32 sums over panels of other heights: as in test_kernel_heights_agree
            assert (got - want).abs().max() <= 1e-5 * want.abs().max(), g
