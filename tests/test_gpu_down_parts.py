"""(1) in workgroups of eight rows and of a part of the rank's columns: on both sides of the lines between them (asked of the library), rows and stages that are not
whole, adapters of lower rank whose padding holds NaN; S' bit for bit against 32-row workgroups, and against the oracle."""
import pytest
import torch

import oracle
from gpu_util import TOL, f64, launch_names, rel_err
from paper_2510_00206_amd import binding, workloads

pytestmark = pytest.mark.gpu

# (K, r, segments): rows of a workgroup / workgroups that share the rank
CASES = {
    (1024, 16, (2048,)): "8", (832, 16, (2049,)): "16", (384, 16, (1, 9, 15)): "8", (320, 16, (2048,)): "16 direct",
    (576, 32, (1024,)): "8/2", (576, 32, (1025,)): "8", (832, 32, (2049,)): "16",
    (576, 64, (512,)): "8/4", (576, 64, (513,)): "8/2", (1088, 64, (1025,)): "16/2", (1088, 64, (2049,)): "16",
    (448, 64, (7, 0, 8, 17, 33)): "8/4", (1024, 64, (700, 331, 500)): "16/2", (320 + 64, 32, (300, 5, 0, 41)): "8/2",
}


@pytest.mark.parametrize("K,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_same_bits(K, r, lens):
    L = workloads.custom_layer(sum(lens), K, 64, r, 1.5, 0.1, seg_lens=lens, cfg=75)
    print(f"(1) in parts {L}", flush=True)
    assert launch_names(K, 64, r, lens)[0] == CASES[K, r, lens]
    X, W, A, B, _ = (t.cuda() for t in workloads.make_inputs(L))
    G, o = L.G, L.seg_offsets
    A, B = A.reshape(G, r, K).clone(), B.reshape(G, 64, r).clone()
    ranks = [(16, r, 32 if r == 64 else r)[g % 3] if G > 1 else r for g in range(G)]
    for g, q in enumerate(ranks):
        A[g, q:], B[g, :, q:] = float("nan"), float("nan")
    s, p = [1.5] * G, [(0.1, 0.0, 0.5)[g % 3] for g in range(G)]

    def run():
        return binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds, ranks=ranks)

    Y, S = run()
    binding.lora_set_row_tile(256)
    try:
        Y0, S0 = run()
    finally:
        binding.lora_set_row_tile(0)
    assert torch.equal(S.view(torch.int16), S0.view(torch.int16)) and torch.equal(Y.view(torch.int16), Y0.view(torch.int16))
    for g, q in enumerate(ranks):
        seg = slice(o[g], o[g + 1])
        assert not S[seg, q:].any()
        if o[g] < o[g + 1]:
            Sg = oracle.lora_fwd(f64(X[seg]), f64(W), f64(A[g, :q]), f64(B[g, :, :q]), s[g], p[g], L.seeds[g])[1]
            assert rel_err(S[seg, :q], s[g] * Sg) <= TOL
