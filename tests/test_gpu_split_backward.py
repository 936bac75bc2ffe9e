"""Operation (3) in its two forms: dS by itself with dB as further strips beside (4) (batches of up to 6144 rows, N <= 4096), and one
pass over dY with partial sums (the large heights fixed).  Sizes at the edges of the 16-row workgroups, the 256- and 512-column
stages, the 64-column strips and the panels whose sums meet in the last workgroup of a strip."""
import pytest
import torch

from paper_2510_00206_amd import binding, workloads
from gpu_util import compare, f64, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# K, N, r, segments
CASES = [
    (64, 64, 16, (1,)),
    (128, 320, 64, (15, 16, 17)),
    (192, 512, 32, (33, 0, 31)),
    (64, 576, 16, (100, 64)),
    (128, 832, 64, (48, 5)),
    (64, 4096, 64, (40,)),
    (64, 4160, 16, (40,)),                         # past the rule: the same route both times
    (192, 1088, 16, (2600, 0, 700)),               # panels of 512 rows with a remainder, an empty segment, a segment of one panel
    (320, 576, 64, (1536, 1024)),                  # whole panels
    (64, 64, 32, (6143,)),
    (64, 64, 32, (6145,)),
    # dS by four, two and one workgroups to 16 rows: 64 and 65, 128 and 129 groups of 16 rows
    (64, 832, 64, (1024,)),
    (64, 832, 64, (1000, 0, 17)),
    (64, 576, 64, (2048,)),
    (64, 576, 64, (2040, 9)),
    (128, 576, 32, (2048,)),
    (128, 576, 32, (2049,)),
]


@pytest.mark.parametrize("K,N,r,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_both_forms(K, N, r, lens):
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, 0.1, seg_lens=lens, cfg=91)
    print(f"both forms of (3) {L}", flush=True)
    inp = workloads.make_inputs(L)
    auto = run_gpu(L, *inp)
    compare(auto, run_oracle(L, *inp), label=f"(3) {K} {N} {r} {lens}")
    binding.lora_set_row_tile(256)
    try:
        one_pass = run_gpu(L, *inp)
    finally:
        binding.lora_set_row_tile(0)
    assert torch.equal(auto["dX"], one_pass["dX"])         # dS is the same bits, and with it dX
    for name in ("dA", "dB"):                              # fp32 sums of the same products in another order: as in test_kernel_heights_agree
        assert rel_err(auto[name], f64(one_pass[name])) <= 1e-5


@pytest.mark.parametrize("lens,ranks", [((2600, 0, 700), (64, 16, 32)), ((300, 20), (16, 64))], ids=["panels", "whole"])
def test_counters_ranks_and_accumulation(lens, ranks):
    """Whatever the workspace holds, two calls give the same bits; accumulate adds those; padding and empty segments are zeros."""
    L = workloads.custom_layer(sum(lens), 192, 320, 64, 1.0, 0.1, seg_lens=lens, cfg=92)
    print(f"counters {L}", flush=True)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    s, p, o = [L.s] * L.G, [L.p] * L.G, L.seg_offsets
    _, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds, ranks=ranks)
    ws = binding.alloc_workspace(L.M, L.K, L.N, L.r, L.G)
    outs = []
    for fill in (0, 255):
        ws.fill_(fill)
        outs.append(binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, workspace=ws, ranks=ranks))
    base = [torch.randn_like(t) for t in outs[0][1:]]
    got = [t.clone() for t in base]
    ws.fill_(170)
    binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, need_dx=False, dA=got[0], dB=got[1], accumulate=True, workspace=ws, ranks=ranks)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    assert all(torch.equal(g, b + t) for g, b, t in zip(got, base, outs[0][1:]))
    for g in range(L.G):
        assert not outs[0][1][g, ranks[g]:].any() and not outs[0][2][g, :, ranks[g]:].any()
        if o[g] == o[g + 1]:
            assert not outs[0][1][g].any() and not outs[0][2][g].any()


@pytest.mark.parametrize("r,ranks", [(64, (16, 64, 32)), (32, (16, 32, 16))])
def test_rank_parts_of_ds(r, ranks):
    """Adapters below the call's rank where several workgroups share the columns of 16 rows: dX, dA and dB are those of the one-pass
    form, and padding that holds non-finite values is not used."""
    lens = (33, 100, 16)
    L = workloads.custom_layer(sum(lens), 128, 1088, r, 1.0, 0.1, seg_lens=lens, cfg=94)
    print(f"rank parts {L} {ranks}", flush=True)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    for g, q in enumerate(ranks):
        A[g, q:], B[g, :, q:] = float("nan"), float("inf")
    s, p, o = [L.s] * L.G, [L.p] * L.G, L.seg_offsets
    _, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds, ranks=ranks)
    out = []
    try:
        for rows in (0, 256):
            binding.lora_set_row_tile(rows)
            out.append(binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, ranks=ranks))
    finally:
        binding.lora_set_row_tile(0)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0]) and torch.isfinite(out[0][0].float()).all()
    for a, b in zip(out[0][1:], out[1][1:]):           # (fp32 sums in another order, as above)
        assert rel_err(a, f64(b)) <= 1e-5


# K, N, segments: whether dS goes by itself.  One round of its 16-row groups (256), or short sweeps (M N up to 7 Mi), up to 6144 rows
ROUTES = [(64, 4096, (4096,), True), (64, 4096, (4097,), False), (64, 4096, (2049, 2040), False), (64, 1152, (6144,), True),
          (64, 1216, (6144,), False), (64, 64, (6144,), True), (64, 64, (6145,), False), (64, 4160, (64,), False), (4096, 64, (6144,), True),
          (4160, 64, (6144,), False)]


@pytest.mark.parametrize("K,N,lens,alone", ROUTES, ids=str)
def test_which_form(K, N, lens, alone):
    L = workloads.custom_layer(sum(lens), K, N, 16, 1.5, 0.1, seg_lens=lens, cfg=95)
    print(f"form of (3) {L}", flush=True)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    S = torch.randn((L.M, L.r), device="cuda").bfloat16()
    args = (X, W, A, B, S, dY, L.seg_offsets, [L.s] * L.G, [L.p] * L.G, L.seeds)
    out, finalized = [], []
    try:
        for rows in (0, 256):
            binding.lora_set_row_tile(rows)
            binding.profile_begin()
            out.append(binding.multi_lora_bwd(*args))
            finalized.append(binding.profile_end()["finalize_ds_db"][1])
    finally:
        binding.lora_set_row_tile(0)
    assert finalized == [int(not alone), 1]
    assert torch.equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1:], out[1][1:]):           # (fp32 sums in another order, as above)
        assert rel_err(a, f64(b)) <= 1e-5


@pytest.mark.parametrize("M", [1793, 2047])
def test_db_rounding_error(M):
    """fp32 error of dB's sum over the rows (dY and S' are its exact bf16 factors).  Bound: between that of the panels plan_db states
    (0.75e-7 to 0.78e-7) and that of one panel over the segment (0.93e-7 to 0.98e-7)."""
    K, N, r = 1024, 4096, 16
    print(f"rounding error of dB {M} rows", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    new = lambda *shape: torch.randn(shape, generator=gen, device="cuda").bfloat16()
    X, dY, A, B, S, W = new(M, K), new(M, N), new(r, K), new(N, r), new(M, r), torch.zeros((N, K), dtype=torch.bfloat16, device="cuda")
    dB = binding.lora_bwd(X, W, A, B, S, dY, 1.0, 0.0, 1, need_dx=False)[2]
    want = dY.double().t() @ S.double()
    assert float((dB.double() - want).norm() / want.norm()) <= 0.86e-7
