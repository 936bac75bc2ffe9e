"""Operations (1) and (4) at the edges of their tilings: rows around the 16- and 32-row blocks and the 256 rows that the
waves of a workgroup walk together, contractions that end inside a 256-column stage, empty segments, ranks below the
allocated one, no dropout, gradients written by the kernel itself, through pieces and through partial planes, accumulation."""
import pytest
import torch

import oracle
from paper_2510_00206_amd import binding, workloads
from gpu_util import TOL, compare, f64, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# K (64 columns: one strip, a quarter of a stage), N, r, p, segments
CASES = [
    (64, 64, 16, 0.5, (1, 15, 16, 17)),
    (192, 128, 32, 0.1, (31, 33, 0, 32)),
    (320, 192, 64, 0.0, (255, 257)),
    (832, 64, 16, 0.25, (2305,)),
    (1088, 128, 64, 0.1, (289, 0, 64)),
    (4160, 64, 32, 0.1, (48, 5)),
]


@pytest.mark.parametrize("K,N,r,p,lens", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_down_projection_and_da(K, N, r, p, lens):
    print(f"(1) and (4) K={K} N={N} r={r} p={p} lens={lens}", flush=True)
    L = workloads.custom_layer(sum(lens), K, N, r, 1.5, p, seg_lens=lens, cfg=71)
    inp = workloads.make_inputs(L)
    auto = run_gpu(L, *inp)
    compare(auto, run_oracle(L, *inp), label=f"(1) (4) {K} {N} {r} {p} {lens}")
    binding.lora_set_row_tile(256)                 # 32-row workgroups in (1), panels of 256 rows and more and partial planes in (4)
    try:
        planes = run_gpu(L, *inp)
    finally:
        binding.lora_set_row_tile(0)
    assert torch.equal(auto["S"], planes["S"])     # same order of summation in (1)
    # (4): fp32 sums of the same products in another order; 1e-5 of the largest element as in test_kernel_heights_agree
    assert rel_err(auto["dA"], f64(planes["dA"])) <= 1e-5


# K, r, rows of the long segment: (1) loads fragments straight into registers for short contractions, the shorter the fewer
# rows there are, and goes through LDS otherwise; the batch and its short segments by themselves lie on both sides of that rule
MIXED_ROUTES = [(320, 16, 700), (384, 64, 700), (512, 16, 8200), (512, 64, 8200), (448, 32, 8200), (576, 32, 8200), (768, 32, 16400),
                (704, 16, 16400), (1024, 32, 8200)]


@pytest.mark.parametrize("K,r,rows", MIXED_ROUTES, ids=lambda v: str(v))
def test_down_projection_same_bits_by_every_route(K, r, rows):
    L = workloads.custom_layer(rows + 373, K, 64, r, 1.5, 0.1, seg_lens=(rows, 40, 333), cfg=73)
    print(f"(1) by every route {L}", flush=True)
    inp = workloads.make_inputs(L)
    X, W, A, B, _ = (t.cuda() for t in inp)
    s, p, o = [L.s] * L.G, [0.1, 0.0, 0.5], L.seg_offsets
    _, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds)
    one = [binding.lora_fwd(X[o[g]:o[g + 1]], W, A[g], B[g], s[g], p[g], L.seeds[g])[1] for g in range(L.G)]
    by_height = []
    try:
        for height in (128, 256):
            binding.lora_set_row_tile(height)
            by_height.append(binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds)[1])
    finally:
        binding.lora_set_row_tile(0)
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(one), S) and all(torch.equal(h, S) for h in by_height)
    for g in range(L.G):
        Sg = oracle.lora_fwd(f64(inp[0][o[g]:o[g + 1]]), f64(inp[1]), f64(inp[2][g]), f64(inp[3][g]), s[g], p[g], L.seeds[g])[1]
        assert rel_err(S[o[g]:o[g + 1]], s[g] * Sg) <= TOL


@pytest.mark.parametrize("rows,lens,added", [(0, (300, 0, 400), 0), (256, (300, 0, 400), 1), (256, (48, 5), 0)], ids=["whole", "counters", "planes"])
def test_da_accumulates(rows, lens, added):
    """accumulate adds to what dA holds; an empty segment's gradient stays untouched.  "planes": no room for counters, finalize launch."""
    L = workloads.custom_layer(sum(lens), 192, 128, 16, 1.0, 0.1, seg_lens=lens, cfg=72)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    s, p = [L.s] * L.G, [L.p] * L.G
    print(f"accumulate rows={rows}", flush=True)
    binding.lora_set_row_tile(rows)
    try:
        plan = binding.lora_debug_bwd_plan(L.K, L.N, L.r, L.seg_offsets)
        assert (plan.panel_rows_da, plan.added_in_strips) == (rows, added)
        _, S = binding.multi_lora_fwd(X, W, A, B, L.seg_offsets, s, p, L.seeds)
        args = (X, W, A, B, S, dY, L.seg_offsets, s, p, L.seeds)
        _, dA, _ = binding.multi_lora_bwd(*args)
        base = torch.randn(L.G, L.r, L.K, device="cuda")
        got = base.clone()
        binding.multi_lora_bwd(*args, dA=got, dB=torch.zeros(L.G, L.N, L.r, device="cuda"), accumulate=True)
        torch.cuda.synchronize()
    finally:
        binding.lora_set_row_tile(0)
    assert torch.equal(got, base + dA)
    for g in range(L.G):
        if lens[g] == 0:
            assert torch.equal(got[g], base[g]) and not dA[g].any()


@pytest.mark.parametrize("M,K,bound", [(4096, 20480, 1.1e-7), (8192, 26496, 1.4e-7)])
def test_da_rounding_error(M, K, bound):
    """fp32 error of dA's sum over the rows.  B picks the first r columns of dY, so dS is dY[:, :r] exactly (s = 1, no dropout) and the
    64-bit result has the same bf16 factors.  Bounds: between the error of the panels that plan_da states (0.92e-7, 0.99e-7) and
    that of whole segments (1.34e-7, 1.90e-7), whose waves chain four and eight times the MFMAs on a sum."""
    r, N = 16, 64
    print(f"rounding error of dA {M} x {K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    X = torch.randn((M, K), generator=gen, device="cuda").bfloat16()
    dY = torch.randn((M, N), generator=gen, device="cuda").bfloat16()
    W, A = torch.zeros((N, K), dtype=torch.bfloat16, device="cuda"), torch.zeros((r, K), dtype=torch.bfloat16, device="cuda")
    B = torch.eye(N, r, device="cuda").bfloat16()
    S = torch.zeros((M, r), dtype=torch.bfloat16, device="cuda")
    dA = binding.lora_bwd(X, W, A, B, S, dY, 1.0, 0.0, 1, need_dx=False)[1]
    want = torch.cat([dY[:, :r].double().t() @ X[:, k:k + 4096].double() for k in range(0, K, 4096)], dim=1)
    err = float((dA.double() - want).norm() / want.norm())
    print(f"{err:.3e}", flush=True)
    assert err <= bound


# rows of the first segment, K: its panels, on both sides of the rule's 12 (r = 16 and 32) and 3 (r = 64)
PIECES = {(3072, 4096): 3, (4352, 8192): 4, (6144, 1024): 12, (3328, 1024): 13, (4096, 512): 16}


@pytest.mark.parametrize("rows,K", list(PIECES), ids=str)
def test_pieces_added_either_way(rows, K):
    """The sum over the panels by the last workgroup of a strip and by the finalize launch: an adapter of rank 16 has the same dA
    whichever rank the call allocates, and with it whichever way the call takes; gradients are added to under accumulate."""
    N, lens = 4160, (rows, 0, 40)                  # (N past the rule for dS by itself)
    L = workloads.custom_layer(sum(lens), K, N, 64, 1.0, 0.1, seg_lens=lens, cfg=74)
    print(f"pieces either way {L}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    new = lambda *shape: torch.randn(shape, generator=gen, device="cuda").mul_(0.05).bfloat16()
    X, W, A, B, dY, S = new(L.M, K), new(N, K), new(3, 64, K), new(3, N, 64), new(L.M, N), new(L.M, 64)
    s, p, o, out, launches = [L.s] * 3, [L.p] * 3, L.seg_offsets, [], []
    for r in (16, 32, 64):
        S[:, 16:] = 0
        args = (X, W, A[:, :r].contiguous(), B[:, :, :r].contiguous(), S[:, :r].contiguous(), dY, o, s, p, L.seeds)
        binding.profile_begin()
        dA = binding.multi_lora_bwd(*args, need_dx=False, ranks=[16] * 3)[1]
        launches.append(binding.profile_end()["finalize_da"][1])
        base = torch.randn_like(dA)
        got = base.clone()
        binding.multi_lora_bwd(*args, need_dx=False, ranks=[16] * 3, dA=got, dB=torch.zeros(3, N, r, device="cuda"), accumulate=True)
        torch.cuda.synchronize()
        assert torch.equal(got, base + dA) and not dA[:, 16:].any() and not dA[1].any()
        out.append(dA[:, :16])
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    assert launches == [int(PIECES[rows, K] > most) for most in (12, 12, 3)]
