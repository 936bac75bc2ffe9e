"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.
Mask: bit-exact.  Y, S_saved, dX, dA, dB: max|err|/max|ref| <= 2e-2 (bf16 in, fp32 accumulate)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_00206_amd import binding, workloads
from gpu_util import TOL, compare, f64, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True, params=[(256, 1), (128, 1), (256, 2), (128, 2)],
                ids=["tile256-ahead1", "tile128-ahead1", "tile256-ahead2", "tile128-ahead2"])
def _lib(request):
    """Every test of this module runs with the large and with the small height of the kernels that
    have two (GEMM tiles of 256 / 128 rows, down-projection workgroups of 32 / 16 rows) fixed: small
    shapes would otherwise all take the small one; and with the GEMMs' slab copies one and two slabs ahead
    (small weights would otherwise never take the second in operation (5); the 128-row tiles have one distance, so
    tile128-ahead2 runs the GEMMs of tile128-ahead1).  The automatic choices are what the full-size tests and
    test_gpu_small_tiles.py run."""
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.load_library()          # raises if the HIP library is not built: no fallback
    binding.lora_set_row_tile(request.param[0])
    binding.lora_set_slab_lookahead(request.param[1])
    yield
    binding.lora_set_row_tile(0)
    binding.lora_set_slab_lookahead(0)


@pytest.mark.parametrize("M,K,p,seed", [(256, 1024, 0.1, 0x25100206), (37, 130, 0.5, 0), (5, 7, 0.05, 1),
                                         (1000, 2050, 0.9, 0xFFFFFFFFFFFFFFFF), (64, 64, 0.0, 3)])
def test_mask_bit_exact(M, K, p, seed):
    print(f"mask M={M} K={K} p={p} seed={seed:#x}", flush=True)
    got = binding.lora_debug_mask(M, K, p, seed).cpu().numpy().astype(bool)
    ref = oracle.keep_mask(seed, M, K, oracle.dropout_threshold(p))
    assert np.array_equal(got, ref)


SHAPES = [  # M, K, N, r, s, p
    (256, 1024, 1024, 16, 2.0, 0.1),       # configuration 1
    (64, 64, 64, 16, 1.0, 0.1),            # one block everywhere
    (1, 64, 128, 16, 2.0, 0.5),            # a single token
    (300, 320, 448, 16, 2.0, 0.1),         # ragged row tile, column tiles of 64 and 192
    (777, 576, 832, 32, 0.5, 0.25),        # several row tiles with a ragged tail, r = 32
    (520, 1088, 640, 64, 0.5, 0.1),        # r = 64, more than one column chunk in the streaming kernels
    (1100, 256, 192, 16, 1.0, 0.9),        # heavy dropout; 1100 rows: regular row panels and a long last one
    (384, 512, 256, 32, 2.0, 0.99999),     # threshold clipped to 65535: one element in 65536 survives, q = 65536
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(v) for v in s[:4]))
@pytest.mark.parametrize("zero_w", [False, True], ids=["W", "W0"])
def test_single_adapter_parity(shape, zero_w):
    M, K, N, r, s, p = shape
    L = workloads.custom_layer(M, K, N, r, s, p, cfg=7)
    print(f"single {L} zero_w={zero_w}", flush=True)
    inp = workloads.make_inputs(L, zero_w=zero_w)
    gpu = run_gpu(L, *inp, single_api=True)
    compare(gpu, run_oracle(L, *inp), label=f"single {shape} W0={zero_w}")


def test_mask_is_read_back_bit_exact_through_dx_and_s():
    """With W = 0, dX != 0 exactly where the element is kept; with X = 1 and a one-hot A row the
    saved S' column is s*q*keep."""
    L = workloads.custom_layer(200, 192, 128, 16, 1.0, 0.5, cfg=6)
    X, W, A, B, dY = workloads.make_inputs(L, zero_w=True)
    print("mask through dX", flush=True)
    gpu = run_gpu(L, X, W, A, B, dY)
    keep = oracle.keep_mask(L.seeds[0], L.M, L.K, oracle.dropout_threshold(L.p))
    assert np.array_equal(f64(gpu["dX"]) != 0, keep)
    j = 77
    A1 = torch.zeros_like(A)
    A1[0, 0, j] = 1.0
    gpu = run_gpu(L, torch.ones_like(X), W, A1, B, dY)
    assert np.array_equal(f64(gpu["S"])[:, 0], np.where(keep[:, j], 2.0, 0.0))


def test_p0_b0_is_the_frozen_linear():
    """p = 0 and B = 0: Y = X W and dX = dY W^T - the plain products, and the same bits as the library's own
    frozen-linear GEMMs (the LoRA steps add exact zeros to the same accumulation order); dA = 0."""
    L = workloads.custom_layer(320, 256, 192, 16, 2.0, 0.0, cfg=5)
    X, W, A, B, dY = workloads.make_inputs(L)
    B = torch.zeros_like(B)
    print("p0 b0", flush=True)
    gpu = run_gpu(L, X, W, A, B, dY)
    assert rel_err(gpu["Y"], f64(X) @ f64(W).T) <= TOL / 4
    assert rel_err(gpu["dX"], f64(dY) @ f64(W)) <= TOL / 4
    assert not gpu["dA"].any()
    assert torch.equal(gpu["Y"], binding.frozen_fwd(X.cuda(), W.cuda()))
    assert torch.equal(gpu["dX"], binding.frozen_bwd(dY.cuda(), W.cuda()))


ISOLATION = [  # M, K, N, r, segment lengths (boundaries on 64: uniform tiles that hold several adapters), poisoned adapter
    (832, 256, 320, 16, (64, 64, 64, 64, 192, 0, 64, 320), 2),
    (704, 192, 448, 32, (64, 64, 64, 64, 128, 192, 128), 1),
    (576, 256, 256, 64, (64, 128, 64, 320), 1),
    (768, 320, 576, 64, (128, 64, 64, 256, 256), 3),
    (601, 320, 192, 32, (100, 37, 300, 164), 2),          # boundaries off the grid: per-segment tiles
]


@pytest.mark.parametrize("case", ISOLATION, ids=lambda c: "x".join(str(v) for v in c[:4]))
@pytest.mark.parametrize("poison", ["nan", "inf"])
def test_adapters_do_not_interfere_under_non_finite_values(case, poison):
    """One adapter of a packed batch has diverged: its A and B hold NaN (or +-Inf).  Every other
    segment's Y, S', dX, dA and dB must stay what its single-adapter call gives, bit for bit
    (Section 5.1, FusedMultiLoRA: independent jobs share the kernels without interference)."""
    M, K, N, r, lens, bad = case
    L = workloads.custom_layer(M, K, N, r, 2.0, 0.1, seg_lens=lens, cfg=14)
    print(f"isolation {L} poison={poison} adapter={bad}", flush=True)
    X, W, A, B, dY = workloads.make_inputs(L)
    A, B = A.clone(), B.clone()
    if poison == "nan":
        A[bad], B[bad] = float("nan"), float("nan")
    else:
        A[bad, ::2], A[bad, 1::2] = float("inf"), float("-inf")
        B[bad, ::2], B[bad, 1::2] = float("-inf"), float("inf")
    s = [0.5 + g for g in range(L.G)]
    p = [0.05 * (g + 1) for g in range(L.G)]
    dev = "cuda"
    Xg, Wg, Ag, Bg, dYg = (t.to(dev) for t in (X, W, A, B, dY))
    Y, S = binding.multi_lora_fwd(Xg, Wg, Ag, Bg, L.seg_offsets, s, p, L.seeds)
    dX, dA, dB = binding.multi_lora_bwd(Xg, Wg, Ag, Bg, S, dYg, L.seg_offsets, s, p, L.seeds)
    torch.cuda.synchronize()
    o = L.seg_offsets
    assert o[bad + 1] > o[bad]
    assert not torch.isfinite(Y[o[bad]:o[bad + 1]]).all()          # the poison is really there
    for g in range(L.G):
        if g == bad or o[g + 1] == o[g]:
            continue
        sl = slice(o[g], o[g + 1])
        Y1, S1 = binding.lora_fwd(Xg[sl].contiguous(), Wg, Ag[g].contiguous(), Bg[g].contiguous(), s[g], p[g], L.seeds[g])
        dX1, dA1, dB1 = binding.lora_bwd(Xg[sl].contiguous(), Wg, Ag[g].contiguous(), Bg[g].contiguous(), S1,
                                         dYg[sl].contiguous(), s[g], p[g], L.seeds[g])
        for name, one, packed in (("Y", Y1, Y[sl]), ("S", S1, S[sl]), ("dX", dX1, dX[sl]), ("dA", dA1, dA[g]), ("dB", dB1, dB[g])):
            assert torch.isfinite(packed).all(), (g, name)
            assert torch.equal(one, packed), (g, name)


MULTI = [  # M, K, N, r, segment lengths
    (768, 256, 320, 16, (256, 128, 384)),
    (640, 192, 256, 16, (64, 0, 320, 256)),            # an empty segment
    (601, 320, 192, 32, (100, 37, 300, 164)),          # boundaries off the 64 grid
    (1024, 512, 1088, 64, (128, 640, 256)),            # r = 64, row tiles with two adapters
    (832, 256, 320, 16, (64, 64, 64, 64, 192, 0, 64, 320)),   # four adapters inside one 256-row tile
    (704, 192, 448, 32, (64, 64, 64, 64, 128, 192, 128)),     # r = 32 x 4 adapters: the widest mixed LoRA step
    (576, 256, 256, 64, (64, 128, 64, 320)),           # r = 64 x 3 adapters in a tile: per-segment tiles instead
]


@pytest.mark.parametrize("case", MULTI, ids=lambda c: "x".join(str(v) for v in c[:4]))
def test_multi_adapter_parity(case):
    M, K, N, r, lens = case
    L = workloads.custom_layer(M, K, N, r, 2.0, 0.1, seg_lens=lens, cfg=4)
    print(f"multi {L}", flush=True)
    X, W, A, B, dY = workloads.make_inputs(L)
    # distinct per-adapter scale and dropout
    s = [0.5 + g for g in range(L.G)]
    p = [0.05 * (g + 1) for g in range(L.G)]
    dev = "cuda"
    Xg, Wg, Ag, Bg, dYg = (t.to(dev) for t in (X, W, A, B, dY))
    Y, S = binding.multi_lora_fwd(Xg, Wg, Ag, Bg, L.seg_offsets, s, p, L.seeds)
    dX, dA, dB = binding.multi_lora_bwd(Xg, Wg, Ag, Bg, S, dYg, L.seg_offsets, s, p, L.seeds)
    torch.cuda.synchronize()
    Yr, Sr = oracle.multi_lora_fwd(f64(X), f64(W), f64(A), f64(B), L.seg_offsets, s, p, L.seeds)
    dXr, dAr, dBr, _ = oracle.multi_lora_bwd(f64(X), f64(W), f64(A), f64(B), f64(dY), L.seg_offsets, s, p, L.seeds)
    o = L.seg_offsets
    for g in range(L.G):
        Sr[o[g]:o[g + 1]] *= float(np.float32(s[g]))
    compare(dict(Y=Y, S=S, dX=dX, dA=dA, dB=dB), dict(Y=Yr, S=Sr, dX=dXr, dA=dAr, dB=dBr), label=f"multi {case}")
    # per-adapter gradients are judged on their own scale too
    for g in range(L.G):
        if o[g + 1] > o[g]:
            assert rel_err(dA[g], dAr[g]) <= TOL and rel_err(dB[g], dBr[g]) <= TOL
        else:
            assert not dA[g].any() and not dB[g].any()
    # multi == per-segment single-adapter calls, bit for bit
    for g in range(L.G):
        if o[g + 1] == o[g]:
            continue
        sl = slice(o[g], o[g + 1])
        Y1, S1 = binding.lora_fwd(Xg[sl].contiguous(), Wg, Ag[g].contiguous(), Bg[g].contiguous(), s[g], p[g], L.seeds[g])
        dX1, dA1, dB1 = binding.lora_bwd(Xg[sl].contiguous(), Wg, Ag[g].contiguous(), Bg[g].contiguous(), S1,
                                         dYg[sl].contiguous(), s[g], p[g], L.seeds[g])
        assert torch.equal(Y1, Y[sl]) and torch.equal(S1, S[sl]) and torch.equal(dX1, dX[sl])
        assert torch.equal(dA1, dA[g]) and torch.equal(dB1, dB[g])


def test_accumulate_skip_dx_and_repeatability():
    L = workloads.custom_layer(384, 256, 256, 16, 2.0, 0.1, seg_lens=(128, 256), cfg=3)
    inp = workloads.make_inputs(L)
    print("accumulate / repeat", flush=True)
    a = run_gpu(L, *inp)
    b = run_gpu(L, *inp)
    for k in ("Y", "S", "dX", "dA", "dB"):
        assert torch.equal(a[k], b[k]), k                      # fixed-order reductions: bitwise repeatable
    dA0 = torch.full_like(a["dA"], 1.5)
    dB0 = torch.full_like(a["dB"], -2.0)
    c = run_gpu(L, *inp, need_dx=False, dA=dA0.clone(), dB=dB0.clone(), accumulate=True)
    assert c["dX"] is None
    assert torch.allclose(c["dA"], a["dA"] + 1.5, rtol=1e-6, atol=1e-6)
    assert torch.allclose(c["dB"], a["dB"] - 2.0, rtol=1e-6, atol=1e-6)


def test_error_paths_on_gpu():
    L = workloads.custom_layer(128, 128, 128, 16, cfg=2)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    with pytest.raises(binding.LoraError) as e:
        binding.lora_fwd(X, W, A[0].contiguous(), B[0].contiguous(), 1.0, 1.0, 1)
    assert e.value.status == 4
    with pytest.raises(binding.LoraError) as e:
        binding.multi_lora_fwd(X, W, A, B, [0, 64], [1.0], [0.1], [1])
    assert e.value.status == 5
    Y, S = binding.lora_fwd(X, W, A[0].contiguous(), B[0].contiguous(), 1.0, 0.1, 1)
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.LoraError) as e:
        binding.lora_bwd(X, W, A[0].contiguous(), B[0].contiguous(), S, dY, 1.0, 0.1, 1, workspace=small)
    assert e.value.status == 6
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape", [(256, 1024, 1024, 16, 2.0, 0.1), (777, 576, 832, 32, 0.5, 0.25),
                                   (520, 1088, 640, 64, 0.5, 0.1)], ids=lambda s: "x".join(str(v) for v in s[:4]))
def test_unfused_baseline_parity(shape):
    """The op-by-op baseline computes the same layer (its extra bf16 intermediates stay inside the bar)."""
    M, K, N, r, s, p = shape
    L = workloads.custom_layer(M, K, N, r, s, p, cfg=7)
    print(f"unfused {L}", flush=True)
    X, W, A, B, dY = workloads.make_inputs(L)
    Xg, Wg, Ag, Bg, dYg = (t.cuda() for t in (X, W, A[0].contiguous(), B[0].contiguous(), dY))
    ws = binding.unfused_workspace(M, K, N, r)
    Y = binding.lora_unfused_fwd(Xg, Wg, Ag, Bg, s, p, L.seeds[0], ws)
    dX, dA, dB = binding.lora_unfused_bwd(Wg, Ag, Bg, dYg, s, p, L.seeds[0], ws)
    torch.cuda.synchronize()
    ref = run_oracle(L, X, W, A, B, dY)
    compare(dict(Y=Y, dX=dX, dA=dA[None], dB=dB[None]), ref, label=f"unfused {shape}")


def test_frozen_linear_reference_line():
    """The frozen linear alone (the reference line of the LoRA-overhead sweep) is the plain products."""
    L = workloads.custom_layer(300, 320, 448, 16, cfg=5)
    X, W, A, B, dY = workloads.make_inputs(L)
    print("frozen linear", flush=True)
    Y = binding.frozen_fwd(X.cuda(), W.cuda())
    dX = binding.frozen_bwd(dY.cuda(), W.cuda())
    torch.cuda.synchronize()
    assert rel_err(Y, f64(X) @ f64(W).T) <= TOL / 4
    assert rel_err(dX, f64(dY) @ f64(W)) <= TOL / 4


def test_empty_batch_and_many_adapters():
    """M = 0 is a no-op forward and a zero-fill backward; 64 adapters (the table's capacity) with
    short uneven segments, several of them empty."""
    K, N, r = 128, 192, 16
    dev = "cuda"
    W = torch.randn(N, K, device=dev).to(torch.bfloat16)
    A = torch.randn(1, r, K, device=dev).to(torch.bfloat16)
    B = torch.randn(1, N, r, device=dev).to(torch.bfloat16)
    X0 = torch.empty((0, K), dtype=torch.bfloat16, device=dev)
    dY0 = torch.empty((0, N), dtype=torch.bfloat16, device=dev)
    print("M = 0", flush=True)
    Y, S = binding.multi_lora_fwd(X0, W, A, B, [0, 0], [1.0], [0.1], [1])
    assert Y.shape == (0, N)
    dA = torch.full((1, r, K), 7.0, device=dev)
    dB = torch.full((1, N, r), 7.0, device=dev)
    binding.multi_lora_bwd(X0, W, A, B, S, dY0, [0, 0], [1.0], [0.1], [1], dA=dA, dB=dB)
    torch.cuda.synchronize()
    assert not dA.any() and not dB.any()

    G = 64
    rng = np.random.default_rng(11)
    lens = [int(v) for v in rng.integers(0, 40, size=G)]
    lens[3] = lens[17] = 0
    L = workloads.custom_layer(sum(lens), 192, 128, 16, 2.0, 0.1, seg_lens=lens, cfg=1)
    print(f"G = 64, M = {L.M}", flush=True)
    inp = workloads.make_inputs(L)
    gpu = run_gpu(L, *inp)
    compare(gpu, run_oracle(L, *inp), label="64 adapters")
    with pytest.raises(binding.LoraError) as e:
        binding.multi_lora_fwd(gpu["Y"].new_empty((L.M, 192)), W[:, :192].contiguous(), inp[2].cuda().repeat(2, 1, 1)[:65],
                               inp[3].cuda().repeat(2, 1, 1)[:65], list(range(0, 65)) + [L.M], [1.0] * 65, [0.1] * 65, [1] * 65)
    assert e.value.status in (5, 7)


HETERO = [  # M, K, N, allocated r, segment lengths, ranks
    (832, 256, 320, 64, (192, 64, 128, 448), (16, 64, 32, 16)),          # boundaries on 64: tiles with several adapters
    (601, 320, 192, 32, (100, 37, 300, 164), (32, 16, 16, 32)),          # boundaries off the 64 grid
    (768, 192, 448, 64, (64, 64, 128, 0, 512), (32, 16, 64, 16, 32)),    # three ranks inside one row tile
]


@pytest.mark.parametrize("case", HETERO, ids=lambda c: "x".join(str(v) for v in c[:4]))
def test_heterogeneous_rank(case):
    """Adapters of different rank in one packed batch (arrays allocated at the largest rank): every
    segment equals the single-adapter call at its own rank on the compact arrays, bit for bit, and the
    oracle run per segment; padding of A and B is never used (it holds NaN here) and the padding of
    S', dA and dB comes out as zeros."""
    M, K, N, r, lens, ranks = case
    L = workloads.custom_layer(M, K, N, r, 2.0, 0.1, seg_lens=lens, cfg=8)
    print(f"hetero rank {L} ranks={ranks}", flush=True)
    X, W, A, B, dY = workloads.make_inputs(L)
    A, B = A.clone(), B.clone()
    for g, rg in enumerate(ranks):
        A[g, rg:] = float("nan")
        B[g, :, rg:] = float("nan")
    s = [0.5 + g for g in range(L.G)]
    p = [0.05 * (g + 1) for g in range(L.G)]
    dev = "cuda"
    Xg, Wg, Ag, Bg, dYg = (t.to(dev) for t in (X, W, A, B, dY))
    Y, S = binding.multi_lora_fwd(Xg, Wg, Ag, Bg, L.seg_offsets, s, p, L.seeds, ranks=ranks)
    dX, dA, dB = binding.multi_lora_bwd(Xg, Wg, Ag, Bg, S, dYg, L.seg_offsets, s, p, L.seeds, ranks=ranks)
    torch.cuda.synchronize()
    o = L.seg_offsets
    for g, rg in enumerate(ranks):
        sl = slice(o[g], o[g + 1])
        assert not S[sl, rg:].any() and torch.isfinite(S[sl]).all()
        if o[g + 1] == o[g]:
            assert not dA[g].any() and not dB[g].any()
            continue
        assert not dA[g, rg:].any() and not dB[g, :, rg:].any()
        Ac, Bc = Ag[g, :rg].contiguous(), Bg[g, :, :rg].contiguous()
        # oracle on the compact adapter
        Yr, Sr = oracle.lora_fwd(f64(X[sl]), f64(W), f64(A[g, :rg]), f64(B[g, :, :rg]), s[g], p[g], L.seeds[g])
        dXr, dAr, dBr, _ = oracle.lora_bwd(f64(X[sl]), f64(W), f64(A[g, :rg]), f64(B[g, :, :rg]), f64(dY[sl]),
                                           s[g], p[g], L.seeds[g])
        compare(dict(Y=Y[sl], S=S[sl, :rg], dX=dX[sl], dA=dA[g, :rg], dB=dB[g, :, :rg]),
                dict(Y=Yr, S=Sr * float(np.float32(s[g])), dX=dXr, dA=dAr, dB=dBr), label=f"hetero {case} g={g}")
        # the single-adapter entry point at rank rg
        Y1, S1 = binding.lora_fwd(Xg[sl].contiguous(), Wg, Ac, Bc, s[g], p[g], L.seeds[g])
        dX1, dA1, dB1 = binding.lora_bwd(Xg[sl].contiguous(), Wg, Ac, Bc, S1, dYg[sl].contiguous(), s[g], p[g], L.seeds[g])
        assert torch.equal(Y1, Y[sl]) and torch.equal(S1, S[sl, :rg]) and torch.equal(dX1, dX[sl])
        assert torch.equal(dA1, dA[g, :rg]) and torch.equal(dB1, dB[g, :, :rg])
    with pytest.raises(binding.LoraError) as e:        # a rank above the allocated one
        binding.multi_lora_fwd(Xg, Wg, Ag, Bg, L.seg_offsets, s, p, L.seeds, ranks=[2 * r] + list(ranks[1:]))
    assert e.value.status == 7
    with pytest.raises(binding.LoraError) as e:
        binding.multi_lora_fwd(Xg, Wg, Ag, Bg, L.seg_offsets, s, p, L.seeds, ranks=[24] + list(ranks[1:]))
    assert e.value.status == 7


def test_fused_qkv_as_one_lora_linear():
    """Three projections that share their input (q, k, v of a decoder layer) run as one LoRA linear with
    W = [Wq; Wk; Wv], A = [Aq; Ak; Av; 0] and a block-diagonal B: with one dropout seed the forward
    equals the three separate calls bit for bit, dA and the diagonal blocks of dB too, and dX is the sum
    of the three input gradients (checked against the oracle's sum)."""
    M, K, r = 320, 256, 16
    Ns = (256, 64, 64)
    s, p, seed = 2.0, 0.1, 77
    dev = "cuda"
    parts = [workloads.make_inputs(workloads.custom_layer(M, K, n, r, s, p, cfg=13), layer_index=i) for i, n in enumerate(Ns)]
    X = parts[0][0]
    Wc = torch.cat([q[1] for q in parts])
    dYc = torch.cat([q[4] for q in parts], dim=1).contiguous()
    Ac = torch.zeros((64, K), dtype=torch.bfloat16)
    Bc = torch.zeros((sum(Ns), 64), dtype=torch.bfloat16)
    n0 = 0
    for i, (q, n) in enumerate(zip(parts, Ns)):
        Ac[16 * i:16 * i + 16] = q[2][0]
        Bc[n0:n0 + n, 16 * i:16 * i + 16] = q[3][0]
        n0 += n
    print("fused qkv", flush=True)
    Xg = X.to(dev)
    Y, S = binding.lora_fwd(Xg, Wc.to(dev), Ac.to(dev), Bc.to(dev), s, p, seed)
    dX, dA, dB = binding.lora_bwd(Xg, Wc.to(dev), Ac.to(dev), Bc.to(dev), S, dYc.to(dev), s, p, seed)
    torch.cuda.synchronize()
    assert not S[:, 48:].any() and not dA[48:].any()
    dX_ref = np.zeros((M, K))
    n0 = 0
    for i, (q, n) in enumerate(zip(parts, Ns)):
        _, W, A, B, dY = q
        Y1, S1 = binding.lora_fwd(Xg, W.to(dev), A[0].to(dev), B[0].to(dev), s, p, seed)
        _, dA1, dB1 = binding.lora_bwd(Xg, W.to(dev), A[0].to(dev), B[0].to(dev), S1, dY.to(dev), s, p, seed)
        assert torch.equal(Y1, Y[:, n0:n0 + n]) and torch.equal(S1, S[:, 16 * i:16 * i + 16])
        assert torch.equal(dA1, dA[16 * i:16 * i + 16]) and torch.equal(dB1, dB[n0:n0 + n, 16 * i:16 * i + 16])
        dX_ref += oracle.lora_bwd(f64(X), f64(W), f64(A[0]), f64(B[0]), f64(dY), s, p, seed)[0]
        n0 += n
    assert rel_err(dX, dX_ref) <= TOL
