"""Workloads of the LoRA linear layer that the library is timed on, through its public entry points
(`paper_2510_00206_amd.binding`): forward, backward and whole training steps of one layer, from a
launch-bound microbatch to the widest projection of the benchmark configurations.

A case is a dict of plain values:
  do      "fwd" | "bwd" | "step" (forward, then backward)
  K, N    input and output features;  r  allocated rank
  segs    token counts of the packed segments, one adapter each ("8192", "10944,2752,1408,1280")
  ranks   per-adapter ranks ("16,64,32") or "" (all r)
  s, p    LoRA scale and dropout probability (the same for every adapter)
  dx      whether the backward returns dX (the first layer of a frozen model needs none)
  micro   microbatches whose adapter gradients are summed (the second and later ones accumulate)
Values follow the repository's input recipe: X, dY ~ N(0,1), W ~ N(0,1/K), A ~ U(-K^-1/2, K^-1/2),
B ~ N(0, 0.02^2), all bf16.  Weights, adapters, outputs and the backward's workspace are held from pass
to pass, as a training program holds them.
"""
import math

import torch

from paper_2510_00206_amd import binding

_DEFAULTS = dict(do="step", ranks="", s=2.0, p=0.1, dx=True, micro=1)


def _case(name, K, N, r, segs, **kw):
    return dict(_DEFAULTS, name=name, K=K, N=N, r=r, segs=segs, **kw)


def listed():
    return [
        # one short sequence through a small layer: launches and latency only (benchmark configuration 1)
        _case("small_step", 1024, 1024, 16, "256"),
        # scoring one short prompt with the adapter on: no dropout, a token count off every grid, MLP-wide weight
        _case("prompt_eval", 4096, 14336, 16, "77", do="fwd", p=0.0),
        # a microbatch of one 1024-token sequence on an attention projection (smallest of the token sweep)
        _case("short_step", 4096, 4096, 16, "1024"),
        # three tenants' short samples packed end to end, boundaries as they fall, adapters of different rank,
        # key/value projection
        _case("packed_ragged_step", 4096, 1024, 64, "700,331,500", ranks="16,64,32"),
        # unpadded batch of odd length, rank 32
        _case("odd_step", 4096, 4096, 32, "2999"),
        # gradient accumulation over two microbatches in the first layer (its input needs no gradient)
        _case("accumulate_first_layer", 4096, 4096, 16, "2048", do="bwd", dx=False, micro=2),
        # the headline projection (8192 tokens, 4096 x 4096), each direction by itself
        _case("attn_fwd", 4096, 4096, 16, "8192", do="fwd"),
        _case("attn_bwd", 4096, 4096, 16, "8192", do="bwd"),
        # four adapters packed on 64-row boundaries (benchmark configuration 4)
        _case("packed4_step", 4096, 4096, 16, "10944,2752,1408,1280"),
        # MLP down projection, unpadded token count
        _case("mlp_down_odd_step", 14336, 4096, 16, "5003", p=0.05),
        # MLP gate/up projection (benchmark configuration 3)
        _case("mlp_gate_step", 4096, 14336, 16, "8192", p=0.05),
        # wide projection at rank 64 (benchmark configuration 5)
        _case("wide_r64_step", 8192, 28672, 64, "4096", s=0.5),
    ]


def _ints(text):
    return [int(v) for v in text.split(",")] if text else []


def _cost(case):
    w = work(case)
    return w["flops"] / 1e15 + w["bytes"] / 5e12


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    cap = max(_cost(c) for c in listed())
    while True:
        M = _log_int(rng, 16, 16384)
        if rng.random() < 0.4:
            M = max(64, M // 64 * 64)
        K, N = (min(28672, max(64, _log_int(rng, 256, 28672) // 64 * 64)) for _ in range(2))
        r = rng.choice((16, 16, 32, 64))
        G = rng.choice((1, 1, 2, 3, 5, 8))
        if M < 4 * G:
            G = 1
        grid = 64 if M % 64 == 0 and M // 64 >= G and rng.random() < 0.7 else 1
        cuts = sorted(rng.sample(range(1, M // grid), G - 1))
        lens = [(b - a) * grid for a, b in zip([0] + cuts, cuts + [M // grid])]
        ranks = ",".join(str(rng.choice([v for v in (16, 32, 64) if v <= r])) for _ in lens) if G > 1 and rng.random() < 0.4 else ""
        do = rng.choice(("fwd", "bwd", "step", "step"))
        case = dict(_DEFAULTS, do=do, K=K, N=N, r=r, segs=",".join(map(str, lens)), ranks=ranks,
                    s=rng.choice((0.5, 1.0, 2.0)), p=0.0 if do == "fwd" and rng.random() < 0.5 else rng.choice((0.05, 0.1, 0.25)),
                    dx=do != "bwd" or rng.random() < 0.7, micro=2 if do == "bwd" and M <= 4096 and rng.random() < 0.3 else 1)
        if _cost(case) <= cap:
            return case


# ---- inputs ------------------------------------------------------------------------------------------
def _seeds(case, micro):
    return [0x25100206 + 1000 * micro + g for g in range(len(_ints(case["segs"])))]


def _inputs(case, seed):
    """Weights and adapters, then X and dY of every microbatch, from the seed alone."""
    dev = "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) % (1 << 63))
    K, N, r, lens = case["K"], case["N"], case["r"], _ints(case["segs"])
    M, G = sum(lens), len(lens)

    def normal(shape, std):
        t = torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)
        return t.mul_(std).to(torch.bfloat16)

    W = normal((N, K), K ** -0.5)
    A = ((torch.rand((G, r, K), generator=gen, device=dev) * 2 - 1) * K ** -0.5).to(torch.bfloat16)
    B = normal((G, N, r), 0.02)
    mbs = []
    for _ in range(case["micro"]):
        X = normal((M, K), 1.0)
        mbs.append((X, normal((M, N), 1.0) if case["do"] != "fwd" else None))
    return W, A, B, mbs


class _State:
    pass


def prepare(case, seed):
    st = _State()
    lens = _ints(case["segs"])
    M, G, K, N, r = sum(lens), len(lens), case["K"], case["N"], case["r"]
    st.case, st.G = case, G
    st.W, A, B, st.mbs = _inputs(case, seed)
    st.A, st.B = (A, B) if G > 1 else (A[0].contiguous(), B[0].contiguous())
    st.off = [0]
    for n in lens:
        st.off.append(st.off[-1] + n)
    st.ranks = _ints(case["ranks"]) or None
    st.s, st.p = [case["s"]] * G, [case["p"]] * G
    st.seeds = [_seeds(case, m) for m in range(case["micro"])]
    new = lambda shape, dt: torch.empty(shape, dtype=dt, device="cuda")
    st.Y, st.S = new((M, N), torch.bfloat16), [new((M, r), torch.bfloat16) for _ in st.mbs]
    st.dX = st.dA = st.dB = st.ws = None
    if case["do"] != "fwd":
        lead = (G,) if G > 1 else ()
        st.dX = new((M, K), torch.bfloat16) if case["dx"] else None
        st.dA, st.dB = new(lead + (r, K), torch.float32), new(lead + (N, r), torch.float32)
        st.ws = binding.alloc_workspace(M, K, N, r, G)
    if case["do"] == "bwd":                      # the forward of these microbatches has been run
        for m in range(case["micro"]):
            _forward(st, m)
    return st


def _forward(st, m):
    X = st.mbs[m][0]
    if st.G == 1:
        binding.lora_fwd(X, st.W, st.A, st.B, st.s[0], st.p[0], st.seeds[m][0], Y=st.Y, S=st.S[m])
    else:
        binding.multi_lora_fwd(X, st.W, st.A, st.B, st.off, st.s, st.p, st.seeds[m], Y=st.Y, S=st.S[m], ranks=st.ranks)


def _backward(st, m):
    X, dY = st.mbs[m]
    kw = dict(need_dx=st.dX is not None, dA=st.dA, dB=st.dB, accumulate=m > 0, workspace=st.ws, dX=st.dX)
    if st.G == 1:
        binding.lora_bwd(X, st.W, st.A, st.B, st.S[m], dY, st.s[0], st.p[0], st.seeds[m][0], **kw)
    else:
        binding.multi_lora_bwd(X, st.W, st.A, st.B, st.S[m], dY, st.off, st.s, st.p, st.seeds[m], ranks=st.ranks, **kw)


def run(st):
    do = st.case["do"]
    out = {}
    for m in range(len(st.mbs)):
        if do != "bwd":
            _forward(st, m)
        if do != "fwd":
            _backward(st, m)
    if do != "bwd":
        out["Y"], out["S"] = st.Y, st.S[-1]
    if do != "fwd":
        out["dA"], out["dB"] = st.dA, st.dB
        if st.dX is not None:
            out["dX"] = st.dX
    return out


# ---- what a pass cannot do without -------------------------------------------------------------------
def work(case):
    lens = _ints(case["segs"])
    ranks = _ints(case["ranks"]) or [case["r"]] * len(lens)
    M, G, K, N, r = sum(lens), len(lens), case["K"], case["N"], case["r"]
    Mr = sum(n * q for n, q in zip(lens, ranks))                 # rows times the rank they use
    fwd, bwd, dx = case["do"] != "bwd", case["do"] != "fwd", case["dx"]
    lora = sum(ranks) * (K + N)                                  # elements of A and B in use
    nbytes = 2 * M * K + 2 * lora                                # X, A, B
    flops = 0
    if fwd or dx:
        nbytes += 2 * K * N                                      # W
    if fwd:
        nbytes += 2 * M * N + 2 * M * r                          # Y, S
        flops += 2 * M * K * N + 2 * Mr * (K + N)
    if bwd:
        nbytes += 2 * M * N + 4 * G * r * (K + N)                # dY, dA, dB
        flops += 2 * Mr * (K + 2 * N)                            # dA, dS, dB
        if not fwd:
            nbytes += 2 * M * r                                  # S
        if dx:
            nbytes += 2 * M * K                                  # dX
            flops += 2 * M * K * N + 2 * Mr * K
    if case["micro"] > 1:
        once = 2 * lora + 4 * G * r * (K + N) + (2 * K * N if dx else 0)
        nbytes, flops = once + (nbytes - once) * case["micro"], flops * case["micro"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 outputs, and bf16 intermediates (S, dS) behind the fp32 ones: the 2-norm error against the 64-bit
    # result measures 1.6e-3 to 1.7e-3 for every output; four times that.  One element may land on the other
    # side of a rounding step (up to 2^-7 of its value); four times that.
    return {"rel": 7e-3, "max": 3e-2}


# ---- the same in 64 bits, in plain torch ---------------------------------------------------------------
_U = 0xFFFFFFFF
_GOLD, _M1, _M2, _C5, _C7 = 0x9E3779B9, 0x6A09E667, 0xBB67AE85, 0x3C6EF373, 0xA54FF53B


def _mix(x):
    x = x ^ (x >> 16)
    x = (x * _M1) & _U
    x = x ^ (x >> 15)
    x = (x * _M2) & _U
    return x ^ (x >> 16)


def _dropped(X64, p, seed):
    """X64 with dropped elements zeroed (survivors not yet scaled), the keep mask and the survivor scale."""
    T = int(min(65535, math.floor(float(torch.tensor(p, dtype=torch.float32)) * 65536.0)))
    M, K = X64.shape
    dev = X64.device
    k0 = _mix(torch.tensor((seed & _U) ^ _C5, dtype=torch.int64, device=dev))
    k1 = _mix((torch.tensor(seed >> 32, dtype=torch.int64, device=dev) + k0) & _U)
    rows = torch.arange(M, dtype=torch.int64, device=dev)
    ka = _mix(k1 ^ ((rows * _GOLD) & _U))
    kb = _mix((ka + k0 + _C7) & _U)
    cols = (torch.arange(K // 2, dtype=torch.int64, device=dev) * _GOLD) & _U
    x = (ka[:, None] + cols[None, :]) & _U
    x ^= x >> 16
    x = (x * _M1) & _U
    x = (x + kb[:, None]) & _U
    x ^= x >> 15
    x = (x * _M2) & _U
    x ^= x >> 16
    keep = torch.stack(((x & 0xFFFF) >= T, (x >> 16) >= T), dim=2).reshape(M, K)
    return X64 * keep, keep, 65536.0 / (65536.0 - T)


def exact(case, seed):
    lens = _ints(case["segs"])
    ranks = _ints(case["ranks"]) or [case["r"]] * len(lens)
    M, G, K, N, r, s = sum(lens), len(lens), case["K"], case["N"], case["r"], case["s"]
    fwd, bwd = case["do"] != "bwd", case["do"] != "fwd"
    W, A, B, mbs = _inputs(case, seed)
    W64, d = W.double(), torch.float64
    dA, dB = torch.zeros((G, r, K), dtype=d, device="cuda"), torch.zeros((G, N, r), dtype=d, device="cuda")
    out = {}
    for m, (X, dY) in enumerate(mbs):
        S = torch.zeros((M, r), dtype=d, device="cuda")
        Y = X.double() @ W64.t() if fwd else None
        dX = dY.double() @ W64 if bwd and case["dx"] else None
        row = 0
        for g, (n, q) in enumerate(zip(lens, ranks)):
            sl = slice(row, row + n)
            row += n
            Xd, keep, scale = _dropped(X[sl].double(), case["p"], _seeds(case, m)[g])
            A64, B64 = A[g, :q].double(), B[g, :, :q].double()
            Sg = (Xd @ A64.t()) * scale
            S[sl, :q] = s * Sg                                   # the saved intermediate is s * S
            if fwd:
                Y[sl] += (s * Sg) @ B64.t()
            if bwd:
                dYg = dY[sl].double()
                dS = s * (dYg @ B64)
                dB[g, :, :q] += s * (dYg.t() @ Sg)
                dA[g, :q] += (dS * scale).t() @ Xd
                if dX is not None:
                    dX[sl] += keep * scale * (dS @ A64)
        if fwd:
            out["Y"], out["S"] = Y, S
        if dX is not None:
            out["dX"] = dX
    if bwd:
        out["dA"], out["dB"] = (dA, dB) if G > 1 else (dA[0], dB[0])
    return out
