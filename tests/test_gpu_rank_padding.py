"""Padding of adapters whose rank lies below the allocated one, when the incoming gradient holds non-finite values (an
overflowed step): the padding of dB and dA is written as zeros, and left as it is under accumulate; what the non-finite
element does not reach has the bits of the clean call."""
import pytest
import torch

from paper_2510_00206_amd import binding, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("inf"), float("nan")], ids=["inf", "nan"])
@pytest.mark.parametrize("r,ranks", [(32, (16, 32, 16)), (64, (32, 16, 64))])
def test_padding_of_gradients_stays_zero(r, ranks, value):
    L = workloads.custom_layer(330, 192, 576, r, 1.5, 0.1, seg_lens=(130, 64, 136), cfg=81)
    print(f"rank padding {L} ranks={ranks} value={value}", flush=True)
    X, W, A, B, dY = (t.cuda() for t in workloads.make_inputs(L))
    s, p, o = [L.s] * L.G, [L.p] * L.G, L.seg_offsets
    _, S = binding.multi_lora_fwd(X, W, A, B, o, s, p, L.seeds, ranks=ranks)
    clean = binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, ranks=ranks)
    hit = [(o[0] + 70, 5), (o[1] + 3, 515), (o[3] - 1, 575)]          # one in each segment, the last in the last row
    for row, col in hit:
        dY[row, col] = value
    out = binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, ranks=ranks)
    base_a, base_b = torch.randn_like(out[1]), torch.randn_like(out[2])
    acc = binding.multi_lora_bwd(X, W, A, B, S, dY, o, s, p, L.seeds, ranks=ranks, dA=base_a.clone(), dB=base_b.clone(),
                                 accumulate=True)
    torch.cuda.synchronize()
    for g, rg in enumerate(ranks):
        assert not out[1][g, rg:].any() and not out[2][g, :, rg:].any(), g
        assert torch.equal(acc[1][g, rg:], base_a[g, rg:]) and torch.equal(acc[2][g, :, rg:], base_b[g, :, rg:]), g
        row, col = hit[g]
        assert not torch.isfinite(out[2][g, col, :rg]).any(), g        # the value is really there
        rest = [n for n in range(L.N) if n != col]
        assert torch.equal(out[2][g, rest], clean[2][g, rest]), g
    for row, _ in hit:
        assert not torch.isfinite(out[0][row]).any()
    rest = [i for i in range(L.M) if i not in [row for row, _ in hit]]
    assert torch.equal(out[0][rest], clean[0][rest])
