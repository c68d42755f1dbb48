"""The router on both sides of its few-tokens form: a token's logits are the same bits in any batch and from every entry
point, and the routed passes over many routing blocks agree with the counts that their logits imply."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_14800_amd as pkg
from tests.test_gpu_parity import small_layer, to_dev

pytestmark = pytest.mark.gpu
NAMES = ("x", "Wgate", "W1", "W3", "W2")


@pytest.mark.parametrize("E,H", [(8, 64), (8, 1088), (16, 576), (20, 192), (32, 2112)])
def test_logits_of_every_form_are_the_same_bits(E, H):
    _, layer = small_layer("bf16", E, 2, H, 64, 16400, index=27)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    full, _ = pkg.moe_expert_outputs(d["x"], *rest)                 # beyond both limits
    torch.cuda.synchronize()
    ref = layer["x"].double() @ layer["Wgate"].double().t()
    assert (full.cpu().double() - ref).abs().max() <= 1e-5 * ref.abs().max()
    for T in (1, 15, 33, 8192, 8193, 16384):
        x = d["x"][:T].contiguous()
        dense, _ = pkg.moe_expert_outputs(x, *rest)
        _, _, routed, _ = pkg.moe_forward_skip(x, *rest, 0.5)
        torch.cuda.synchronize()
        assert torch.equal(dense, full[:T]) and torch.equal(routed, full[:T])


@pytest.mark.parametrize("E,H,sizes", [
    (8, 1088, (4096, 4097)), (20, 192, (4096, 4097)),               # eight wavefronts per 16 tokens, and two
    (8, 96, (7, 4096)), (32, 320, (16, 4097)),                      # fewer slices than wavefronts, a ragged last slice of each
    (8, 4096, (4097, 32768)), (17, 4160, (777, 8193)),              # long rows: eight wavefronts up to 32768 tokens
])
def test_logits_of_the_forms_by_length_of_a_row_are_the_same_bits(E, H, sizes):
    T = 32769 if H == 4096 else 8400
    _, layer = small_layer("bf16", E, 2, max(H // 64, 1) * 64, 64, T, index=35)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    full, _, _, _ = pkg.moe_expert_outputs_ranked(d["x"], *rest, 1)
    torch.cuda.synchronize()
    some = slice(0, 512)
    ref = layer["x"][some].double() @ layer["Wgate"].double().t()
    assert (full[some].cpu().double() - ref).abs().max() <= 1e-5 * ref.abs().max()
    for n in sizes:
        x = d["x"][:n].contiguous()
        dense, _ = pkg.moe_expert_outputs(x, *rest)
        _, _, routed, _ = pkg.moe_forward_skip(x, *rest, 0.5)
        torch.cuda.synchronize()
        assert torch.equal(dense, full[:n]) and torch.equal(routed, full[:n])


@pytest.mark.parametrize("E", [2, 4, 5])
@pytest.mark.parametrize("H,T", [(4, 3), (516, 65), (2048, 1025)])
def test_fp32_logits_of_few_experts_are_those_among_more(E, H, T):
    """Up to 4, 8 and 16 experts are forms of their own: an expert's logit is the same bits in each, and near its sum in 64 bits
    (H products and at most H additions, each off by 2^-24 of the sum of magnitudes)."""
    _, layer = small_layer("f32", 16, 2, H, 64, T, index=39)
    d = to_dev(layer)
    full, _ = pkg.moe_expert_outputs(*[d[n] for n in NAMES])
    few, _ = pkg.moe_expert_outputs(d["x"], *[d[n][:E].contiguous() for n in NAMES[1:]])
    torch.cuda.synchronize()
    assert torch.equal(few, full[:, :E].contiguous())
    x, w = layer["x"].double(), layer["Wgate"][:E].double()
    assert bool(((few.cpu().double() - x @ w.t()).abs() <= 2 * H * 2.0 ** -24 * (x.abs() @ w.abs().t())).all())


@pytest.mark.parametrize("E,T,n", [(8, 16400, 3), (5, 8193, 2), (32, 9000, 1)])
def test_slots_of_many_routing_blocks(E, T, n):
    """Rows of the rank-limited pass: grouped by expert, ascending token within an expert, nothing left out."""
    _, layer = small_layer("bf16", E, 2, 64, 64, T, index=28)
    d = to_dev(layer)
    lg, experts, slot, _ = pkg.moe_expert_outputs_ranked(*[d[n_] for n_ in NAMES], n)
    torch.cuda.synchronize()
    ids = oracle.routing_order(lg.cpu().numpy())[:, :n]
    assert np.array_equal(experts.cpu().numpy(), ids)
    token = np.repeat(np.arange(T), n)
    rows = np.lexsort((token, ids.reshape(-1)))
    want = np.empty(T * n, dtype=np.int64)
    want[rows] = np.arange(T * n)
    assert np.array_equal(slot.cpu().numpy().reshape(-1), want)
