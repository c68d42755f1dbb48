"""GPU parity of the fp32 expert GEMMs at the edges of their tiles: rows of 32 and 64, columns of 64 and 128, slabs of 32
k-values, and batches of experts whose intermediate sits in the outputs of experts still to come.  Bound: a sum of K
fp32 products carries at most K 2^-24 of the sum of their magnitudes; 1e-5 of the largest output covers K <= 576."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_14800_amd as pkg
from paper_2402_14800_amd import workloads as wl
from tests.test_gpu_parity import small_layer, to_dev

pytestmark = pytest.mark.gpu
NAMES = ("x", "Wgate", "W1", "W3", "W2")


@pytest.mark.parametrize("E,H,F,T", [
    (8, 36, 68, 1),         # one row; K = 36 and 68: a partly filled slab
    (3, 64, 60, 33),        # F < H: two experts' h in the outputs of the third
    (7, 128, 132, 65),      # F just above H, a second tile of one row
    (5, 576, 64, 97),       # h much smaller than the outputs: four experts in a launch
    (2, 4, 260, 130),       # the narrowest H, F = 65 H: a launch per expert
    (8, 192, 128, 1400),    # five experts in a launch, 32 x 64 tiles
    (8, 192, 128, 3000),    # 32 x 128 tiles
    (8, 64, 128, 9001),     # 64 x 128 tiles
])
def test_fp32_expert_outputs_at_tile_edges(E, H, F, T):
    _, layer = small_layer("f32", E, 2, H, F, T, index=25)
    d = to_dev(layer)
    ws = [d[n] for n in NAMES]
    lg, Y = pkg.moe_expert_outputs(*ws)
    n = min(2, E)
    lg_r, experts, slot, Yr = pkg.moe_expert_outputs_ranked(*ws, n)
    torch.cuda.synchronize()
    args = [wl.to_f64(layer[n_]) for n_ in NAMES]
    _, ref = oracle.expert_outputs(*args)
    assert np.abs(wl.to_f64(Y) - ref).max() <= 1e-5 * np.abs(ref).max()
    t = torch.arange(T, device=Y.device)
    assert torch.equal(lg, lg_r)
    for j in range(n):
        assert torch.equal(Yr[slot[:, j].long()], Y[experts[:, j].long(), t])
    if E >= 2:
        out, skip, lg_f, _ = pkg.moe_forward_skip(*ws, 0.5)
        torch.cuda.synchronize()
        ref_out, ref_skip, _, _ = oracle.forward_skip(*args, 0.5, logits=lg_f.cpu().numpy())
        assert np.array_equal(skip.cpu().numpy().astype(bool), ref_skip)
        assert np.abs(wl.to_f64(out) - ref_out).max() <= 1e-5 * np.abs(ref_out).max()


@pytest.mark.parametrize("E,H,F,T", [(8, 64, 128, 9001), (4, 260, 132, 3000)])
def test_fp32_outputs_do_not_depend_on_the_batch(E, H, F, T):
    """A token alone, in small batches and in one that takes the largest tiles: the same bits of its outputs."""
    _, layer = small_layer("f32", E, 2, H, F, T, index=30)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    lg, Y = pkg.moe_expert_outputs(d["x"], *rest)
    out, skip, _, _ = pkg.moe_forward_skip(d["x"], *rest, 0.5)
    torch.cuda.synchronize()
    for t0, rows in ((11, 1), (0, 33), (100, 700)):
        x = d["x"][t0:t0 + rows].contiguous()
        lg_p, Y_p = pkg.moe_expert_outputs(x, *rest)
        out_p, skip_p, _, _ = pkg.moe_forward_skip(x, *rest, 0.5)
        torch.cuda.synchronize()
        assert torch.equal(lg_p, lg[t0:t0 + rows]) and torch.equal(Y_p, Y[:, t0:t0 + rows].contiguous())
        assert torch.equal(skip_p, skip[t0:t0 + rows]) and torch.equal(out_p, out[t0:t0 + rows])


@pytest.mark.parametrize("E,H,F,T", [(8, 192, 128, 700), (3, 64, 60, 33), (8, 64, 128, 9001)])
@pytest.mark.parametrize("offset", [1, 2])
def test_fp32_expert_outputs_at_four_byte_alignment(E, H, F, T, offset):
    """Outputs whose rows are not 16-byte aligned are the bits of aligned ones, and nothing is written around them."""
    _, layer = small_layer("f32", E, 2, H, F, T, index=33)
    d = to_dev(layer)
    ws = [d[n] for n in NAMES]
    _, Y = pkg.moe_expert_outputs(*ws)
    ranked = pkg.moe_expert_outputs_ranked(*ws, 2)
    buf = torch.full((E * T * H + 8,), 7.0, device="cuda:0")
    shifted = buf[offset:offset + E * T * H].view(E, T, H)
    pkg.moe_expert_outputs(*ws, Y=shifted)
    torch.cuda.synchronize()
    assert shifted.data_ptr() % 16 == 4 * offset and torch.equal(shifted, Y)
    assert torch.all(buf[:offset] == 7.0) and torch.all(buf[offset + E * T * H:] == 7.0)
    part = buf[offset:offset + 2 * T * H].view(2 * T, H)
    pkg.moe_expert_outputs_ranked(*ws, 2, out=(*[torch.empty_like(v) for v in ranked[:3]], part))
    torch.cuda.synchronize()
    assert torch.equal(part, ranked[3])


@pytest.mark.parametrize("E,H,F,T", [
    (8, 192, 128, 4000),    # 64 x 128 tiles, one slab in flight
    (8, 192, 128, 5500),    # two
    (8, 96, 100, 700),      # three slabs; three and a partly filled one
    (4, 32, 28, 50),        # one slab, and less than one
])
def test_fp32_weights_of_any_alignment_give_the_same_bits(E, H, F, T):
    """Direct loads take 16-byte aligned weights; weights that begin 4 bytes further are staged through registers."""
    _, layer = small_layer("f32", E, 2, H, F, T, index=36)
    d = to_dev(layer)

    def shifted(w):
        room = torch.empty(w.numel() + 1, dtype=w.dtype, device=w.device)
        room[1:] = w.reshape(-1)
        return room[1:].view(w.shape)

    ws = [d[n] for n in NAMES]
    odd = [d["x"], d["Wgate"], *[shifted(d[n]) for n in NAMES[2:]]]
    assert all(w.data_ptr() % 16 == 4 for w in odd[2:])
    _, Y = pkg.moe_expert_outputs(*ws)
    _, Y_odd = pkg.moe_expert_outputs(*odd)
    out, _, _, _ = pkg.moe_forward_skip(*ws, 0.5)
    out_odd, _, _, _ = pkg.moe_forward_skip(*odd, 0.5)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y_odd) and torch.equal(out, out_odd)
    _, ref = oracle.expert_outputs(*[wl.to_f64(layer[n]) for n in NAMES])
    assert np.abs(wl.to_f64(Y) - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("E,H,F,T,kept", [
    (32, 64, 68, 300, 0x80000001),      # rows for the first and the last expert only
    (32, 36, 132, 2600, 0xffffffff),    # 32-row tiles
    (17, 64, 64, 9001, 0x1a005),        # 64-row tiles, experts without rows on both sides of the 16th
    (16, 128, 192, 700, 0x8001),
    (2, 64, 64, 65, 0x3),
])
def test_fp32_row_tiles_of_each_experts_segment(E, H, F, T, kept):
    """Every routed row is multiplied with its own expert's weights, whichever experts have rows: the outputs are the Eq. 2 sums of
    the dense pass (the same products; three fp32 roundings and expf besides, within the bound above)."""
    _, layer = small_layer("f32", E, 2, H, F, T, index=40)
    d = to_dev(layer)
    ws = [d[n] for n in NAMES]
    lg, Y = pkg.moe_expert_outputs(*ws)
    out, skip, lg_f, top2 = pkg.moe_forward_pruned_skip(*ws, kept, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(lg, lg_f) and not skip.any()
    t = torch.arange(T, device=Y.device)
    e0, e1 = top2[:, 0].long(), top2[:, 1].long()
    assert set(top2.unique().tolist()) <= {e for e in range(E) if kept >> e & 1}
    rho = (lg[t, e1].double() - lg[t, e0].double()).exp()[:, None]
    ref = (Y[e0, t].double() + rho * Y[e1, t].double()) / (1 + rho)
    assert (out.double() - ref).abs().max() <= 1e-5 * ref.abs().max()
