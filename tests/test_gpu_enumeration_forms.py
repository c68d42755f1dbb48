"""The enumeration's reduction on both sides of its one-workgroup form, scoring tiles dealt to strands of wavefronts, and
the record capacities of the routing prep, against the fp64 oracle (losses: fp32 sums within a tile of 32 tokens and up to
a few hundred fp32 operations per term, 1e-5 relative covers both)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2402_14800_amd as pkg
from paper_2402_14800_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,r,T,H,dtype", [
    (8, 2, 4, 14976, 64, "bf16"),      # 468 tiles x 70 subsets, through Gram matrices in memory
    (8, 2, 4, 14977, 64, "bf16"),      # a last tile of one token
    (8, 2, 4, 5600, 64, "bf16"),       # 175 tiles x 70 subsets: the last size of the one-workgroup reduction
    (8, 2, 4, 5601, 64, "bf16"),       # one token more: reduced by a workgroup per subset
    (16, 2, 14, 4608, 64, "bf16"),     # the most tokens of short rows whose records the Gram kernel writes
    (16, 2, 14, 4609, 64, "bf16"),     # one more: through Gram matrices in memory
    (8, 2, 4, 33, 64, "bf16"),         # a tile of one token: strands without work
    (4, 2, 2, 7, 64, "f32"),           # fewer tokens than strands
    (1, 1, 1, 40, 64, "bf16"),         # one expert, one subset
    (10, 3, 5, 600, 64, "bf16"),       # 252 subsets: 256 lanes, several tiles
    (17, 4, 9, 6, 64, "bf16"),         # capacity 12 with more than 16 experts
    (18, 1, 16, 100, 64, "bf16"),      # capacity 4 with more than 16 experts
    (13, 2, 7, 50, 64, "bf16"),        # 8 active ranks of 13 experts, 1716 subsets
    (16, 4, 4, 4033, 64, "bf16"),      # 1820 subsets: 8 x 127 workgroups with strands (16 ranks, all in use)
    (16, 4, 4, 4065, 64, "bf16"),      # 8 x 128 workgroups: one strand
])
def test_enumeration_at_the_edges_of_its_forms(E, k, r, T, H, dtype):
    logits, Y = wl.make_enumeration_inputs(E, T, H, dtype, seed=77 + E + T)
    loss, amin, amask, unaff = pkg.prune_enumerate(logits.to("cuda:0"), Y.to("cuda:0"), k, r)
    torch.cuda.synchronize()
    ref, ref_amin, masks = oracle.prune_enumerate_gram_form(wl.to_f64(logits), wl.to_f64(Y), k, r)[:3]
    got = loss.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * np.abs(ref).max())
    assert int(amin.item()) == int(np.argmin(got))
    assert (int(amask.item()) & 0xFFFFFFFF) == int(masks[int(amin.item())])
    import math
    assert int(unaff.item()) == (T * math.comb(E - k, r - k) if r >= k else 0)


@pytest.mark.parametrize("E,H,T", [(4, 4, 3), (8, 256, 17), (8, 260, 9), (16, 516, 5), (17, 36, 4), (32, 300, 3), (6, 37, 11), (20, 33, 2)])
def test_fp32_gram_at_row_lengths_and_alignments(E, H, T):
    """fp32 outputs: rows of whole and of partly filled 1 KB blocks, of lengths that are no multiple of 16 bytes, and a Y that
    is only 4-byte aligned."""
    logits, Y = wl.make_enumeration_inputs(E, T, H, "f32", seed=5 * E + H)
    k, r = 2, E - 1
    lg = logits.to("cuda:0")
    buf = torch.empty(E * T * H + 1, dtype=torch.float32, device="cuda:0")
    shifted = buf[1:].view(E, T, H)
    shifted.copy_(Y)
    ref, _, _ = oracle.prune_enumerate_gram_form(wl.to_f64(logits), wl.to_f64(Y), k, r)
    for Yd in (Y.to("cuda:0"), shifted):
        loss, amin, _, _ = pkg.prune_enumerate(lg, Yd, k, r)
        torch.cuda.synchronize()
        got = loss.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * np.abs(ref).max())
        assert int(amin.item()) == int(np.argmin(got))


@pytest.mark.parametrize("E,H,T,n", [(8, 37, 11, 3), (8, 260, 9, 8), (20, 33, 5, 4), (4, 64, 7, 3)])
def test_fp32_ranked_gram_at_row_lengths_and_alignments(E, H, T, n):
    """The same for the rows of the rank-limited pass, in any order behind slot_of: each token's n best-ranked experts."""
    logits, Y = wl.make_enumeration_inputs(E, T, H, "f32", seed=7 * E + H)
    k, r = 2, E - 1
    order = oracle.routing_order(logits.numpy())[:, :n]
    slots = np.random.Generator(np.random.PCG64(E + H)).permutation(T * n).reshape(T, n)
    rows = torch.empty((T * n, H), dtype=torch.float32)
    for t in range(T):
        for j in range(n):
            rows[slots[t, j]] = Y[order[t, j], t]
    lg = logits.to("cuda:0")
    experts = torch.from_numpy(order.astype(np.int32)).to("cuda:0")
    slot_of = torch.from_numpy(slots.astype(np.int32)).to("cuda:0")
    buf = torch.empty(T * n * H + 1, dtype=torch.float32, device="cuda:0")
    shifted = buf[1:].view(T * n, H)
    shifted.copy_(rows)
    ref, _, _ = oracle.prune_enumerate_gram_form(wl.to_f64(logits), wl.to_f64(Y), k, r)
    for Yr in (rows.to("cuda:0"), shifted):
        loss, amin, _, _ = pkg.prune_enumerate_ranked(lg, experts, slot_of, Yr, k, r)
        torch.cuda.synchronize()
        got = loss.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * np.abs(ref).max())
        assert int(amin.item()) == int(np.argmin(got))


@pytest.mark.parametrize("E,k,r,T,spread", [
    (16, 1, 13, 5, 1),        # 4 active ranks: pattern tables of 64 entries, 256 threads
    (16, 2, 13, 17, 60),      # 5 ranks; logits so far apart that a pruned layer's exponentials underflow
    (16, 2, 12, 41, 1),       # 6 ranks in records of 6: positions beyond the record
    (16, 2, 11, 300, 60),     # 7 ranks in records of 8, 14 subsets per lane
    (13, 4, 9, 9, 1),         # 5 experts in the high half: fewer masks than lanes
    (12, 3, 6, 1, 1),         # 9 ranks, a token without partner
    (12, 3, 6, 1030, 60),
    (16, 4, 11, 77, 1),       # 9 ranks, 126 selections: the last 64 partly filled
    (15, 2, 7, 130, 1),       # 10 ranks, 4 tokens per barrier
    (16, 4, 9, 33, 1),        # 11 ranks, 330 selections
    (16, 4, 8, 3, 60),        # 12 ranks, 495 selections, 12870 subsets
    (16, 4, 8, 1027, 1),      # several tiles, the last one short
])
def test_scoring_with_tables_in_lds(E, k, r, T, spread):
    logits, Y = wl.make_enumeration_inputs(E, T, 64, "bf16", seed=11 * E + T)
    logits = logits * spread
    loss, amin, amask, unaff = pkg.prune_enumerate(logits.to("cuda:0"), Y.to("cuda:0"), k, r)
    torch.cuda.synchronize()
    ref, _, masks = oracle.prune_enumerate_gram_form(wl.to_f64(logits), wl.to_f64(Y), k, r)
    got = loss.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * np.abs(ref).max())
    assert int(amin.item()) == int(np.argmin(got))
    assert (int(amask.item()) & 0xFFFFFFFF) == int(masks[int(amin.item())])
    import math
    assert int(unaff.item()) == T * math.comb(E - k, r - k)


@pytest.mark.parametrize("E,k,rs,T", [
    (8, 2, (6, 4), 9001),        # 28 subsets in one workgroup, 70 over the chip
    (8, 2, (5, 6, 7), 700),      # three r and four r whose records are written in one pass
    (8, 1, (5, 6, 7, 8), 700),
    (8, 2, (4, 6, 7, 1), 5600),  # four whose records do not fit the workspace: through Gram matrices in memory
    (8, 2, (4, 6, 7, 1, 5), 700),  # five: the same
    (16, 2, (14, 12), 8000),     # written in one pass for both, through Gram matrices for each alone
    (16, 4, (12, 15), 1100),     # tables for one r, records of the same pass for the other
    (5, 2, (3,), 1),
    (12, 3, (6, 11), 77),
])
def test_several_r_give_the_bits_of_each_alone(E, k, rs, T):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(7 * T + E)
    logits = torch.randn((T, E), generator=gen, device="cuda:0")
    Y = torch.randn((E, T, 192), generator=gen, device="cuda:0").to(torch.bfloat16)
    parts = pkg.prune_enumerate_multi(logits, Y, k, list(rs))
    some = T <= 700                                      # (the oracle takes a second for each r)
    l64, y64 = wl.to_f64(logits), wl.to_f64(Y) if some else None
    for r, part in zip(rs, parts):
        alone = pkg.prune_enumerate(logits, Y, k, r)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(part, alone)), r
        if some:
            ref = oracle.prune_enumerate_gram_form(l64, y64, k, r)[0]
            got = part[0].cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * np.abs(ref).max())


def test_a_loss_of_several_r_can_be_written_under_autograd():
    logits = torch.randn((64, 8), device="cuda:0")
    Y = torch.randn((8, 64, 192), device="cuda:0").to(torch.bfloat16)
    weight = torch.ones((), device="cuda:0", requires_grad=True)
    loss = pkg.prune_enumerate_multi(logits, Y, 2, [6, 4])[0][0]
    loss.mul_(weight)                                    # (a view of a multi-output operation would refuse this)
    assert loss.requires_grad


@pytest.mark.parametrize("k,r", [(2, 4), (3, 4), (2, 2)])
def test_unaffected_pairs_are_counted_with_ties_as_without(k, r):
    """Equal logits are ranked by index, so every token leaves C(E - k, r - k) subsets without change, ties or not."""
    E, T = 6, 200
    logits, Y = wl.make_enumeration_inputs(E, T, 64, "bf16", seed=9, device="cuda:0")
    logits[::7, 2] = logits[::7, 0]
    logits[1::7] = 0.5
    unaffected = pkg.prune_enumerate(logits, Y, k, r)[3]
    torch.cuda.synchronize()
    assert unaffected.item() == T * math.comb(E - k, r - k)
