"""GPU parity of the few-rows expert GEMMs and the one-workgroup dispatch, through the C ABI: the sizes at which their
tiles, splits and hand-overs end.  Tolerances are those of test_gpu_parity (each of h and the output is rounded to bf16
once); where two paths sum the same products in the same order the results are the same bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_14800_amd as pkg
from paper_2402_14800_amd import workloads as wl
from tests.test_gpu_parity import check_outputs, small_layer, to_dev

pytestmark = pytest.mark.gpu
NAMES = ("x", "Wgate", "W1", "W3", "W2")


def bits(t):
    return t.view(torch.int16)


@pytest.mark.parametrize("E,H,F,T,kept", [
    (8, 128, 192, 1, 0xff),            # one token; columns end inside a packed tile
    (8, 128, 192, 16, 0xff),
    (8, 576, 1024, 17, 0xff),          # a second group of 16 rows, an odd number of slice pairs
    (4, 4096, 64, 33, 0xf),            # eight wavefronts share a column group in one projection only
    (8, 64, 2112, 63, 0xff),           # one slice pair: no split
    (8, 256, 512, 47, 0b10000010),     # 47 rows for each of two experts
    (8, 128, 256, 192, 0xff),          # the last batch of the few-rows path, and the first beyond it
    (8, 128, 256, 193, 0xff),
    (32, 64, 128, 512, 0xffffffff),    # the same with many experts: eight tiles of 64 rows
    (32, 64, 128, 511, 0xffffffff),    # around the largest batch of the one-workgroup dispatch
    (32, 64, 128, 513, 0xffffffff),
])
def test_forward_with_few_rows_matches_oracle(E, H, F, T, kept):
    _, layer = small_layer("bf16", E, 2, H, F, T, index=21)
    if T in (192, 512):                # all tokens alike: two experts get T rows each, several tiles of 64 rows
        layer["x"][:] = layer["x"][0] * (1 + torch.arange(T)[:, None] % 3).to(layer["x"].dtype)
    d = to_dev(layer)
    beta = 0.6
    out, skip, lg, top2 = pkg.moe_forward_pruned_skip(*[d[n] for n in NAMES], kept, beta)
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    out_p, skip_p, lg_p, top2_p = pkg.moe_forward_pruned_skip_packed(d["x"], d["Wgate"], packed, F, beta, kept_mask=kept)
    torch.cuda.synchronize()
    assert torch.equal(bits(out), bits(out_p)) and torch.equal(skip, skip_p)
    assert torch.equal(lg, lg_p) and torch.equal(top2, top2_p)
    kept_set = [e for e in range(E) if kept >> e & 1]
    ref, ref_skip, e0, e1 = oracle.forward_skip(*[wl.to_f64(layer[n]) for n in NAMES], float(np.float32(beta)),
                                                logits=lg.cpu().numpy(), kept=kept_set)
    assert np.array_equal(skip.cpu().numpy().astype(bool), ref_skip)
    assert np.array_equal(top2.cpu().numpy(), np.stack([e0, e1], axis=1))
    check_outputs(wl.to_f64(out), ref, "out")


@pytest.mark.parametrize("E,H,F,T,k", [(16, 128, 192, 9, 4), (16, 192, 128, 512, 1), (16, 64, 128, 140, 16)])
def test_topk_forward_with_few_rows_matches_oracle(E, H, F, T, k):
    _, layer = small_layer("bf16", E, k, H, F, T, index=22)
    d = to_dev(layer)
    out, used, lg, experts = pkg.moe_forward_skip_topk(*[d[n] for n in NAMES], k, 0.1)
    torch.cuda.synchronize()
    ref, i_star, ids = oracle.forward_skip_topk(*[wl.to_f64(layer[n]) for n in NAMES], k, float(np.float32(0.1)),
                                                logits=lg.cpu().numpy())
    assert np.array_equal(used.cpu().numpy(), i_star) and np.array_equal(experts.cpu().numpy(), ids)
    check_outputs(wl.to_f64(out), ref, "out")


@pytest.mark.parametrize("E,H,F,T", [(8, 128, 192, 1), (3, 576, 320, 17), (8, 64, 64, 47), (20, 128, 64, 48), (5, 256, 512, 49), (4, 2048, 6144, 33)])
def test_expert_outputs_of_few_rows_are_those_of_many(E, H, F, T):
    """A token's expert outputs do not depend on the size of the batch, on who packed the weights, or on whether the
    rank-limited pass computed them: the products are summed in the same order everywhere."""
    _, layer = small_layer("bf16", E, 2, H, F, 300, index=23)
    d = to_dev(layer)
    many_lg, many = pkg.moe_expert_outputs(*[d[n] for n in NAMES])
    x = d["x"][:T].contiguous()
    lg, Y = pkg.moe_expert_outputs(x, *[d[n] for n in NAMES[1:]])
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    lg_p, Y_p = pkg.moe_expert_outputs_packed(x, d["Wgate"], packed, F)
    n = min(3, E)
    lg_r, experts, slot, Yr = pkg.moe_expert_outputs_ranked(x, *[d[n_] for n_ in NAMES[1:]], n)
    torch.cuda.synchronize()
    assert torch.equal(lg, many_lg[:T]) and torch.equal(lg_p, lg) and torch.equal(lg_r, lg)
    assert torch.equal(bits(Y), bits(many[:, :T].contiguous())) and torch.equal(bits(Y_p), bits(Y))
    t = torch.arange(T, device=Y.device)
    for j in range(n):
        assert torch.equal(bits(Yr[slot[:, j].long()]), bits(Y[experts[:, j].long(), t]))
    _, ref = oracle.expert_outputs(*[wl.to_f64(v) for v in (x, *[layer[n_] for n_ in NAMES[1:]])])
    check_outputs(wl.to_f64(Y), ref, "Y")


@pytest.mark.parametrize("E,H,F,T,n", [(2, 64, 64, 6144, 1), (2, 64, 64, 6145, 1), (3, 192, 448, 300, 2), (4, 320, 1088, 257, 4)])
def test_weights_in_place_give_the_bits_of_packed_weights(E, H, F, T, n):
    """Row-major weights read where they lie, at even and odd row counts and at column counts that end inside a tile (64, 192 and
    320 of 256 columns, 448 and 1088 of 128); the row count up to which that is done: the two tests below."""
    _, layer = small_layer("bf16", E, 2, H, F, T, index=24)
    d = to_dev(layer)
    ws = [d[n_] for n_ in NAMES]
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    lg, Y = pkg.moe_expert_outputs(*ws)
    lg_p, Y_p = pkg.moe_expert_outputs_packed(d["x"], d["Wgate"], packed, F)
    out, skip, _, _ = pkg.moe_forward_skip(*ws, 0.5)
    out_p, skip_p, _, _ = pkg.moe_forward_pruned_skip_packed(d["x"], d["Wgate"], packed, F, 0.5)
    _, experts, slot, Yr = pkg.moe_expert_outputs_ranked(*ws, n)
    torch.cuda.synchronize()
    assert torch.equal(lg, lg_p) and torch.equal(bits(Y), bits(Y_p))
    assert torch.equal(bits(out), bits(out_p)) and torch.equal(skip, skip_p)
    t = torch.arange(T, device=Y.device)
    for j in range(n):
        assert torch.equal(bits(Yr[slot[:, j].long()]), bits(Y[experts[:, j].long(), t]))


@pytest.mark.parametrize("E,H,F,T", [(2, 64, 64, 32768), (2, 64, 64, 32769), (1, 192, 320, 32768), (5, 64, 8256, 700)])
def test_whole_line_loads_of_weights_give_the_bits_of_packed_weights(E, H, F, T):
    """Weights read in units of two slices: at the row count up to which that is done, at K = 64 (a pair of slices per tile, so
    that the loader changes tile in every pair) with more tiles than compute units, and at column counts that end inside a
    unit (64 and 320 of 256 or 128 columns)."""
    _, layer = small_layer("bf16", E, 2, H, F, T, index=27)
    d = to_dev(layer)
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    _, Y = pkg.moe_expert_outputs(*[d[n] for n in NAMES])
    _, Y_p = pkg.moe_expert_outputs_packed(d["x"], d["Wgate"], packed, F)
    torch.cuda.synchronize()
    assert torch.equal(bits(Y), bits(Y_p))
    rows = torch.tensor([0, T // 2, T - 1])
    _, ref = oracle.expert_outputs(*[wl.to_f64(v) for v in (layer["x"][rows], *[layer[n] for n in NAMES[1:]])])
    check_outputs(wl.to_f64(Y[:, rows.to(Y.device)].contiguous()), ref, "Y")


@pytest.mark.parametrize("E,H,F,k", [(2, 64, 64, 2), (4, 192, 320, 3)])
def test_routed_weights_packed_inside_the_call_give_the_bits_of_weights_in_place(E, H, F, k):
    """The skipping forwards around the nominal 32768 rows per expert beyond which a call re-lays the weights out itself: the
    last batch that reads them in place, the first that does not, and that one on weights packed before."""
    last, last_k = 32768 * E // 2, 32768 * E // k           # tokens: 2 T and k T up to 32768 E
    _, layer = small_layer("bf16", E, 2, H, F, max(last, last_k) + 1, index=30)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    x, inside = d["x"][:last + 1].contiguous(), d["x"][:last].contiguous()

    def launches(call, *args):
        """The call's outputs, and how often it packed weights."""
        pkg.kernel_timing_enable(True)
        pkg.kernel_timing_reset()
        got = call(*args)
        torch.cuda.synchronize()
        names = [name for name, _ in pkg.kernel_timing_records()]
        pkg.kernel_timing_enable(False)
        return (*got, names.count("pack_w"))

    out, skip, lg, _, packs = launches(pkg.moe_forward_skip, x, *rest, 0.6)
    out_i, skip_i, _, _, packs_i = launches(pkg.moe_forward_skip, inside, *rest, 0.6)
    out_k, used, lg_k, _, packs_k = launches(pkg.moe_forward_skip_topk, d["x"][:last_k + 1].contiguous(), *rest, k, 0.1)
    out_ki, used_i, _, _, packs_ki = launches(pkg.moe_forward_skip_topk, d["x"][:last_k].contiguous(), *rest, k, 0.1)
    out_p, skip_p, _, _ = pkg.moe_forward_pruned_skip_packed(x, d["Wgate"], packed, F, 0.6)
    torch.cuda.synchronize()
    assert (packs, packs_i, packs_k, packs_ki) == (2, 0, 2, 0)      # W1 with W3, and W2
    assert torch.equal(bits(out), bits(out_p)) and torch.equal(skip, skip_p)
    assert torch.equal(bits(out[:last]), bits(out_i)) and torch.equal(skip[:last], skip_i)
    assert torch.equal(bits(out_k[:last_k]), bits(out_ki)) and torch.equal(used[:last_k], used_i)
    rows = torch.tensor([0, last // 3, last - 1, last])
    few = [wl.to_f64(v) for v in (layer["x"][rows], *[layer[n] for n in NAMES[1:]])]
    ref, _, _, _ = oracle.forward_skip(*few, float(np.float32(0.6)), logits=lg[rows.to(lg.device)].cpu().numpy())
    check_outputs(wl.to_f64(out[rows.to(out.device)].contiguous()), ref, "out")
    rows = torch.tensor([0, last_k // 3, last_k - 1, last_k])
    few[0] = wl.to_f64(layer["x"][rows])
    ref, _, _ = oracle.forward_skip_topk(*few, k, float(np.float32(0.1)), logits=lg_k[rows.to(lg_k.device)].cpu().numpy())
    check_outputs(wl.to_f64(out_k[rows.to(out_k.device)].contiguous()), ref, "out")


@pytest.mark.parametrize("E,H,F,T,prefixes,grouped_crosses", [
    (1, 64, 64, 32769, (32768, 16384, 100), True),        # 129 tiles against 128
    (2, 320, 192, 8193, (8192, 4096, 100), False),
    (4, 576, 448, 12000, (8000, 5000, 300), True),        # several experts and N tiles, the last of them ragged in both widths
    (7, 320, 832, 18000, (9000, 2000, 400), True),
])
def test_half_width_tiles_give_the_bits_of_full_width_tiles(E, H, F, T, prefixes, grouped_crosses):
    """Launches of more than 128 full-width tiles walk those, smaller ones tiles of half the width: the rows that both batches
    hold are the same bits, dense and through the tile order of the routed pass."""
    _, layer = small_layer("bf16", E, 2, H, F, T, index=26)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    _, many = pkg.moe_expert_outputs(d["x"], *rest)
    _, experts, slot, Yr = pkg.moe_expert_outputs_ranked(d["x"], *rest, 1)
    torch.cuda.synchronize()

    def full_width(rows):
        """Whether the (gate/up, down) launches of the dense and of the routed pass take full-width tiles."""
        of_expert = np.bincount(experts[:rows, 0].cpu().numpy(), minlength=E)
        m_tiles = E * -(-rows // 256), int(sum(-(-c // 256) for c in of_expert))
        return [tuple(m * -(-n // cols) > 128 for n, cols in ((F, 128), (H, 256))) for m in m_tiles]

    widths = [full_width(rows) for rows in (T, *prefixes)]
    for launch in (0, 1):                                  # gate/up, down
        assert {w[0][launch] for w in widths} == {True, False}
        assert not grouped_crosses or {w[1][launch] for w in widths} == {True, False}
    for rows in prefixes:
        x = d["x"][:rows].contiguous()
        _, Y = pkg.moe_expert_outputs(x, *rest)
        _, experts_s, slot_s, Yr_s = pkg.moe_expert_outputs_ranked(x, *rest, 1)
        torch.cuda.synchronize()
        assert torch.equal(bits(Y), bits(many[:, :rows].contiguous()))
        assert torch.equal(experts_s, experts[:rows])
        assert torch.equal(bits(Yr_s[slot_s[:, 0].long()]), bits(Yr[slot[:rows, 0].long()]))
        t = torch.arange(rows, device=Y.device)
        assert torch.equal(bits(Yr_s[slot_s[:, 0].long()]), bits(Y[experts_s[:, 0].long(), t]))


@pytest.mark.parametrize("E,H,F", [(8, 1024, 2048), (4, 2112, 576), (8, 128, 4160)])
def test_forward_bits_do_not_depend_on_the_batch(E, H, F):
    """Decoded alone, in a batch or as part of a prompt, a token has the same output: its products are summed over K in one
    order on every path.  k T of 48 E is the last batch of the few-rows path; the reference batch is beyond it."""
    T = 24 * E + 100
    _, layer = small_layer("bf16", E, 2, H, F, T, index=29)
    d = to_dev(layer)
    x, rest = d["x"], [d[n] for n in NAMES[1:]]
    packed = pkg.moe_pack_weights(*rest[1:])
    beta, k = 0.6, min(3, E)
    out, skip, _, _ = pkg.moe_forward_skip(x, *rest, beta)
    out_k, used, _, _ = pkg.moe_forward_skip_topk(x, *rest, k, 0.1)
    torch.cuda.synchronize()
    for t0, rows in ((0, 1), (7, 1), (3, 4), (5, 17), (0, 48), (0, 16 * E), (0, 16 * E + 1), (0, 24 * E), (0, 24 * E + 1)):
        part = x[t0:t0 + rows].contiguous()
        want, want_k = bits(out[t0:t0 + rows]), bits(out_k[t0:t0 + rows])
        got, got_skip, _, _ = pkg.moe_forward_skip(part, *rest, beta)
        got_p, _, _, _ = pkg.moe_forward_pruned_skip_packed(part, rest[0], packed, F, beta)
        got_k, got_used, _, _ = pkg.moe_forward_skip_topk(part, *rest, k, 0.1)
        torch.cuda.synchronize()
        assert torch.equal(got_skip, skip[t0:t0 + rows]) and torch.equal(got_used, used[t0:t0 + rows])
        assert torch.equal(bits(got), want) and torch.equal(bits(got_p), want)
        assert torch.equal(bits(got_k), want_k)


def test_streamed_weights_give_the_bits_of_many_rows():
    """A layer whose launches read more than 192 MB of weights (402 and 201 MB here): they come past the caches, except where
    an expert has several tiles.  The reference is the 256-row path on a larger batch."""
    E, H, F, T = 8, 2048, 6144, 300
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(31)

    def normal(*shape, std):
        return torch.randn(shape, generator=gen, device="cuda:0").mul_(std).to(torch.bfloat16)

    x = normal(T, H, std=1.0)
    x[64:128] = x[0]                    # one pair of experts has several tiles
    rest = [normal(E, H, std=H ** -0.5), normal(E, F, H, std=H ** -0.5), normal(E, F, H, std=H ** -0.5), normal(E, H, F, std=F ** -0.5)]
    packed = pkg.moe_pack_weights(*rest[1:])
    out, _, _, _ = pkg.moe_forward_skip(x, *rest, 0.5)
    _, Y = pkg.moe_expert_outputs(x, *rest)
    torch.cuda.synchronize()
    for rows in (5, 48, 128, 129):      # (128: the last batch of the few-rows path for a layer that no cache holds)
        part = x[:rows].contiguous()
        got, _, _, _ = pkg.moe_forward_skip(part, *rest, 0.5)
        got_p, _, _, _ = pkg.moe_forward_pruned_skip_packed(part, rest[0], packed, F, 0.5)
        torch.cuda.synchronize()
        assert torch.equal(bits(got), bits(out[:rows])) and torch.equal(bits(got_p), bits(out[:rows]))
    part = x[:33].contiguous()
    _, Y_r = pkg.moe_expert_outputs(part, *rest)
    _, Y_p = pkg.moe_expert_outputs_packed(part, rest[0], packed, F)
    torch.cuda.synchronize()
    assert torch.equal(bits(Y_r), bits(Y[:, :33].contiguous())) and torch.equal(bits(Y_p), bits(Y_r))


@pytest.mark.parametrize("E,H,F,T,kept,rows", [
    (4, 128, 320, 300, 0b0011, 300),       # every kept expert gets all 300 rows: two tiles of 192 for two of 256
    (3, 64, 192, 384, 0b0101, 384),        # two full tiles of 192
    (3, 64, 192, 385, 0b0101, 385),        # three of 192 against two of 256: 256
    (2, 192, 448, 129, 0b11, 129),         # one tile of 192 rows
    (2, 192, 448, 128, 0b11, 128),         # one of 128
    (2, 64, 64, 192, 0b11, 192),
    (2, 64, 64, 193, 0b11, 193),           # one of 256
    (2, 128, 320, 2300, 0b11, 2300),       # 12 tiles of 192 for 9 of 256, by the three-kernel dispatch
    (6, 64, 8256, 800, 0b101011, 0),       # more tiles than compute units
])
def test_short_tiles_give_the_bits_of_full_ones(E, H, F, T, kept, rows):
    """Routed launches whose tiles are 256, 192 or 128 rows tall, without skipping, in place and on packed weights: the same
    bits as the token's rows in a batch whose experts fill 256-row tiles, and as the dense pass of the same rows."""
    _, layer = small_layer("bf16", E, 2, H, F, 6144, index=28)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    out_many, _, _, _ = pkg.moe_forward_skip(d["x"], *rest, 0.0, kept_mask=kept)
    x = d["x"][:T].contiguous()
    out, _, _, top = pkg.moe_forward_skip(x, *rest, 0.0, kept_mask=kept)
    out_p, _, _, _ = pkg.moe_forward_pruned_skip_packed(x, d["Wgate"], packed, F, 0.0, kept_mask=kept)
    _, Y = pkg.moe_expert_outputs(x, *rest)
    _, Y_many = pkg.moe_expert_outputs(d["x"], *rest)
    torch.cuda.synchronize()
    if rows:                               # what the routing was made to give
        counts = np.bincount(top.cpu().numpy().reshape(-1), minlength=E)
        assert all(counts[e] == (rows if kept >> e & 1 else 0) for e in range(E))
    assert torch.equal(bits(out), bits(out_many[:T].contiguous())) and torch.equal(bits(out_p), bits(out))
    assert torch.equal(bits(Y), bits(Y_many[:, :T].contiguous()))
    pick = torch.tensor([0, T // 2, T - 1])
    _, ref = oracle.expert_outputs(*[wl.to_f64(v) for v in (layer["x"][pick], *[layer[n] for n in NAMES[1:]])])
    check_outputs(wl.to_f64(Y[:, pick.to(Y.device)].contiguous()), ref, "Y")


@pytest.mark.parametrize("rounds", [5, 9])
def test_a_partly_filled_last_round_takes_no_longer_than_a_full_one(rounds):
    """The persistent workgroups of the 256-row GEMM line up after every fourth tile.  Where some have their last tile just then,
    the others wait for the arrivals of that line-up only: with fewer tiles in the last round a launch is not slower."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("tile counts for 256 compute units")
    E, H, T = 8, 512, 1024                 # 4 row tiles of 8 experts: 32 gate/up tiles per 128 columns, 8 columns of them a round

    def gate_up_ms(columns):
        F = 128 * columns
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(41)
        x, Wg, W1, W3, W2 = (torch.randn(s, generator=gen, device="cuda:0").mul_(0.05).to(torch.bfloat16)
                             for s in ((T, H), (E, H), (E, F, H), (E, F, H), (E, H, F)))
        pkg.kernel_timing_enable(True)
        pkg.kernel_timing_reset()
        for _ in range(12):
            pkg.moe_expert_outputs(x, Wg, W1, W3, W2)
        torch.cuda.synchronize()
        ms = [t for name, t in pkg.kernel_timing_records() if name == "gemm_gate_up_swiglu"]
        pkg.kernel_timing_enable(False)
        assert len(ms) == 12
        return min(ms)

    assert gate_up_ms(8 * rounds - 6) <= 1.05 * gate_up_ms(8 * rounds)


@pytest.mark.parametrize("H,F,T", [
    (1024, 5504, 600),        # gate/up: 6 x 43 tiles, one round of 256 and 2 tiles as 4 of half the width
    (1024, 5440, 600),        # the same with 85 half-width columns: the last tile's second half has none
    (1088, 8192, 600),        # 384 tiles: the most that are halved
    (1024, 8256, 600),        # 390: none
    (11008, 1024, 600),       # down: 6 x 43 tiles
    (960, 5504, 600),         # few K steps: none
    (1024, 16576, 385),       # 4 x 130 tiles, three rounds
])
def test_a_last_round_of_half_width_tiles_gives_the_same_bits(H, F, T):
    """Routed launches whose last round has 1 to 128 tiles walk those as twice as many of half the width: the bits of the same
    rows in a batch without such a round and of the dense pass, row-major and packed weights, scaled and plain rows."""
    E = 2
    _, layer = small_layer("bf16", E, 2, H, F, T, index=33)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    packed = pkg.moe_pack_weights(d["W1"], d["W3"], d["W2"])
    out, skip, _, _ = pkg.moe_forward_skip(d["x"], *rest, 0.6)
    out_all, _, _, _ = pkg.moe_forward_skip(d["x"], *rest, 0.0)                     # every expert gets all T rows
    out_p, _, _, _ = pkg.moe_forward_pruned_skip_packed(d["x"], d["Wgate"], packed, F, 0.0)
    _, experts, slot_of, Yr = pkg.moe_expert_outputs_ranked(d["x"], *rest, E)
    _, Y = pkg.moe_expert_outputs(d["x"], *rest)
    part = d["x"][:190].contiguous()
    few, few_skip, _, _ = pkg.moe_forward_skip(part, *rest, 0.6)
    few_all, _, _, _ = pkg.moe_forward_skip(part, *rest, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(bits(out_all), bits(out_p)) and torch.equal(skip[:190], few_skip)
    assert torch.equal(bits(out[:190].contiguous()), bits(few)) and torch.equal(bits(out_all[:190].contiguous()), bits(few_all))
    rows = Yr[slot_of.reshape(-1).long()].reshape(T, E, H)                          # [token, rank]
    want = Y.permute(1, 0, 2)[torch.arange(T, device=Y.device)[:, None], experts.long()]
    assert torch.equal(bits(rows.contiguous()), bits(want.contiguous()))


@pytest.mark.parametrize("E,H,F,T", [
    (8, 64, 64, 1024), (8, 64, 64, 1025),      # the largest batch of the one-workgroup dispatch, and the next
    (32, 64, 192, 1024), (32, 64, 192, 2049),  # all experts, several routing blocks
    (32, 64, 64, 512), (32, 64, 64, 513),      # with 32 experts
    (8, 64, 16192, 1000), (8, 64, 16256, 1000),  # 16 tiles of 127 + 1 columns, the most entries of tile order, and more
    (8, 64, 64, 65536), (8, 64, 64, 65537),    # the most routing blocks whose counts every workgroup adds up, and one more
])
def test_dispatch_gives_every_token_its_experts(E, H, F, T):
    """Around the hand-overs of the dispatch: tokens at both ends and in the middle of the batch get the bits that they get in a
    batch of their own, by the top-2 rule and by the generalised one, and every rank its row in the rank-limited pass."""
    _, layer = small_layer("bf16", E, 3, H, F, T, index=34)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    kept = (1 << E) - 1 - (2 if E > 4 else 0)
    out, skip, lg, top = pkg.moe_forward_skip(d["x"], *rest, 0.6, kept_mask=kept)
    out_k, used, _, experts = pkg.moe_forward_skip_topk(d["x"], *rest, 3, 0.1)
    _, ranked, slot_of, Yr = pkg.moe_expert_outputs_ranked(d["x"], *rest, 3)
    for t0 in (0, T // 2 - 100, T - 200):
        part = d["x"][t0:t0 + 200].contiguous()
        o, s, _, e = pkg.moe_forward_skip(part, *rest, 0.6, kept_mask=kept)
        o_k, u, _, e_k = pkg.moe_forward_skip_topk(part, *rest, 3, 0.1)
        _, Y = pkg.moe_expert_outputs(part, *rest)
        torch.cuda.synchronize()
        at = slice(t0, t0 + 200)
        assert torch.equal(s, skip[at]) and torch.equal(e, top[at]) and torch.equal(u, used[at]) and torch.equal(e_k, experts[at])
        assert torch.equal(bits(o), bits(out[at].contiguous())) and torch.equal(bits(o_k), bits(out_k[at].contiguous()))
        rows = Yr[slot_of[at].reshape(-1).long()].reshape(200, 3, H)
        want = Y.permute(1, 0, 2)[torch.arange(200, device=Y.device)[:, None], ranked[at].long()]
        assert torch.equal(bits(rows.contiguous()), bits(want.contiguous()))
    want = lg.masked_fill(~torch.tensor([bool(kept >> e & 1) for e in range(E)], device=lg.device), float("-inf"))
    assert torch.equal(torch.argsort(want, dim=1, descending=True, stable=True)[:, :2].to(torch.int32), top)
    assert torch.equal(torch.sort(slot_of.reshape(-1)).values, torch.arange(3 * T, dtype=torch.int32, device=lg.device))


@pytest.mark.parametrize("E,k", [(24, 8), (32, 16), (8, 8)])
def test_dispatch_of_many_slots_gives_every_token_its_experts(E, k):
    """256 tokens, the most that one workgroup dispatches with so many slots, and 257: every token as in a smaller batch."""
    _, layer = small_layer("bf16", E, k, 64, 64, 257, index=38)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    out, used, _, experts = pkg.moe_forward_skip_topk(d["x"], *rest, k, 0.1)
    for t0, t1 in ((0, 256), (1, 257), (100, 229)):
        o, u, _, e = pkg.moe_forward_skip_topk(d["x"][t0:t1].contiguous(), *rest, k, 0.1)
        torch.cuda.synchronize()
        assert torch.equal(u, used[t0:t1]) and torch.equal(e, experts[t0:t1]) and torch.equal(bits(o), bits(out[t0:t1].contiguous()))


@pytest.mark.parametrize("E,H,T,k", [(8, 64, 1, 2), (8, 1088, 16, 2), (17, 128, 15, 2), (32, 4160, 16, 2), (16, 192, 7, 1), (20, 320, 16, 4),
                                     (16, 64, 16, 5)])
def test_routing_with_the_router_in_one_launch_gives_the_same_bits(E, H, T, k):
    """Up to 16 tokens and 4 experts each are routed by the launch that computes their logits: everything as in a batch of 20."""
    _, layer = small_layer("bf16", E, k, H, 64, 20, index=37)
    d = to_dev(layer)
    rest = [d[n] for n in NAMES[1:]]
    x = d["x"][:T].contiguous()
    all_ = pkg.moe_forward_skip_topk(d["x"], *rest, k, 0.1)
    some = pkg.moe_forward_skip_topk(x, *rest, k, 0.1)
    two_all = pkg.moe_forward_skip(d["x"], *rest, 0.6)
    two = pkg.moe_forward_skip(x, *rest, 0.6, want_logits=False, want_top2=False)
    lg, experts, slot, Yr = pkg.moe_expert_outputs_ranked(x, *rest, k)
    _, Y = pkg.moe_expert_outputs(x, *rest)
    torch.cuda.synchronize()
    for a, b in zip(all_, some):
        assert torch.equal(a[:T], b)
    assert torch.equal(bits(two_all[0][:T].contiguous()), bits(two[0])) and torch.equal(two_all[1][:T], two[1])
    assert torch.equal(lg, some[2]) and torch.equal(experts, some[3])
    rows = Yr[slot.reshape(-1).long()].reshape(T, k, H)
    want = Y.permute(1, 0, 2)[torch.arange(T, device=Y.device)[:, None], experts.long()]
    assert torch.equal(bits(rows.contiguous()), bits(want.contiguous()))
