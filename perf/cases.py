"""The work a program has this library do, as timed cases over its public entry points.

Three kinds of work, told apart by a case's "kind":

  forward    one MoE layer served with dynamic skipping: the top-2 rule on the layer's own weights ("skip"), the
             same on weights packed once, as a serving loop keeps them ("packed"), and the generalised top-k rule
             ("topk").  T = 1 is one generated token; tens are a decoding batch; hundreds to tens of thousands a prompt.
  layer      pruning one layer: the outputs of every expert on the calibration tokens ("dense", "packed") or of each
             token's best-ranked experts only ("ranked"), the loss of every kept-expert subset for each r, the selection
             statistics and the calibrated skipping threshold.
  enumerate  the subset losses alone, on expert outputs that are already there.

Ranges: T 1 .. 65536, E 4 .. 32, H 64 .. 4096, F 64 .. 14336 (multiples of 64; the fp32 layers are small ones), bf16 and
fp32 storage.  Layer shapes are those of the benchmark's configurations, of the tests, or of the same ranges at random.
"""
import math

import torch

import paper_2402_14800_amd as pkg
from paper_2402_14800_amd import binding

DEV = "cuda:0"
MIXTRAL = dict(E=8, H=4096, F=14336)
MID = dict(E=8, H=1024, F=3584)
MANY = dict(E=16, H=2048, F=5632)


def _forward(name, api, T, dtype="bf16", k=2, beta=0.6, kept=-1, **shape):
    return dict(name=name, kind="forward", api=api, dtype=dtype, T=T, k=k, beta=beta, kept=kept, **shape)


def _layer(name, api, T, dtype="bf16", k=2, rs="6,4", n_rank=0, **shape):
    return dict(name=name, kind="layer", api=api, dtype=dtype, T=T, k=k, rs=rs, n_rank=n_rank, **shape)


def _enumerate(name, T, E, H, k, rs, dtype="bf16"):
    return dict(name=name, kind="enumerate", api="multi", dtype=dtype, T=T, E=E, H=H, F=0, k=k, rs=rs)


def listed():
    return [
        # one generated token of one sequence: latency, and the weights of one or two experts from memory
        _forward("decode_1", "packed", 1, **MIXTRAL),
        # a decoding batch through the layer as it is deployed after pruning to six experts
        _forward("decode_48_pruned", "packed", 48, kept=0b10110111, **MIXTRAL),
        # a ragged prompt through a layer whose weights are used where they lie (evaluation of a pruned layer)
        _forward("prompt_777", "skip", 777, **MIXTRAL),
        # the benchmark's skipping forward
        _forward("forward_32768", "skip", 32768, **MIXTRAL),
        # the generalised rule on the many-expert layer, an odd number of tokens
        _forward("topk_1001", "topk", 1001, k=4, beta=0.1, **MANY),
        # one calibration sequence of 2048 tokens, batch after batch on packed weights
        _layer("calibrate_2048", "packed", 2048, **MIXTRAL),
        # pruning a mid-sized layer in one call of each entry point
        _layer("prune_16384", "dense", 16384, **MID),
        # the same through the rank-limited pass, ragged
        _layer("ranked_4001", "ranked", 4001, n_rank=6, **MID),
        # the tiny fp32 layer: launches and latency
        _layer("tiny_f32_512", "dense", 512, dtype="f32", rs="2", E=4, H=64, F=128),
        # a small layer in fp32 storage, odd token count
        _layer("f32_1501", "dense", 1501, dtype="f32", E=8, H=512, F=1024),
        # a quarter of the paper's calibration set at the Mixtral width
        _enumerate("enumerate_65536", 65536, 8, 4096, 2, "6,4"),
        # thousands of subsets per token
        _enumerate("enumerate_16_experts", 65536, 16, 2048, 4, "8,12"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


# (E, k, r's): enumeration shapes from a handful of subsets to thousands
_SUBSETS = [(4, 2, "2"), (4, 2, "3,2"), (8, 2, "6,4"), (8, 2, "7"), (8, 3, "5"), (6, 2, "4"), (16, 4, "12"), (16, 4, "8"),
            (12, 3, "6"), (20, 2, "18"), (16, 2, "14,12"), (32, 2, "30")]


def draw(rng):
    while True:
        kind = rng.choice(["forward", "forward", "layer", "enumerate"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        if kind == "enumerate":
            E, k, rs = rng.choice(_SUBSETS)
            c = _enumerate("", _log(rng, 1, 65536), E, 64 * _log(rng, 1, 64), k, rs, dtype)
        else:
            shape = rng.choice([MIXTRAL, MIXTRAL, MID, MANY, None, None])
            if dtype == "f32" or shape is None:
                top = (16, 56) if dtype == "f32" else (64, 224)
                shape = dict(E=rng.choice([4, 8, 16, 32]), H=64 * _log(rng, 1, top[0]), F=64 * _log(rng, 1, top[1]))
            E = shape["E"]
            if kind == "forward":
                api = rng.choice(["skip", "topk"] if dtype == "f32" else ["skip", "packed", "packed", "topk"])
                k = rng.choice([2, 3, 4]) if api == "topk" else 2
                kept = -1
                if rng.random() < 0.3:
                    kept = sum(1 << e for e in rng.sample(range(E), max(k, 3 * E // 4)))
                c = _forward("", api, _log(rng, 1, 32768), dtype=dtype, k=k, beta=rng.choice([0.0, 0.1, 0.6]), kept=kept, **shape)
            else:
                api = "dense" if dtype == "f32" else rng.choice(["dense", "packed", "ranked"])
                k = 2 if E <= 8 else rng.choice([2, 4])
                rs = {4: "2", 8: "6,4", 16: "14,12", 32: "30"}[E]
                most = max(_active(E, k, r) for r in _rs(dict(rs=rs)))
                c = _layer("", api, _log(rng, 1, 16384), dtype=dtype, k=k, rs=rs, n_rank=most if api == "ranked" else 0, **shape)
        w = work(c)
        limit = (1.0e11, 1.0e9) if dtype == "f32" else (1.7e13, 4.4e9)
        if w["flops"] <= limit[0] and w["bytes"] <= limit[1]:
            del c["name"]
            return c


# ---------------------------------------------------------------- helpers
def _rs(case):
    return [int(r) for r in case["rs"].split(",")]


def _active(E, k, r):
    """Rank positions of a token that some pruned layer can select."""
    return min(E, min(k, r) + E - r)


def _kept(case):
    return (1 << case["E"]) - 1 if case["kept"] < 0 else case["kept"]


def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _inputs(case, seed):
    """x with rows of unit RMS and weights of the usual initialisation (logits of about unit variance)."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    E, H, F, T, dt = case["E"], case["H"], case["F"], case["T"], _dt(case)

    def normal(*shape, std=1.0):
        return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).mul_(std)

    x = normal(T, H)
    x = (x / x.pow(2).mean(dim=1, keepdim=True).sqrt()).to(dt)
    out = dict(x=x, Wgate=normal(E, H, std=H ** -0.5).to(dt))
    for n, shape, std in (("W1", (F, H), H ** -0.5), ("W3", (F, H), H ** -0.5), ("W2", (H, F), F ** -0.5)):
        w = torch.empty((E, *shape), dtype=dt, device=DEV)
        for e in range(E):
            w[e] = normal(*shape, std=std).to(dt)
        out[n] = w
    return out


def _enumeration_inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    T, E, H = case["T"], case["E"], case["H"]
    logits = torch.randn((T, E), generator=gen, device=DEV) + 0.5 ** 0.5 * torch.randn((E,), generator=gen, device=DEV)
    Y = torch.empty((E, T, H), dtype=_dt(case), device=DEV)
    for e in range(E):
        Y[e] = torch.randn((T, H), generator=gen, device=DEV).to(_dt(case))
    return logits, Y


def _buffer(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


# ---------------------------------------------------------------- the cases' life
def prepare(case, seed):
    c, T, E, H, F, k = case, case["T"], case["E"], case["H"], case["F"], case["k"]
    code = binding.MOEP_F32 if c["dtype"] == "f32" else binding.MOEP_BF16
    st = {"case": case}
    if c["kind"] == "enumerate":
        st["logits"], st["Y"] = _enumeration_inputs(c, seed)
        st["ws"] = _buffer(binding.prune_enumerate_multi_workspace(T, E, H, k, _rs(c), code))
        return st
    st.update(_inputs(c, seed))
    lib = binding._lib
    if c["api"] == "packed":                      # a serving or calibration loop keeps the packed copy only
        st["packed"] = pkg.moe_pack_weights(st["W1"], st["W3"], st["W2"])
        del st["W1"], st["W3"], st["W2"]
    if c["kind"] == "forward":
        st["ws"] = _buffer(lib.moe_forward_skip_topk_workspace(T, E, H, F, code, k) if c["api"] == "topk"
                           else binding.moe_forward_skip_workspace(T, E, H, F, code))
        return st
    st["ws"] = _buffer({"dense": lambda: binding.moe_expert_outputs_workspace(T, E, H, F, code),
                        "packed": lambda: lib.moe_expert_outputs_packed_workspace(T, E, H, F, code),
                        "ranked": lambda: lib.moe_expert_outputs_ranked_workspace(T, E, H, F, code, c["n_rank"])}[c["api"]]())
    st["ws_enum"] = _buffer(max(binding.prune_enumerate_multi_workspace(T, E, H, k, _rs(c), code), 1))
    st["ws_beta"] = _buffer(lib.skip_calibrate_beta_workspace(T))
    return st


def _losses(results):
    return [dict(loss=loss, argmin=a, mask=m, unaffected=u) for loss, a, m, u in results]


def run(st):
    c = st["case"]
    k = c["k"]
    if c["kind"] == "enumerate":
        return _losses(pkg.prune_enumerate_multi(st["logits"], st["Y"], k, _rs(c), workspace=st["ws"]))
    if c["kind"] == "forward":
        if c["api"] == "packed":
            out, skip, logits, top = pkg.moe_forward_pruned_skip_packed(st["x"], st["Wgate"], st["packed"], c["F"], c["beta"],
                                                                        kept_mask=_kept(c), workspace=st["ws"])
        elif c["api"] == "skip":
            out, skip, logits, top = pkg.moe_forward_pruned_skip(st["x"], st["Wgate"], st["W1"], st["W3"], st["W2"], _kept(c),
                                                                 c["beta"], workspace=st["ws"])
        else:
            out, skip, logits, top = pkg.moe_forward_skip_topk(st["x"], st["Wgate"], st["W1"], st["W3"], st["W2"], k, c["beta"],
                                                               kept_mask=_kept(c), workspace=st["ws"])
        return dict(out=out, kept=skip, logits=logits, experts=top)
    r = {}
    if c["api"] == "ranked":
        logits, experts, slot_of, Y = pkg.moe_expert_outputs_ranked(st["x"], st["Wgate"], st["W1"], st["W3"], st["W2"],
                                                                    c["n_rank"], workspace=st["ws"])
        r.update(experts=experts, slot_of=slot_of)
        losses = [pkg.prune_enumerate_ranked(logits, experts, slot_of, Y, k, rr, workspace=st["ws_enum"]) for rr in _rs(c)]
    else:
        if c["api"] == "packed":
            logits, Y = pkg.moe_expert_outputs_packed(st["x"], st["Wgate"], st["packed"], c["F"], workspace=st["ws"])
        else:
            logits, Y = pkg.moe_expert_outputs(st["x"], st["Wgate"], st["W1"], st["W3"], st["W2"], workspace=st["ws"])
        losses = pkg.prune_enumerate_multi(logits, Y, k, _rs(c), workspace=st["ws_enum"])
    count, co, often = pkg.expert_selection_stats(logits, k, _rs(c)[0])
    beta = pkg.skip_calibrate_beta(logits, workspace=st["ws_beta"])
    r.update(logits=logits, Y=Y, losses=_losses(losses), count=count, co=co, often=often, beta=beta)
    return r


def work(case):
    c, T, E, H, F = case, case["T"], case["E"], case["H"], case["F"]
    es = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "forward":
        kept = bin(_kept(c)).count("1")
        share = 1.0 if c["beta"] == 0.0 else 0.75        # of a token's k routed slots, about
        slots = max(1.0, c["k"] * share) * T
        hit = kept * (1.0 - (1.0 - 1.0 / kept) ** slots)  # experts that some slot is routed to, expected
        return {"bytes": hit * 3 * H * F * es + 2.0 * T * H * es + E * H * es + 4.0 * T * E,
                "flops": 6.0 * H * F * slots + 2.0 * T * E * H}
    subsets = sum(math.comb(E, r) for r in _rs(c))
    scoring = 2.0 * T * sum(math.comb(_active(E, c["k"], r), min(c["k"], r)) for r in _rs(c)) + 1.0 * T * subsets
    per_token = c.get("n_rank") or E
    gram = 1.0 * T * per_token * (per_token + 1) * H
    if c["kind"] == "enumerate":
        return {"bytes": 1.0 * T * E * H * es + 4.0 * T * E + 4.0 * subsets, "flops": gram + scoring}
    return {"bytes": 3.0 * E * H * F * es + 1.0 * T * H * es + 1.0 * per_token * T * H * es + 4.0 * T * E,
            "flops": 6.0 * H * F * per_token * T + 2.0 * T * E * H + gram + scoring}


def tolerance(case):
    # Four times what is seen against 64 bits, and rounded up.  bf16: every product is exact and summed in fp32, but the
    # SwiGLU product and the result are rounded to bf16 once each: 2.3e-3.  fp32 storage: fp32 sums of up to a few
    # thousand products, 1e-6.  Losses on given expert outputs: 8e-8 over thousands of tokens, more where T is 1 and
    # nothing averages.  Whole values: a token whose two best logits differ by one rounding.
    if case["kind"] == "enumerate":
        return {"rel": 4e-6, "max": 4e-5, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4, "differ": 1e-4}
    return {"rel": 1e-2, "max": 0.3, "differ": 1e-4}


# ---------------------------------------------------------------- the same in 64 bits
def _experts64(x, W1, W3, W2):
    g = x @ W1.double().t()
    return (torch.nn.functional.silu(g) * (x @ W3.double().t())) @ W2.double().t()


def _masks(E, r):
    import itertools

    m = torch.zeros((math.comb(E, r), E), dtype=torch.bool)
    for i, t in enumerate(itertools.combinations(range(E), r)):
        m[i, list(t)] = True
    return m.to(DEV)


def _mask_int(row):
    v = sum(1 << e for e, b in enumerate(row.tolist()) if b)
    return torch.tensor([v - (1 << 32) if v >= 1 << 31 else v], dtype=torch.int32)


def _loss64(logits, gram, E, k, r):
    """Subset losses from the logits and the tokens' Gram matrices, with the argmin, its mask and the unaffected pairs."""
    T = logits.shape[0]
    n, kk = _active(E, k, r), min(k, r)
    order = torch.argsort(logits, dim=1, descending=True, stable=True)
    top = order[:, :n]
    lr = torch.gather(logits, 1, order)[:, :n]
    g = torch.gather(torch.gather(gram, 1, top[:, :, None].expand(T, n, E)), 2, top[:, None, :].expand(T, n, n)).contiguous()
    a = torch.zeros((T, n), dtype=torch.float64, device=DEV)
    a[:, :k] = torch.softmax(lr[:, :k], dim=1) if k <= n else 0.0
    first = torch.arange(n, device=DEV) < k
    masks = _masks(E, r)
    loss = torch.zeros(len(masks), dtype=torch.float64, device=DEV)
    same = 0
    chunk = max(1, min(len(masks), (1 << 24) // max(1, T * n)))
    for s0 in range(0, len(masks), chunk):
        kept = masks[s0:s0 + chunk].t().contiguous()[top]                  # [T, n, subsets]
        taken = kept & (torch.cumsum(kept, dim=1, dtype=torch.int32) <= kk)
        same += int((taken == first[None, :, None]).all(dim=1).sum())
        d = torch.softmax(lr[:, :, None].masked_fill(~taken, -math.inf), dim=1) - a[:, :, None]
        loss[s0:s0 + chunk] = (d * torch.bmm(g, d)).sum(dim=(0, 1))
    best = int(torch.argmin(loss))
    return dict(loss=loss, argmin=torch.tensor([best], dtype=torch.int32), mask=_mask_int(masks[best].cpu()),
                unaffected=torch.tensor([same], dtype=torch.int64))


def _gram64(Y):
    E, T, H = Y.shape
    gram = torch.empty((T, E, E), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // (E * H))
    for t0 in range(0, T, step):
        y = Y[:, t0:t0 + step].double().transpose(0, 1).contiguous()
        gram[t0:t0 + step] = torch.bmm(y, y.transpose(1, 2).contiguous())
    return gram


def _best_two_ratio(logits):
    v = torch.topk(logits, 2, dim=1).values
    s = torch.sort(torch.exp(v[:, 1] - v[:, 0])).values
    T = s.numel()
    return (0.5 * (s[(T - 1) // 2] + s[T // 2])).reshape(1)


def exact(case, seed):
    c, T, E, H, k = case, case["T"], case["E"], case["H"], case["k"]
    if c["kind"] == "enumerate":
        logits, Y = _enumeration_inputs(c, seed)
        gram = _gram64(Y)
        return [_loss64(logits.double(), gram, E, k, r) for r in _rs(c)]
    w = _inputs(c, seed)
    x = w["x"].double()
    logits = x @ w["Wgate"].double().t()
    if c["kind"] == "forward":
        keep = torch.tensor([bool(_kept(c) >> e & 1) for e in range(E)], device=DEV)
        order = torch.argsort(logits.masked_fill(~keep, -math.inf), dim=1, descending=True, stable=True)[:, :k]
        lv = torch.gather(logits, 1, order)
        p = torch.softmax(lv, dim=1)
        if c["api"] == "topk":
            tail = p.sum(dim=1, keepdim=True) - torch.cumsum(p, dim=1)      # weights beyond the i-th
            stay = torch.cumsum((tail <= c["beta"] + 1e-15).int(), dim=1) <= 1
            stay[:, 1:] &= ~(tail[:, :-1] <= c["beta"] + 1e-15)
            used = stay.sum(dim=1).to(torch.int32)
        else:
            stay = torch.ones_like(p, dtype=torch.bool)
            if c["beta"] > 0.0:
                stay[:, 1] = ~(lv[:, 1] - lv[:, 0] < math.log(c["beta"]))
            used = (~stay[:, 1]).to(torch.uint8)
        p = torch.where(stay, p, torch.zeros_like(p))
        p = p / p.sum(dim=1, keepdim=True)
        out = torch.zeros((T, H), dtype=torch.float64, device=DEV)
        for e in range(E):
            t, m = torch.nonzero((order == e) & stay, as_tuple=True)
            if t.numel():
                out.index_add_(0, t, p[t, m][:, None] * _experts64(x[t], w["W1"][e], w["W3"][e], w["W2"][e]))
        return dict(out=out, kept=used, logits=logits, experts=order.to(torch.int32))
    Y = torch.stack([_experts64(x, w["W1"][e], w["W3"][e], w["W2"][e]) for e in range(E)])
    gram = _gram64(Y)
    order = torch.argsort(logits, dim=1, descending=True, stable=True)
    r = {}
    if c["api"] == "ranked":
        n = c["n_rank"]
        experts = order[:, :n].contiguous()
        rows = torch.argsort((experts * T + torch.arange(T, device=DEV)[:, None]).reshape(-1))   # by expert, then token
        slot = torch.empty_like(rows)
        slot[rows] = torch.arange(rows.numel(), device=DEV)
        Y = Y[experts.reshape(-1)[rows], rows // n]
        r.update(experts=experts.to(torch.int32), slot_of=slot.reshape(T, n).to(torch.int32))
    chosen = torch.zeros((T, E), dtype=torch.float64, device=DEV)
    chosen.scatter_(1, order[:, :k], 1.0)
    co = (chosen.t() @ chosen).round().to(torch.int64)
    count = torch.diagonal(co).contiguous()
    often = torch.zeros(E, dtype=torch.bool)
    often[torch.argsort(count, descending=True, stable=True)[:_rs(c)[0]].cpu()] = True
    r.update(logits=logits, Y=Y, losses=[_loss64(logits, gram, E, k, rr) for rr in _rs(c)], count=count, co=co,
             often=_mask_int(often), beta=_best_two_ratio(logits))
    return r
