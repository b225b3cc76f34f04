"""Workloads of the library as a user's program runs them, through the public entry points.

A case belongs to one of five families:

``layer``    one pass of the sparse FFN path: compact the predicted block mask, mask the shares of
             both operands of every projection, open them, and compute the output shares of Eq. 1.
             ``parties`` = 2 plays both parties in one process (as the benchmark does); 1 is one
             party's own device, which holds what the other party sent.  ``form`` says how the
             weight side travels: ``planes`` (digit planes, SOMM weights one row per neuron, the
             products that are ready together in one grouped call), ``words`` (row-major words,
             one call per product, results allocated by the call) or ``unopened`` (decoding, at
             most eight rows: the opening of F is folded into the share call).
``general``  per-token masks of a batch of unrelated requests: component search and the share on
             the result blocks (Protocol 2), then the share with per-token row sets (Protocol 3).
``mha``      the attention shape: QKV product of the current tokens and the merged cache-refill
             rows with head-granular masks, then the output layer with per-token head sets.
``glue``     the local steps around the products: two steps of the oblivious shuffle, the rescaling
             of a fixed-point product and the merge of a compact result to the full width.
``compact``  the predictor's per-token flags to the ordered list of active blocks.

Shares, triple parts and masked values are uniform over Z_{2^64} whatever the secrets are, so all
of them are drawn as uniform words.  Every output is an integer and has to be exact.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2505_07239_amd as comet
from workloads import configs, masks

# Two products per party (Eq. 1 with E and A stacked), and per 64-bit multiply-add 36 products of
# signed base-256 digits, two operations each: the fewest exact int8 operations a word product takes.
INT8_OPS_PER_MAC = 72


def listed():
    layer = dict(family="layer", mask="clustered", parties=2)
    return [
        # the smallest layer of the test configurations: a handful of microseconds of arithmetic,
        # so launches and host work are what a caller waits for
        dict(layer, name="tiny_layer", form="words", proj="up_down", tokens=16, d_model=64, d_ff=256, bs=16,
             density=0.25, mask="uniform"),
        # OPT-125m prompt of 128 tokens, one mask for the batch, 10 % of the blocks
        dict(layer, name="opt125m_prompt", form="planes", proj="up_down", tokens=128, d_model=768, d_ff=3072, bs=32,
             density=0.10),
        # LLaMA-7B prompt of 256 tokens, gated FFN, 15 % of the blocks: the benchmark's headline
        dict(layer, name="llama7b_prompt", form="planes", proj="gate_up_down", tokens=256, d_model=4096, d_ff=11008,
             bs=32, density=0.15),
        # down projection with every block kept, 512 tokens: the densest and largest product
        dict(layer, name="llama7b_down_dense", form="planes", proj="down", tokens=512, d_model=4096, d_ff=11008,
             bs=32, density=1.0),
        # a decoding batch of eight tokens with a mask each, both parties: reads nearly all weights
        dict(layer, name="llama13b_decode", form="unopened", proj="gate_up_down", tokens=8, d_model=5120, d_ff=13824,
             bs=64, density=0.20, mask="per_token"),
        # one party's device generating one token at a time
        dict(layer, name="llama7b_one_token", form="unopened", proj="gate_up_down", tokens=1, d_model=4096,
             d_ff=11008, bs=32, density=0.15, parties=1),
        # one party's device serving a batch of 32 decoding requests that share a mask
        dict(layer, name="llama13b_batch32", form="planes", proj="gate_up_down", tokens=32, d_model=5120, d_ff=13824,
             bs=64, density=0.20, parties=1),
        # a prompt of odd length through a model of odd widths, weights as plain words, one call per
        # product: nothing is a multiple of a tile and no row starts on 16 bytes
        dict(layer, name="odd_sizes_words", form="words", proj="up_down", tokens=77, d_model=1001, d_ff=2730, bs=21,
             density=0.30, parties=1),
        # four unrelated requests of 64 tokens in one batch, every token with its own mask
        dict(family="general", name="four_requests", form="words", tokens=256, groups=4, d_model=4096, d_ff=11008,
             bs=32, density=0.15),
        # LLaMA-2-7B attention: 8 decoding tokens and 56 merged cache-refill rows, half of the heads
        dict(family="mha", name="llama7b_heads", d_model=4096, n_heads=32, head_dim=128, tokens=8, refill_rows=56,
             density=0.5),
        # shuffle, rescaling and merge of a prompt's activations at the FFN width
        dict(family="glue", name="shuffle_and_merge", rows=4096, cols=11008, bs=32, density=0.15),
        # element-granular flags of 4096 tokens at the FFN width
        dict(family="compact", name="token_flags", tokens=4096, blocks=13824, density=0.10),
    ]


# ---------------------------------------------------------------------------
# further cases of the same ranges
# ---------------------------------------------------------------------------

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_layer(rng, form):
    low, high = (1, 8) if form == "unopened" else (5, 512)
    c = dict(family="layer", form=form, tokens=_log(rng, low, high), parties=rng.choice((1, 2)),
             proj=rng.choice(("up", "down", "up_down", "gate_up_down")),
             mask=rng.choice(("uniform", "clustered", "per_token")),
             density=round(math.exp(rng.uniform(math.log(0.05), 0.0)), 3))
    # planes of a full-size triple share are gathered in units of sixteen rows
    c["bs"] = 16 * rng.randint(1, 8) if form == "planes" else rng.choice((1, 7, 8, 16, 21, 32, 64, 128))
    c["d_model"] = _log(rng, 64, 5120)
    c["d_ff"] = c["bs"] * max(2, _log(rng, 256, 13824) // c["bs"])
    c["density"] = max(c["density"], round(c["bs"] / c["d_ff"], 3))      # at least one block
    if rng.random() < 0.5:                       # half of the widths as models have them
        c["d_model"] = max(64, c["d_model"] // 64 * 64)
    return c


def _draw_general(rng):
    bs = 16 * rng.randint(1, 4)
    groups = rng.randint(2, 6)
    return dict(family="general", form=rng.choice(("words", "planes")), tokens=rng.randint(groups * 8, 400), groups=groups,
                d_model=_log(rng, 512, 5120), d_ff=bs * (_log(rng, 2048, 13824) // bs), bs=bs,
                density=round(rng.uniform(0.05, 0.9 / groups), 3))


def _draw_mha(rng):
    heads, dim = rng.randint(8, 40), rng.choice((64, 80, 128))
    return dict(family="mha", d_model=heads * dim, n_heads=heads, head_dim=dim, tokens=rng.randint(1, 16),
                refill_rows=rng.randint(0, 100), density=round(rng.uniform(0.2, 0.8), 2))


def _draw_glue(rng):
    bs = rng.choice((1, 16, 21, 32, 64))
    return dict(family="glue", rows=_log(rng, 8, 4096), cols=bs * max(2, _log(rng, 256, 20000) // bs), bs=bs,
                density=round(rng.uniform(0.05, 1.0), 3))


def _draw_compact(rng):
    return dict(family="compact", tokens=_log(rng, 1, 16384), blocks=_log(rng, 64, 262144),
                density=round(math.exp(rng.uniform(math.log(0.02), math.log(0.8))), 3))


def draw(rng):
    make = rng.choice((lambda r: _draw_layer(r, "planes"), lambda r: _draw_layer(r, "planes"),
                       lambda r: _draw_layer(r, "words"), lambda r: _draw_layer(r, "unopened"),
                       _draw_general, _draw_mha, _draw_glue, _draw_compact))
    largest = max(_seconds(c) for c in listed())
    while True:
        c = make(rng)
        if _seconds(c) <= largest and _state_bytes(c) < 16e9:
            return c


def _seconds(case):
    """A rough cost, to compare cases by."""
    w = work(case)
    return max(w["bytes"] / 5e12, w["flops"] / 2.5e15)


def _state_bytes(case):
    if case["family"] == "compact":
        return case["tokens"] * case["blocks"]
    if case["family"] == "glue":
        return 48 * case["rows"] * case["cols"]
    copies = len(_projections(case)) * 6 if case["family"] == "layer" else 6
    return 8 * case["d_model"] * (case["d_ff"] if case["family"] != "mha" else 3 * case["d_model"]) * copies


# ---------------------------------------------------------------------------
# states
# ---------------------------------------------------------------------------

class _Words:
    """Uniform words from a seed, drawn on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def __call__(self, *shape):
        return torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda", generator=self.gen)


def _projections(case):
    """(kind, ...) of the projections of a layer, in order."""
    return [("simm" if p == "down" else "somm") for p in case["proj"].split("_")]


def _empty(*shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda")


def _kept_blocks(case):
    """Active blocks of a layer case: exact for one mask, the expectation for the union of masks."""
    nb = case["d_ff"] // case["bs"]
    if case["mask"] != "per_token":
        return masks.kept_blocks(case["density"], nb)
    each = masks.kept_blocks(case["density"], nb) / nb
    return nb * (1.0 - (1.0 - each) ** case["tokens"])


def _layer_mask(case, seed):
    nb, density = case["d_ff"] // case["bs"], case["density"]
    if case["mask"] == "uniform":
        return masks.uniform_block_mask(seed, 1, nb, density)[None, :]
    if case["mask"] == "clustered":
        return masks.clustered_block_mask(seed, 1, nb, density)[None, :]
    return masks.per_token_masks(seed, 1, case["tokens"], nb, density, clustered=False)


def _prepare_layer(case, seed):
    words = _Words(seed)
    ctx = comet.Context(0)
    m, d, f, bs = case["tokens"], case["d_model"], case["d_ff"], case["bs"]
    both = case["parties"] == 2
    mine = (0, 1) if both else (1,)                       # the parties this process computes for
    planes, neuron_major = case["form"] == "planes", case["form"] == "planes"
    mask = _layer_mask(case, seed)
    n_blk = int(np.count_nonzero(mask.max(axis=0)))       # the sparsity level is public
    n_act = n_blk * bs
    products = []
    for kind in _projections(case):
        k, n = (d, f) if kind == "somm" else (f, d)
        nm = neuron_major and kind == "somm"
        wshape = (n, k) if nm else (k, n)
        if kind == "somm":
            dshape, gshape, zshape = (m, k), ((n_act, k) if nm else (k, n_act)), (m, n_act)
        else:
            dshape, gshape, zshape = (m, n_act), (n_act, n), (m, n)
        q = dict(kind=kind, nm=nm, x={}, a={}, y={}, b={}, bw={}, c={}, z={})
        for i in mine:
            q["x"][i], q["a"][i] = words(m, k), words(m, k)
            q["y"][i], q["b"][i] = words(*wshape), words(*wshape)
            q["c"][i], q["z"][i] = words(*zshape), _empty(*zshape)
            # the triple share is offline material: packed once
            q["bw"][i] = ctx.open_weight_planes(q["b"][i], neuron_major=nm) if planes else q["b"][i]
        # masked shares: this process writes its own; a single party holds what the other one sent
        q["d"] = {i: _empty(*dshape) if i in mine else words(*dshape) for i in (0, 1)}
        q["g"] = {i: _empty(*gshape) if i in mine else words(*gshape) for i in (0, 1)}
        q["e"] = _empty(*dshape)
        if planes:
            kf, nf = (gshape[1], gshape[0]) if nm else gshape
            size = comet.binding.load_library().comet_weight_planes_bytes(kf, nf)
            q["f"] = torch.empty(max(int(size), 16), dtype=torch.uint8, device="cuda")
        elif case["form"] == "words":
            q["f"] = _empty(*gshape)
        products.append(q)
    nb = f // bs
    return dict(case=case, ctx=ctx, mask=torch.from_numpy(mask).cuda(), mine=mine, n_blk=n_blk, products=products,
                idx=torch.zeros(nb, dtype=torch.int32, device="cuda"),
                n_dev=torch.zeros(1, dtype=torch.int32, device="cuda"))


def _run_layer(s):
    case, ctx, mine, bs = s["case"], s["ctx"], s["mine"], s["case"]["bs"]
    idx, n_dev, cap = s["idx"], s["n_dev"], s["n_blk"]
    ctx.compact_mask(s["mask"], idx, n_dev)
    outs = []
    for kind in ("somm", "simm"):
        group = [q for q in s["products"] if q["kind"] == kind]
        if not group:
            continue
        members, zs = [], []
        for q in group:
            for i in mine:
                if kind == "somm":
                    ctx.mask_share(q["x"][i], q["a"][i], out=q["d"][i])
                    ctx.mask_share_gather(q["y"][i], q["b"][i], comet.AXIS_ROWS if q["nm"] else comet.AXIS_COLS, bs,
                                          idx, n_dev, cap, out=q["g"][i])
                else:
                    ctx.mask_share_gather(q["x"][i], q["a"][i], comet.AXIS_COLS, bs, idx, n_dev, cap, out=q["d"][i])
                    ctx.mask_share_gather(q["y"][i], q["b"][i], comet.AXIS_ROWS, bs, idx, n_dev, cap, out=q["g"][i])
            ctx.open(q["d"][0], q["d"][1], out=q["e"])
            if case["form"] == "planes":
                f = ctx.open_weight_planes(q["g"][0], q["g"][1], out=q["f"], neuron_major=q["nm"])
                members += [(i, q["e"], f, q["a"][i], q["bw"][i], q["c"][i]) for i in mine]
                zs += [q["z"][i] for i in mine]
            elif case["form"] == "words":
                f = ctx.open(q["g"][0], q["g"][1], out=q["f"])
                call = ctx.somm_share if kind == "somm" else ctx.simm_share
                outs += [call(i, bs, idx, n_dev, cap, q["e"], f, q["a"][i], q["bw"][i], q["c"][i]) for i in mine]
            else:
                call = ctx.somm_share_unopened if kind == "somm" else ctx.simm_share_unopened
                outs += [call(i, bs, idx, n_dev, cap, q["e"], q["g"][0], q["g"][1], q["a"][i], q["bw"][i],
                              q["c"][i], out=q["z"][i]) for i in mine]
        if members:
            outs += ctx.share_group(kind, bs, idx, n_dev, cap, members, out=zs)
    sent = [q[t][i] for q in s["products"] for t in ("d", "g") for i in mine]
    return dict(shares=outs, sent=sent, blocks=idx[:cap], count=n_dev)


def _prepare_general(case, seed):
    words = _Words(seed)
    ctx = comet.Context(0)
    m, d, f, bs = case["tokens"], case["d_model"], case["d_ff"], case["bs"]
    nb = f // bs
    mask = masks.grouped_token_masks(seed, 1, m, nb, case["groups"], case["density"])
    n_blk, n_row = int(np.count_nonzero(mask.max(axis=0))), int(np.count_nonzero(mask.max(axis=1)))
    n_act = n_blk * bs
    # the opened operands and the triple shares of one party; rows and kept columns as listed
    s = dict(case=case, ctx=ctx, mask=torch.from_numpy(mask).cuda(), n_blk=n_blk, n_row=n_row,
             e=words(n_row, d), a=words(n_row, d), f=words(d, n_act), b=words(d, f), c=words(n_row, n_act),
             z=_empty(n_row, n_act), e2=words(m, n_act), a2=words(m, f), f2=words(n_act, d), b2=words(f, d),
             c2=words(m, d), z2=_empty(m, d))
    if case["form"] == "planes":
        for name in ("f", "b", "f2", "b2"):
            s[name] = ctx.open_weight_planes(s[name])
    return s


def _run_general(s):
    ctx, bs, cap = s["ctx"], s["case"]["bs"], s["n_blk"]
    comp = ctx.components(s["mask"])
    z = ctx.somm_share_blocks(1, bs, comp["blk_idx"], comp["blk_comp"], comp["n_blk"], cap, comp["row_comp"],
                              comp["n_row"], s["e"], s["f"], s["a"], s["b"], s["c"], out=s["z"])
    idx, n_dev = ctx.compact_mask(s["mask"])
    z2 = ctx.simm_share_masked(1, bs, idx, n_dev, cap, s["mask"], s["e2"], s["f2"], s["a2"], s["b2"], s["c2"],
                               out=s["z2"])
    return dict(blocks_share=z, row_sets_share=z2, rows=comp["row_idx"][:s["n_row"]],
                row_comp=comp["row_comp"][:s["n_row"]], blocks=comp["blk_idx"][:cap],
                blk_comp=comp["blk_comp"][:cap], n_comp=comp["n_comp"], union=idx[:cap], count=n_dev)


def _prepare_mha(case, seed):
    words = _Words(seed)
    ctx = comet.Context(0)
    cfg = configs.MhaConfig("heads", case["d_model"], case["n_heads"], case["head_dim"], case["tokens"],
                            case["refill_rows"], case["density"])
    qkv, heads = configs.mha_head_masks(cfg, seed)
    d, h, bs, m = cfg.d_model, cfg.n_heads, cfg.head_dim, cfg.tokens
    n_blk, n_row = int(np.count_nonzero(qkv.max(axis=0))), int(np.count_nonzero(qkv.max(axis=1)))
    used = int(np.count_nonzero(heads.max(axis=0)))
    n_act, kc = n_blk * bs, used * bs
    return dict(case=case, ctx=ctx, qkv=torch.from_numpy(qkv).cuda(), heads=torch.from_numpy(heads).cuda(),
                n_blk=n_blk, n_row=n_row, used=used,
                e=words(n_row, d), a=words(n_row, d), f=words(d, n_act), b=words(d, 3 * h * bs),
                c=words(n_row, n_act), z=_empty(n_row, n_act), e2=words(m, kc), a2=words(m, h * bs),
                f2=words(kc, d), b2=words(h * bs, d), c2=words(m, d), z2=_empty(m, d))


def _run_mha(s):
    ctx, bs, cap = s["ctx"], s["case"]["head_dim"], s["n_blk"]
    comp = ctx.components(s["qkv"])
    z = ctx.somm_share_blocks(1, bs, comp["blk_idx"], comp["blk_comp"], comp["n_blk"], cap, comp["row_comp"],
                              comp["n_row"], s["e"], s["f"], s["a"], s["b"], s["c"], out=s["z"])
    idx, n_dev = ctx.compact_mask(s["heads"])
    z2 = ctx.simm_share_masked(1, bs, idx, n_dev, s["used"], s["heads"], s["e2"], s["f2"], s["a2"], s["b2"],
                               s["c2"], out=s["z2"])
    return dict(qkv_share=z, output_share=z2, rows=comp["row_idx"][:s["n_row"]], blocks=comp["blk_idx"][:cap],
                n_comp=comp["n_comp"], heads=idx[:s["used"]], count=n_dev)


def _prepare_glue(case, seed):
    words = _Words(seed)
    rows, cols, bs = case["rows"], case["cols"], case["bs"]
    keep = max(1, masks.kept_blocks(case["density"], cols // bs))
    perm = lambda n: torch.randperm(n, device="cuda", generator=words.gen).to(torch.int32)
    mask = masks.clustered_block_mask(seed, 1, cols // bs, keep / (cols // bs))
    idx = torch.from_numpy(np.nonzero(mask)[0].astype(np.int32)).cuda()
    out = [_empty(rows, cols) for _ in range(4)]
    return dict(case=case, ctx=comet.Context(0), x=words(rows, cols), other=words(rows, cols), mask=words(rows, cols),
                pc=perm(cols), pr=perm(rows), idx=idx, n_dev=torch.tensor([idx.numel()], dtype=torch.int32, device="cuda"),
                keep=idx.numel(), compact=words(rows, idx.numel() * bs), out=out)


def _run_glue(s):
    ctx, out = s["ctx"], s["out"]
    ctx.permute_mask(s["x"], s["pc"], s["mask"], comet.AXIS_COLS, +1, out=out[0])
    ctx.permute_mask(s["other"], s["pr"], s["mask"], comet.AXIS_ROWS, -1, out=out[1])
    ctx.truncate_share(1, s["x"], 16, out=out[2])
    ctx.scatter_cols(s["compact"], s["case"]["bs"], s["idx"], s["n_dev"], s["keep"], s["case"]["cols"], out=out[3])
    return out


def _prepare_compact(case, seed):
    n_tok, nb = case["tokens"], case["blocks"]
    flags = masks.stress_mask_device(seed, n_tok * nb, torch.device("cuda"), 0.5).view(n_tok, nb)
    # the tokens of a batch agree on most of their blocks
    common = masks.stress_mask_device(seed + 1, nb, torch.device("cuda"), case["density"]).view(1, nb)
    return dict(case=case, ctx=comet.Context(0), mask=(flags & common).contiguous(),
                idx=torch.zeros(nb, dtype=torch.int32, device="cuda"),
                n_dev=torch.zeros(1, dtype=torch.int32, device="cuda"))


def _run_compact(s):
    idx, n_dev = s["ctx"].compact_mask(s["mask"], s["idx"], s["n_dev"])
    return dict(blocks=idx, count=n_dev)             # entries beyond the count stay as they were


_PREPARE = dict(layer=_prepare_layer, general=_prepare_general, mha=_prepare_mha, glue=_prepare_glue,
                compact=_prepare_compact)
_RUN = dict(layer=_run_layer, general=_run_general, mha=_run_mha, glue=_run_glue, compact=_run_compact)


def prepare(case, seed):
    return _PREPARE[case["family"]](case, seed)


def run(state):
    return _RUN[state["case"]["family"]](state)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    fam = case["family"]
    if fam == "compact":
        return dict(bytes=case["tokens"] * case["blocks"] + 4.0 * case["density"] * case["blocks"], flops=0)
    if fam == "glue":
        n = float(case["rows"] * case["cols"])
        # two shuffle steps (source, mask, result), the rescaling (in, out), the merge (kept in, all out)
        return dict(bytes=8 * n * (3 + 3 + 2 + 1 + case["density"]), flops=0)
    if fam == "mha":
        d, h, bs, m, r = case["d_model"], case["n_heads"], case["head_dim"], case["tokens"], case["refill_rows"]
        used = h * (1.0 - (1.0 - case["density"]) ** m)
        n_act, kc, rows = 3 * used * bs, used * bs, m + r
        # a current token asks for all three blocks of its heads, a refill row for about two and a half heads' K and V
        cells = (m * case["density"] * h * 3 + r * 5.0) * bs
        return dict(bytes=8 * (2 * rows * d + 2 * d * n_act + 2 * rows * n_act + 2 * m * kc + 2 * kc * d + 2 * m * d),
                    flops=INT8_OPS_PER_MAC * 2 * (cells * d + m * kc * d * case["density"]))
    m, d, bs = case["tokens"], case["d_model"], case["bs"]
    if fam == "general":
        nb, g = case["d_ff"] // bs, case["groups"]
        per_group = case["density"] * g
        # every token's blocks lie in its request's share of them; a request of some dozen tokens uses nearly all of it
        used = nb * min(1.0, 1.0 - (1.0 - per_group) ** (m / g))
        n_act = used * bs
        macs = 2.0 * m * d * n_act / g + 2.0 * m * case["density"] * case["d_ff"] * d
        return dict(bytes=8 * (2 * m * d + 2 * d * n_act + 2 * m * n_act + 2 * m * n_act + 2 * n_act * d + 2 * m * d),
                    flops=INT8_OPS_PER_MAC * macs)
    n_act = _kept_blocks(case) * bs
    total, macs = 0.0, 0.0
    for kind in _projections(case):
        k, n = (d, n_act) if kind == "somm" else (n_act, d)
        # per party: x, a, y, b, c in (the kept part), the masked shares of both operands and z out
        one = 3 * m * k + 3 * k * n + 2 * m * n
        if case["form"] == "planes":
            one += k * n                                   # the triple share once more, as packed offline
        total += case["parties"] * one
        if case["parties"] == 1:
            total += m * k + k * n                         # what the other party sent
        macs += case["parties"] * 2.0 * m * k * n
    return dict(bytes=8 * total, flops=INT8_OPS_PER_MAC * macs)


def tolerance(case):
    return "exact"                                         # whole numbers mod 2^64
