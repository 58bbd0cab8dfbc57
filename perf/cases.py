"""Timed cases of the block-sparse attention layer, through the entry points a program calls.

A case names a stage and a configuration:

  layer      one whole layer: permutation + pooling, mask prediction, attention, inverse permutation, as
             `Plan.layer_fused` (inverse permutation in the attention kernel) or `Plan.layer` (`fused` False)
  attn       `rf2_block_sparse_attn_unpermuted` on permuted tensors and block lists, as a program calls it
             that keeps a mask for several denoising steps or brings lists of its own
  permute    `rf2_permute` with block means
  mask       `rf2_predict_mask`
  unpermute  `rf2_unpermute`

The plan, the inputs and the buffers are made in `prepare`; `run` is one pass.  The inputs are smooth fields over
the (T, H, W) grid plus noise, unit variance, in bf16 (what neighbouring tokens of a diffusion transformer look
like), and independent rows for text tokens.  The sizes are the workloads of `paper_2512_24086_amd/inputs.py`,
the options `bench.py` times on them, and ragged grids between them.
"""
import math

import torch

from paper_2512_24086_amd import rf2

DEV = "cuda"
WAVES = 24          # sinusoids of a field
MAX_CYCLES = 2.0    # per axis

DEFAULTS = dict(stage="layer", fused=True, batch=1, heads=40, d=128, T=21, H=45, W=80, block=128, block_k=0,
                sparsity=0.8, sink=1, text=0, bnhd=False, cdf=0.0, lse=False, sigma=0.3)


def _case(name, **over):
    return dict(DEFAULTS, name=name, **over)


def listed():
    return [
        # The smallest whole call of the workload list: 1,536 tokens, where launches and latency count.
        _case("layer_tiny", heads=2, d=64, T=6, H=16, W=16, block=64, sparsity=0.5),
        # One layer of an image model: 1,024 x 1,024 pixels as 64 x 64 tokens, no first frame.
        _case("layer_image", heads=24, T=1, H=64, W=64, sparsity=0.5, sink=0),
        # An image of odd size with a text prompt, tensors as the model's projections leave them
        # ([B, N, Hh, d]), the four separate calls.
        _case("layer_image_text", heads=24, T=1, H=61, W=67, sparsity=0.6, sink=0, text=77, bnhd=True, fused=False),
        # One layer of a 480p video model.
        _case("layer_480p", H=30, W=52),
        # The headline: one layer of a 720p video model, 75,600 tokens.
        _case("layer_720p"),
        # 480p with the finer 64-token blocks (a sharper mask for the same budget).
        _case("layer_480p_b64", H=30, W=52, block=64),
        # Attention of a video model with 64 channels a head, on lists it already has.
        _case("attn_480p_d64", stage="attn", H=30, W=52, d=64),
        # The longest sequence, at the highest sparsity, with the log-sum-exp that a caller needs who merges
        # this attention with another over further keys.
        _case("attn_long", stage="attn", heads=24, T=33, sparsity=0.9, sigma=0.5, lse=True),
        # A ragged clip with large Q blocks over smaller K/V blocks, few heads (a shard of the model).
        _case("attn_clip_q256", stage="attn", heads=10, T=13, H=29, W=51, block=256, block_k=128, sparsity=0.7),
        # Permutation and pooling of token-major tensors, 480p.
        _case("permute_480p", stage="permute", H=30, W=52, bnhd=True),
        # Mask prediction of the headline layer.
        _case("mask_720p", stage="mask"),
        # Mask prediction by cumulative mass on the long video.
        _case("mask_long_cdf", stage="mask", heads=24, T=33, sigma=0.5, cdf=0.9),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    c = dict(DEFAULTS)
    c["stage"] = rng.choices(["layer", "attn", "mask", "permute", "unpermute"], [8, 5, 3, 2, 1])[0]
    c["fused"] = rng.random() < 0.75
    c["batch"] = 2 if rng.random() < 0.15 else 1
    c["heads"] = rng.choice([1, 2, 3, 5, 8, 10, 12, 16, 20, 24, 32, 40])
    c["d"] = rng.choice([128, 128, 64])
    c["block"], c["block_k"] = rng.choice([(128, 0), (128, 0), (128, 0), (64, 0), (64, 0), (256, 128), (256, 64), (128, 64),
                                           (64, 128)])
    tokens = _log_uniform(rng, 1200, 118800)
    if tokens < 8000 and rng.random() < 0.6:
        c["T"], c["sink"] = 1, 0
    else:
        c["T"] = rng.randint(5, 33)
        c["sink"] = rng.choice([1, 1, 1, 0])
    frame = tokens / c["T"]
    c["H"] = max(6, int(round(math.sqrt(frame) * rng.uniform(0.6, 1.0))))
    c["W"] = max(8, int(round(frame / c["H"])))
    c["text"] = rng.choice([0, 0, rng.randint(20, 512)])
    c["sparsity"] = round(rng.uniform(0.5, 0.9), 2)
    c["bnhd"] = rng.random() < 0.4
    c["cdf"] = rng.choice([0.0, 0.0, 0.0, 0.0, 0.7, 0.9]) if c["stage"] in ("layer", "mask") else 0.0
    c["lse"] = c["stage"] == "attn" and rng.random() < 0.4
    c["sigma"] = rng.choice([0.3, 0.5])
    # no more than the headline layer costs: half its products at most (a 64-token block or a short row runs at a
    # lower rate than the headline's), and no more elements
    while c["heads"] > 1 and (_products(c) > 1.1e13 or c["batch"] * c["heads"] * _tokens(c) > 75600 * 40):
        c["heads"] = max(1, c["heads"] // 2)
    return c


def _tokens(c):
    return c["T"] * c["H"] * c["W"] + c["text"]


def _products(c):
    """Upper estimate of the attention's operations from the sizes alone (all-column sink rows included)."""
    n = _tokens(c)
    if c["stage"] not in ("layer", "attn"):
        return 0.0
    density = max(1.0 - c["sparsity"], (c["sink"] * c["H"] * c["W"] + c["text"] + 2 * c["block"]) * 2 / n, c["cdf"])
    return 4.0 * n * n * c["d"] * c["heads"] * c["batch"] * min(1.0, density)


def _plan(c):
    return rf2.Plan(batch=c["batch"], heads=c["heads"], head_dim=c["d"], T=c["T"], H=c["H"], W=c["W"], block=c["block"],
                    block_k=c["block_k"], sparsity=c["sparsity"], sink_frames=c["sink"], text_tokens=c["text"],
                    qkv_layout=rf2.RF2_LAYOUT_BNHD if c["bnhd"] else rf2.RF2_LAYOUT_BHND,
                    cdf_threshold=c["cdf"] or None)


# ---- inputs -------------------------------------------------------------------------------------------------

def _field(c, gen):
    """One tensor [B, N, Hh, d] (or [B, Hh, N, d]) bf16: smooth over the grid, plus noise, unit variance."""
    T, H, W, channels = c["T"], c["H"], c["W"], c["heads"] * c["d"]
    n = T * H * W
    idx = torch.arange(n, device=DEV)
    at = torch.stack([(idx // (H * W)).float() / T, (idx // W % H).float() / H, (idx % W).float() / W], 1)
    out = []
    for _ in range(c["batch"]):
        freq = (torch.rand(3, WAVES, generator=gen, device=DEV) * 2 - 1) * MAX_CYCLES
        if T == 1:
            freq[0] = 0
        arg = (at @ freq) * (2 * math.pi)
        amp = torch.randn(2 * WAVES, channels, generator=gen, device=DEV) / math.sqrt(WAVES)
        x = torch.cat([arg.cos(), arg.sin()], 1) @ amp
        x += c["sigma"] * torch.randn(n, channels, generator=gen, device=DEV)
        x /= math.sqrt(1 + c["sigma"] ** 2)
        if c["text"]:
            x = torch.cat([x, torch.randn(c["text"], channels, generator=gen, device=DEV)])
        out.append(x.to(torch.bfloat16).view(-1, c["heads"], c["d"]))
    x = torch.stack(out)
    return x if c["bnhd"] else x.transpose(1, 2).contiguous()


def _inputs(c, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return [_field(c, gen) for _ in range(3)]


# ---- plain torch, 64 bits: block means, masks, attention ----------------------------------------------------

def _heads_first(c, x):
    """[B * Hh, N, d] view or copy of a caller's tensor."""
    x = x.transpose(1, 2) if c["bnhd"] else x
    return x.reshape(-1, x.shape[-2], x.shape[-1])


def _permuted(c, x, perm, n_pad):
    """[B * Hh, n_pad, d]: the tokens in permuted order, zero rows after them."""
    x = _heads_first(c, x)[:, perm]
    return torch.nn.functional.pad(x, (0, 0, 0, n_pad - x.shape[1]))


def _means(xp, b, n):
    """Block means in 64 bits, one head at a time (a whole layer in 64 bits is large)."""
    blocks = xp.shape[1] // b
    count = torch.full((blocks, 1), b, dtype=torch.float64, device=DEV)
    count[-1] = n - (blocks - 1) * b
    return torch.stack([h.double().view(blocks, b, -1).sum(1) / count for h in xp])


def _mask(c, info, qbar, kbar):
    """[B * Hh, Tq, Tk] truth values from block means: eqs. (7), (8), sink rows and columns."""
    keep = torch.zeros(qbar.shape[0], info.n_blocks, info.n_blocks_k, dtype=torch.bool, device=DEV)
    sink = slice(info.sink_block_begin_k, info.sink_block_end_k)
    for h in range(qbar.shape[0]):
        s = qbar[h].double() @ kbar[h].double().t().contiguous()
        s[:, sink] = -math.inf
        order = torch.sort(s, dim=1, descending=True, stable=True)[1]
        if c["cdf"]:
            p = torch.softmax(s / math.sqrt(c["d"]), dim=1).gather(1, order)
            take = p.cumsum(1) - p < c["cdf"]
            take &= s.gather(1, order) > -math.inf
        else:
            take = (torch.arange(info.n_blocks_k, device=DEV) < info.k_sel).expand_as(order)
        keep[h].scatter_(1, order, take)
    keep[:, :, sink] = True
    keep[:, info.sink_block_begin:info.sink_block_end] = True
    return keep


def _lists(c, info, keep):
    """The block lists of rf2_predict_mask for a mask of k_row (or all) columns a row."""
    idx = torch.sort((~keep).to(torch.uint8), dim=2, stable=True)[1][:, :, :info.k_row].to(torch.int32)
    shape = (c["batch"], c["heads"], info.n_blocks)
    return idx.reshape(*shape, info.k_row).contiguous(), keep.sum(2, dtype=torch.int32).reshape(shape)


def _attention(c, info, qp, kp, vp, keep):
    """Softmax attention over the kept blocks, 64 bits; ([B * Hh, N_pad, d], [B * Hh, N_pad])."""
    bh, bk, d = qp.shape[0], info.block_k, c["d"]
    o = torch.zeros(bh, info.N_pad, d, dtype=torch.float64, device=DEV)
    lse = torch.zeros(bh, info.N_pad, dtype=torch.float64, device=DEV)
    heads = torch.arange(bh, device=DEV)[:, None]
    kb, vb = kp.view(bh, -1, bk, d), vp.view(bh, -1, bk, d)
    inside = torch.arange(bk, device=DEV)
    # as many Q blocks at a time as fit 8 GB of logits
    for i in range(info.n_blocks):
        rows = slice(i * c["block"], (i + 1) * c["block"])
        most = int(keep[:, i].sum(1).max())
        step = max(1, int(8e9 / (c["block"] * most * bk * 8)))
        kept, cols = torch.sort(keep[:, i].to(torch.uint8), dim=1, descending=True, stable=True)
        kept, cols = kept[:, :most].bool(), cols[:, :most]
        for h in range(0, bh, step):
            at = slice(h, h + step)
            k = kb[heads[at], cols[at]].double().flatten(1, 2)
            s = qp[at, rows].double() @ k.transpose(1, 2).contiguous() / math.sqrt(d)
            fine = kept[at, :, None] & (cols[at, :, None] * bk + inside < info.N)
            s.masked_fill_(~fine.flatten(1)[:, None], -math.inf)
            lse[at, rows] = torch.logsumexp(s, 2)
            s = torch.exp_(s - lse[at, rows, None])
            o[at, rows] = s @ vb[heads[at], cols[at]].double().flatten(1, 2)
    return o, lse


def _to_tokens(c, info, perm, xp):
    """Permuted order -> the caller's order and layout."""
    out = torch.empty(xp.shape[0], info.N, *xp.shape[2:], dtype=xp.dtype, device=DEV)
    out[:, perm] = xp[:, :info.N]
    out = out.view(c["batch"], c["heads"], *out.shape[1:])
    return out.transpose(1, 2).contiguous() if c["bnhd"] and out.dim() == 4 else out


def _perm(plan):
    return torch.from_numpy(plan.rf2_plan_perm()[0]).to(DEV).long()


# ---- the cases ----------------------------------------------------------------------------------------------

def prepare(case, seed):
    c = case
    plan = _plan(c)
    info = plan.info
    s = dict(case=c, plan=plan)
    if c["stage"] == "unpermute":
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed)
        s["op"] = torch.randn(c["batch"], c["heads"], info.N_pad, c["d"], generator=gen, device=DEV).to(torch.bfloat16)
        s["buf"] = {"o": plan.alloc(DEV)["o"]}
        return s
    q, k, v = _inputs(c, seed)
    buf = s["buf"] = plan.alloc(DEV)
    if c["cdf"]:
        buf["blk_idx"].fill_(-1)      # what lies behind a row's count stays as the caller left it
    if c["stage"] in ("layer", "permute"):
        s["qkv"] = (q, k, v)
        return s
    perm = _perm(plan)
    qbar = _means(_permuted(c, q, perm, info.N_pad), c["block"], info.N)
    kbar = _means(_permuted(c, k, perm, info.N_pad_k), info.block_k, info.N)
    if c["stage"] == "mask":
        s["qbar"] = qbar.float().view(buf["qbar"].shape)
        s["kbar"] = kbar.float().view(buf["kbar"].shape)
        for name in ("qp", "kp", "vp", "op", "o"):
            del buf[name]
        return s
    plan.rf2_permute(q, k, v, buf["qp"], buf["kp"], buf["vp"])
    s["lists"] = _lists(c, info, _mask(c, info, qbar, kbar))
    if c["lse"]:
        buf["lse"] = torch.empty(c["batch"], c["heads"], info.N, dtype=torch.float32, device=DEV)
    return s


def run(state):
    c, plan, buf = state["case"], state["plan"], state["buf"]
    if c["stage"] == "layer":
        return {"o": (plan.layer_fused if c["fused"] else plan.layer)(*state["qkv"], buf)}
    if c["stage"] == "attn":
        plan.rf2_block_sparse_attn_unpermuted(buf["qp"], buf["kp"], buf["vp"], *state["lists"], buf["o"], buf.get("lse"))
        return {"o": buf["o"], "lse": buf["lse"]} if c["lse"] else {"o": buf["o"]}
    if c["stage"] == "permute":
        names = ("qp", "kp", "vp", "qbar", "kbar")
        plan.rf2_permute(*state["qkv"], *(buf[n] for n in names))
        return {n: buf[n] for n in names}
    if c["stage"] == "mask":
        plan.rf2_predict_mask(state["qbar"], state["kbar"], buf["blk_idx"], buf["blk_cnt"])
        return {n: buf[n] for n in ("blk_idx", "blk_cnt")}
    plan.rf2_unpermute(state["op"], buf["o"])
    return {"o": buf["o"]}


def work(case):
    c = case
    plan = _plan(c)
    info = plan.info
    plan.close()
    bh, n, d = c["batch"] * c["heads"], info.N, c["d"]
    tensor = bh * n * d * 2
    means = bh * (info.n_blocks + info.n_blocks_k) * d * 4
    # a cumulative-mass row keeps about as large a share of the blocks as of the mass (flat rows)
    pairs = info.kept_pairs_per_head if not c["cdf"] else c["cdf"] * info.n_blocks * info.n_blocks_k
    entries = bh * (min(pairs, info.n_blocks * info.k_row) + info.n_blocks) * 4
    scores = 2.0 * bh * info.n_blocks * info.n_blocks_k * d
    products = 4.0 * bh * d * pairs * (n / info.n_blocks) * (n / info.n_blocks_k)
    if c["stage"] == "layer":
        return {"bytes": 4.0 * tensor, "flops": products + scores}
    if c["stage"] == "attn":
        return {"bytes": 4.0 * tensor + entries + (bh * n * 4 if c["lse"] else 0), "flops": products}
    if c["stage"] == "permute":
        return {"bytes": 6.0 * tensor + means, "flops": 2.0 * bh * n * d}
    if c["stage"] == "mask":
        return {"bytes": float(means + entries), "flops": scores}
    return {"bytes": 2.0 * tensor, "flops": 0}


def tolerance(case):
    if case["stage"] == "unpermute":
        return "exact"
    if case["stage"] == "permute":
        return {"rel": 1e-7}            # copies are exact; fp32 means of up to 256 values (7e-9 off the 64-bit ones)
    if case["stage"] == "mask":
        # rows whose boundary scores tie in fp32: against 64-bit scores up to 9e-5 of the entries differ
        return {"rel": 0.0, "differ": 5e-4}
    return {"rel": 7e-3}                # probabilities and outputs in bf16: 1.7e-3 off the 64-bit result


def exact(case, seed):
    c = case
    if c["stage"] in ("mask", "unpermute"):
        return None                     # whole numbers; copies
    if _products(c) > 6e13:
        return None
    plan = _plan(c)
    info, perm = plan.info, _perm(plan)
    q, k, v = _inputs(c, seed)
    qp, kp, vp = (_permuted(c, x, perm, m) for x, m in ((q, info.N_pad), (k, info.N_pad_k), (v, info.N_pad_k)))
    del q, k, v
    qbar, kbar = _means(qp, c["block"], info.N), _means(kp, info.block_k, info.N)
    lead = (c["batch"], c["heads"])
    if c["stage"] == "permute":
        return {"qp": None, "kp": None, "vp": None, "qbar": qbar.view(*lead, *qbar.shape[1:]),
                "kbar": kbar.view(*lead, *kbar.shape[1:])}
    o, lse = _attention(c, info, qp, kp, vp, _mask(c, info, qbar, kbar))
    out = {"o": _to_tokens(c, info, perm, o)}
    if c["lse"]:
        out["lse"] = _to_tokens(c, info, perm, lse)
    return out
