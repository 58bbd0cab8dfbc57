"""The attention kernel in each way a launch is cut (wavefronts that share a list, halves of a Q block), on lists
of every length from none to all columns: rows shorter than the number of shares, odd numbers of parts, a ragged last
block, logits whose reference differs from share to share.  Reference: masked softmax attention in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2512_24086_amd import rf2
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda"

# (tokens, block, block_k, head_dim, heads): few and long rows = several wavefronts to a list, many or short = one (see
# rf2_attn_cut.h; the host test of the cut asks for every instance, together with test_gpu_attn_stream)
SHAPES = [(2000, 128, 128, 128, 2), (1000, 128, 128, 128, 33), (2000, 128, 64, 128, 3), (999, 64, 64, 128, 2),
          (999, 64, 128, 128, 3), (999, 64, 128, 128, 17), (700, 64, 64, 64, 2), (700, 64, 128, 64, 3), (1000, 64, 64, 64, 20),
          (2500, 64, 64, 64, 2), (2500, 64, 128, 64, 1), (2000, 128, 128, 64, 2), (2000, 128, 64, 64, 2),
          (6200, 128, 64, 64, 1), (6200, 128, 128, 64, 1), (2500, 256, 128, 128, 2), (2500, 256, 64, 128, 2),
          (1000, 256, 64, 128, 41), (2500, 256, 128, 64, 2), (900, 256, 64, 64, 70), (40, 64, 64, 64, 1), (130, 256, 128, 128, 1),
          (1000, 64, 128, 64, 40), (1000, 128, 128, 64, 40), (999, 64, 64, 128, 24), (600, 256, 64, 64, 700),
          (600, 256, 128, 64, 700), (600, 256, 64, 128, 350), (600, 256, 128, 128, 350)]


def lists(plan, seed):
    """Masks [heads][Tq, Tk]: rows of 0, 1, 2, ... columns, of k_row, and of all."""
    i, rng = plan.info, np.random.default_rng(seed)
    out = []
    for _ in range(plan.cfg.heads):
        M = np.zeros((i.n_blocks, i.n_blocks_k), dtype=bool)
        for r in range(i.n_blocks):
            n = (r % 6 if r % 6 < 4 else i.k_row if r % 6 == 4 else i.n_blocks_k) if i.n_blocks > 2 else i.k_row
            n = n if n == i.n_blocks_k else min(n, i.k_row)
            M[r, rng.choice(i.n_blocks_k, n, replace=False)] = True
        out.append(M)
    return out


@pytest.mark.parametrize("scale", [1.0, 24.0])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_lists_of_every_length(shape, scale):
    tokens, block, block_k, d, heads = shape
    print(f"[case] {shape} scale {scale}", flush=True)
    plan = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3,
                    window=(1, 1, 16))
    i = plan.info
    g = torch.Generator().manual_seed(7)
    q, k, v = (torch.randn(1, heads, tokens, d, generator=g) for _ in range(3))
    # later keys are larger: the softmax reference has to move, by other amounts in each group
    k = k * torch.linspace(1.0, scale, tokens)[:, None]
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    masks = lists(plan, 5)
    idx, cnt = hp.lists_to_device(masks, i.k_row, i.n_blocks, DEV)
    buf = plan.alloc(DEV, lse=True)
    plan.rf2_permute(*(x.to(DEV) for x in (q, k, v)), buf["qp"], buf["kp"], buf["vp"])
    buf["op"].fill_(float("nan"))
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], idx, cnt, buf["op"], buf["lse"])
    o = torch.full_like(buf["o"], float("nan"))
    lse = torch.full((1, heads, tokens), float("nan"), device=DEV)
    plan.rf2_block_sparse_attn_unpermuted(buf["qp"], buf["kp"], buf["vp"], idx, cnt, o, lse)
    torch.cuda.synchronize()
    perm = plan.rf2_plan_perm()[0]
    assert torch.equal(o[:, :, perm].view(torch.int16), buf["op"][:, :, :tokens].view(torch.int16))
    assert torch.equal(lse[:, :, perm], buf["lse"][:, :, :tokens])
    for h in sorted({0, heads // 2, heads - 1}):
        Q, K, V = (x[0, h][perm].double() for x in (q, k, v))
        keep = torch.from_numpy(masks[h]).repeat_interleave(block, 0).repeat_interleave(block_k, 1)[:tokens, :tokens]
        S = (Q @ K.T / d ** 0.5).masked_fill(~keep, -torch.inf)
        empty = ~keep.any(1)
        P = torch.softmax(S, 1).nan_to_num(0.0)     # a row without a block: zeros, lse = -inf
        want = P @ V
        err = (buf["op"][0, h, :tokens].cpu().double() - want).abs()
        # probabilities and outputs rounded to bf16 (2^-8 each, relative), fp32 logits of up to ~1e3 (1e-3 at most)
        assert (err <= 2.0 ** -8 * (P @ V.abs() + want.abs()) + 1e-3).all(), (h, err.max())
        assert err.mean() <= hp.ATTN_MEAN_ABS, (h, err.mean())
        got = buf["lse"][0, h, :tokens].cpu().double()
        ref = torch.logsumexp(S, 1)
        assert torch.equal(torch.isneginf(got), empty)
        # fp32 logits and sums: 2e-3 as everywhere, and a few units in the last place of the largest logits
        assert ((got - ref)[~empty].abs() <= 2e-3 + 1e-6 * ref[~empty].abs()).all()
    plan.close()


# no ragged block: every number of parts, also such as wavefronts cannot share evenly.  (The first eleven have four or eight wavefronts
# to a list, the others one and two, for one and two tiles of rows, and both in one launch: the host test of the cut asks for that.)
NONFINITE = [(1920, 128, 128, 128, 2), (1920, 128, 64, 128, 3), (960, 64, 64, 128, 2), (1024, 64, 128, 128, 3),
             (704, 64, 64, 64, 2), (2496, 64, 64, 64, 2), (2560, 64, 128, 64, 1), (1920, 128, 128, 64, 2),
             (6144, 128, 64, 64, 1), (2560, 256, 128, 128, 2), (2560, 256, 64, 64, 2),
             (768, 64, 128, 128, 100), (640, 128, 128, 128, 8), (2560, 128, 64, 128, 24), (768, 128, 128, 128, 100),
             (6272, 128, 64, 128, 5), (768, 128, 64, 64, 64), (1536, 64, 64, 64, 24), (1024, 128, 128, 64, 36)]


def run_lists(shape, q, k, v, masks_seed=5):
    """(plan, masks, output in permuted order, lse, q, k, v in permuted order) of one call on `lists`."""
    tokens, block, block_k, d, heads = shape
    plan = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3,
                    window=(1, 1, 16))
    masks = lists(plan, masks_seed)
    idx, cnt = hp.lists_to_device(masks, plan.info.k_row, plan.info.n_blocks, DEV)
    buf = plan.alloc(DEV, lse=True)
    plan.rf2_permute(*(x.to(DEV) for x in (q, k, v)), buf["qp"], buf["kp"], buf["vp"])
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], idx, cnt, buf["op"], buf["lse"])
    torch.cuda.synchronize()
    perm = plan.rf2_plan_perm()[0]
    return plan, masks, buf["op"][0, :, :tokens].cpu().double(), buf["lse"][0, :, :tokens].cpu().double(), *(
        x[0][:, perm].double() for x in (q, k, v))


@pytest.mark.parametrize("shape", NONFINITE, ids=lambda s: "x".join(map(str, s)))
def test_infinite_values_reach_only_their_own_channel(shape):
    """One key of every part has an infinite value in a channel of that part's: the channel is infinite in the rows that
    keep the block, and every other channel is what it is without the infinities (no product of zero and infinity)."""
    tokens, block, block_k, d, heads = shape
    print(f"[case] {shape}", flush=True)
    g = torch.Generator().manual_seed(11)
    q, k, v = (torch.randn(1, heads, tokens, d, generator=g).to(torch.bfloat16) for _ in range(3))
    perm = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3,
                    window=(1, 1, 16)).rf2_plan_perm()[0]
    # parts (of 64 keys) and the block row of the key: first tile of a part for even blocks, second for odd ones (where a
    # list begins with such a block, step 0 multiplies that tile by zero: left out below)
    n_k, per = tokens // block_k, block_k // 64
    channel = np.zeros((n_k, per), dtype=int)
    clean = v.clone()
    for j in range(n_k):
        for p in range(per):
            channel[j, p] = (j * per + p) % d
            row = j * block_k + 32 * p + (5 if j % 2 == 0 else block_k // 2 + 5)
            v[:, :, perm[row], channel[j, p]] = float("inf")
            clean[:, :, perm[row], channel[j, p]] = 0
    plan, masks, o, _, Q, K, V = run_lists(shape, q, k, v)
    V = clean[0][:, perm].double()
    for h in sorted({0, heads // 2, heads - 1}):
        keep = torch.from_numpy(masks[h])
        token_keep = keep.repeat_interleave(block, 0).repeat_interleave(block_k, 1)[:tokens, :tokens]
        P = torch.softmax((Q[h] @ K[h].T / d ** 0.5).masked_fill(~token_keep, -torch.inf), 1).nan_to_num(0.0)
        want = P @ V[h]
        unsure = torch.zeros_like(want, dtype=torch.bool)
        for r in range(keep.shape[0]):
            rows = slice(r * block, min((r + 1) * block, tokens))
            cols = np.flatnonzero(masks[h][r])
            for n, j in enumerate(cols):
                want[rows, channel[j]] = torch.inf
            if cols.size and cols[0] % 2:
                unsure[rows, channel[cols[0], 0]] = True
        inf = torch.isinf(want) & ~unsure
        assert (o[h][inf] == torch.inf).all(), (h, o[h][inf])
        rest = ~torch.isinf(want) & ~unsure
        bound = 2.0 ** -8 * (P @ V[h].abs() + want.abs()) + 1e-3
        assert ((o[h] - want).abs() <= bound)[rest].all(), h
    plan.close()


@pytest.mark.parametrize("shape", NONFINITE, ids=lambda s: "x".join(map(str, s)))
def test_products_of_minus_infinity_and_far_below_zero(shape):
    """Blocks whose products are all minus infinity weigh nothing, also where they are the first of a group's share, and
    the reference finds the others' level however low it is: logits around -2,500 / sqrt(d)."""
    tokens, block, block_k, d, heads = shape
    print(f"[case] {shape}", flush=True)
    g = torch.Generator().manual_seed(12)
    q, k, v = (torch.randn(1, heads, tokens, d, generator=g) for _ in range(3))
    q[..., :2] = 1.0
    k[..., 1] = -2496.0
    perm = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3,
                    window=(1, 1, 16)).rf2_plan_perm()[0]
    gone = torch.arange(tokens) // block_k % 3 == 1
    k[..., 0] = 0.0
    k[:, :, perm[gone.numpy()], 0] = -torch.inf
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    plan, masks, o, lse, Q, K, V = run_lists(shape, q, k, v)
    for h in sorted({0, heads // 2, heads - 1}):
        keep = torch.from_numpy(masks[h])
        # (a list that begins with such a block has no number to refer to: not a number before and after)
        first = torch.where(keep.any(1), keep.to(torch.uint8).argmax(1), 0)
        rows = ((first % 3 != 1) & keep.any(1)).repeat_interleave(block)[:tokens]
        token_keep = keep.repeat_interleave(block, 0).repeat_interleave(block_k, 1)[:tokens, :tokens] & ~gone
        S = (Q[h] @ K[h].T / d ** 0.5).masked_fill(~token_keep, -torch.inf)
        P = torch.softmax(S, 1).nan_to_num(0.0)
        want, ref = P @ V[h], torch.logsumexp(S, 1)
        # fp32 products of 2,500: logits off by 2^-24 x 2,500 x (d terms, a few ulp each) / sqrt(d), under 1e-3
        assert ((o[h] - want).abs() <= 2.0 ** -7 * (P @ V[h].abs() + want.abs()) + 2e-3)[rows].all(), h
        assert ((lse[h] - ref).abs() <= 2e-3 + 1e-6 * ref.abs())[rows].all(), h
    plan.close()
