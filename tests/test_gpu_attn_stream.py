"""The attention kernel in every way a launch is cut (64-row tiles of a workgroup, wavefronts that share a list), on the
lists, logits and bounds of test_gpu_attn_cut: rows of no block up to all, a ragged last block with and without a part that holds
no key, a reference that moves.  Launches of 256-row workgroups are as large as a 720p layer: test_gpu_fullsize has them."""
import ctypes as C
import os
import subprocess

import pytest
import torch

from paper_2512_24086_amd import build as b
from paper_2512_24086_amd import rf2
from tests import helpers as hp
from tests import test_gpu_attn_cut as cut_tests

# (tokens, block, block_k, head_dim, heads) -> (rows of a workgroup, wavefronts that share a list)
SHAPES = {(330, 64, 64, 128, 200): (64, 1), (330, 64, 128, 128, 200): (64, 1), (2450, 128, 64, 128, 12): (64, 2),
          (2450, 64, 128, 128, 8): (64, 2), (657, 64, 64, 128, 1): (64, 4), (2450, 256, 128, 128, 2): (64, 4),
          (4000, 128, 64, 128, 41): (128, 1), (4001, 128, 128, 128, 41): (128, 1), (6177, 128, 64, 128, 5): (128, 2),
          (6200, 256, 128, 128, 5): (128, 2),
          (999, 64, 64, 64, 100): (64, 1), (2450, 128, 128, 64, 41): (64, 1), (1500, 64, 64, 64, 23): (64, 2),
          (600, 128, 128, 64, 24): (64, 2), (657, 64, 64, 64, 17): (64, 4), (900, 128, 128, 64, 3): (64, 4),
          (2450, 64, 64, 64, 1): (64, 8), (4000, 128, 128, 64, 1): (64, 8), (2450, 128, 64, 64, 24): (128, 2),
          (2450, 128, 128, 64, 24): (128, 2), (900, 256, 64, 64, 64): (128, 2)}

# the same -> row slots of an XCD that are cut as workgroups of 128 rows; those behind them as two of 64 rows and two shares
MIXED = {(2450, 128, 64, 128, 27): 64, (2450, 128, 128, 128, 32): 64, (2450, 256, 128, 128, 30): 32, (2433, 256, 64, 128, 26): 32}

# (tokens, text tokens, block, block_k, heads) -> the same, with all-column text rows in two shares, too
HALVED = {(2450, 200, 128, 128, 27): 64, (2450, 77, 128, 64, 39): 96, (2450, 200, 256, 128, 36): 40, (2433, 77, 256, 64, 30): 32}

# plan -> the same for heads whose K and V are too large to stay whole on an XCD: ordinary rows dealt by the work table, 8 shares of a
# head of slightly different size, so that slots without work lie among the whole rows and the halves
TABLE = {(("W", 50003), ("heads", 3), ("sparsity", 0.7), ("block", 128)): (128, 0),
         (("W", 52003), ("heads", 4), ("sparsity", 0.8), ("block", 256), ("block_k", 64)): (80, 0),
         (("T", 13), ("H", 62), ("W", 62), ("heads", 4), ("sparsity", 0.8), ("block", 128), ("block_k", 64), ("sink_frames", 1)): (128, 1),
         (("T", 21), ("H", 45), ("W", 80), ("heads", 5), ("sparsity", 0.9), ("block", 256), ("block_k", 128), ("sink_frames", 1)): (128, 1)}

SOURCE = """#include "rf2_attn_cut.h"
extern "C" void cut(const rf2_config* c, const rf2_info* i, int* out) {
  const rf2_attn_cut x = rf2_cut_stream(*c, *i);
  out[0] = x.rows, out[1] = x.groups, out[2] = x.whole_heads, out[3] = x.whole_slots, out[4] = x.halved_sinks;
}
"""


def test_cuts(tmp_path):
    (tmp_path / "cut.cpp").write_text(SOURCE)
    lib = str(tmp_path / "cut.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", os.path.join(b.ROOT, "include"),
                    "-I", b.CSRC, str(tmp_path / "cut.cpp"), "-o", lib], check=True)
    fn, out = C.CDLL(lib).cut, (C.c_int * 5)()

    def cut(**kw):
        plan = rf2.Plan(**dict(dict(batch=1, head_dim=128, T=1, H=1, sparsity=0.3, window=(1, 1, 16)), **kw))
        fn(C.byref(plan.cfg), C.byref(plan.info), out)
        plan.close()
        return tuple(out)

    for (tokens, block, block_k, d, heads), want in SHAPES.items():
        assert cut(W=tokens, block=block, block_k=block_k, head_dim=d, heads=heads)[:2] == want, (tokens, block, block_k, d, heads)
    for (tokens, block, block_k, d, heads), want in MIXED.items():
        assert cut(W=tokens, block=block, block_k=block_k, head_dim=d, heads=heads) == (128, 1, 1, want, 0), (tokens, block, block_k, heads)
    for (tokens, text, block, block_k, heads), want in HALVED.items():
        assert cut(W=tokens, text_tokens=text, block=block, block_k=block_k, heads=heads, sparsity=0.7) == (128, 1, 1, want, 1), (tokens, heads)
    for case, (whole, halved) in TABLE.items():
        assert cut(**dict(case)) == (128, 1, 0, whole, halved), case
    video = dict(T=21, H=45, W=80, sparsity=0.8, sink_frames=1, window=(0, 0, 0))
    assert cut(**video, heads=40, block=128) == (128, 1, 0, 0, 0)          # 8 heads' K and V are larger than the Infinity Cache
    assert cut(**video, heads=40, block=256, block_k=128) == (256, 1, 0, 0, 0)
    assert cut(**dict(video, H=30, W=52), heads=40, block=128) == (128, 1, 1, 0, 0)
    assert cut(**video, heads=1, block=128)[:2] == (64, 4)
    # a launch of the largest size the limits allow is cut without walking through its rows
    assert cut(T=1, H=1, W=2048 * 64, heads=65535, block=64)[:1] == (64,)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [*SHAPES, *MIXED], ids=lambda s: "x".join(map(str, s)))
def test_every_cut(shape):
    cut_tests.test_lists_of_every_length(shape, 24.0)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(2450, 128, 64, 128, 12), (657, 64, 64, 128, 1), (4001, 128, 128, 128, 41), (6177, 128, 64, 128, 5),
                                   (2450, 128, 128, 64, 41), (2450, 64, 64, 64, 1), (2450, 128, 128, 64, 24)], ids=lambda s: "x".join(map(str, s)))
def test_entries_behind_the_count(shape):
    """A row's first and last entries are asked for before its count is known: what a list holds behind its count, and at all
    where a row keeps every column, changes no bit of the result."""
    tokens, block, block_k, d, heads = shape
    print(f"[case] {shape}", flush=True)
    plan = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3, window=(1, 1, 16))
    i = plan.info
    g = torch.Generator(device="cuda").manual_seed(11)
    q, k, v = (torch.randn(1, heads, tokens, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    idx, cnt = hp.lists_to_device(cut_tests.lists(plan, 5), i.k_row, i.n_blocks, "cuda")
    buf = plan.alloc("cuda", lse=True)
    plan.rf2_permute(q, k, v, buf["qp"], buf["kp"], buf["vp"])
    unused = (torch.arange(i.k_row, device="cuda") >= cnt[..., None]) | (cnt[..., None] == i.n_blocks_k)
    results = []
    for fill in (0, -1, i.n_blocks_k - 1, 2**31 - 1, -2**31):
        plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], idx.masked_fill(unused, fill), cnt, buf["op"], buf["lse"])
        results.append((buf["op"].view(torch.int16).clone(), buf["lse"].clone()))
    assert unused.any()
    for op, lse in results[1:]:
        assert torch.equal(op, results[0][0]) and torch.equal(lse, results[0][1])
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", HALVED, ids=lambda s: "x".join(map(str, s)))
def test_sink_rows_in_halves(shape):
    """A layer whose all-column rows, and last rows, run as halves beside whole ones: every row is written, as softmax attention
    over its kept blocks."""
    tokens, text, block, block_k, heads = shape
    print(f"[case] {shape}", flush=True)
    n, d = tokens + text, 128
    plan = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, text_tokens=text, block=block, block_k=block_k, sparsity=0.7,
                    window=(1, 1, 16))
    i = plan.info
    g = torch.Generator().manual_seed(13)
    q, k, v = (torch.randn(1, heads, n, d, generator=g).to(torch.bfloat16) for _ in range(3))
    buf = plan.alloc("cuda", lse=True)
    plan.rf2_permute(*(x.cuda() for x in (q, k, v)), *(buf[x] for x in ("qp", "kp", "vp", "qbar", "kbar")))
    mask = torch.empty(1, heads, i.n_blocks, i.n_blocks_k, dtype=torch.uint8, device="cuda")
    plan.rf2_predict_mask(buf["qbar"], buf["kbar"], buf["blk_idx"], buf["blk_cnt"], mask)
    buf["op"].fill_(float("nan"))
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], buf["blk_idx"], buf["blk_cnt"], buf["op"], buf["lse"])
    o, lse = torch.full_like(buf["o"], float("nan")), torch.full((1, heads, n), float("nan"), device="cuda")
    plan.rf2_block_sparse_attn_unpermuted(buf["qp"], buf["kp"], buf["vp"], buf["blk_idx"], buf["blk_cnt"], o, lse)
    torch.cuda.synchronize()
    perm = plan.rf2_plan_perm()[0]
    assert torch.equal(o[:, :, perm].view(torch.int16), buf["op"][:, :, :n].view(torch.int16))
    assert torch.equal(lse[:, :, perm], buf["lse"][:, :, :n])
    for h in range(heads):
        Q, K, V = (x[0, h][perm].double() for x in (q, k, v))
        keep = mask[0, h].cpu().bool().repeat_interleave(block, 0).repeat_interleave(block_k, 1)[:n, :n]
        S = (Q @ K.T / d ** 0.5).masked_fill(~keep, -torch.inf)
        P = torch.softmax(S, 1)
        want = P @ V
        err = (buf["op"][0, h, :n].cpu().double() - want).abs()
        # probabilities and outputs rounded to bf16 (2^-8 each, relative); logits below 10 in fp32
        assert (err <= 2.0 ** -8 * (P @ V.abs() + want.abs()) + 1e-4).all(), (h, err.max())
        assert (buf["lse"][0, h, :n].cpu().double() - torch.logsumexp(S, 1)).abs().max() <= 1e-4, h
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("case", TABLE, ids=lambda c: "x".join(str(v) for _, v in c))
def test_halves_of_rows_dealt_by_the_work_table(case):
    """Every row of every head is written, by both exits alike, as softmax attention over its kept blocks."""
    print(f"[case] {case}", flush=True)
    plan = rf2.Plan(**dict(dict(batch=1, head_dim=128, T=1, H=1, window=(1, 1, 16)), **dict(case)))
    i, c, d = plan.info, plan.cfg, 128
    n, heads, block, block_k = i.N, c.heads, c.block, i.block_k
    g = torch.Generator(device="cuda").manual_seed(17)
    q, k, v = (torch.randn(1, heads, n, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    buf = plan.alloc("cuda", lse=True)
    plan.rf2_permute(q, k, v, *(buf[x] for x in ("qp", "kp", "vp", "qbar", "kbar")))
    plan.rf2_predict_mask(buf["qbar"], buf["kbar"], buf["blk_idx"], buf["blk_cnt"])
    buf["op"].fill_(float("nan"))
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], buf["blk_idx"], buf["blk_cnt"], buf["op"], buf["lse"])
    o, lse = torch.full_like(buf["o"], float("nan")), torch.full((1, heads, n), float("nan"), device="cuda")
    plan.rf2_block_sparse_attn_unpermuted(buf["qp"], buf["kp"], buf["vp"], buf["blk_idx"], buf["blk_cnt"], o, lse)
    perm = torch.from_numpy(plan.rf2_plan_perm()[0]).cuda().long()
    assert torch.equal(o[:, :, perm].view(torch.int16), buf["op"][:, :, :n].view(torch.int16))
    assert torch.equal(lse[:, :, perm], buf["lse"][:, :, :n])
    idx, cnt = buf["blk_idx"].cpu(), buf["blk_cnt"].cpu()
    inside = torch.arange(block_k)
    for h in range(heads):
        Q, K, V = (x[0, h][perm].double() for x in (q, k, v))
        over, off = [], []
        for r in range(i.n_blocks):
            rows = slice(r * block, min((r + 1) * block, n))
            cols = torch.arange(i.n_blocks_k) if cnt[0, h, r] == i.n_blocks_k else idx[0, h, r, :cnt[0, h, r]].long()
            keys = (cols[:, None] * block_k + inside).flatten()
            keys = keys[keys < n].cuda()
            S = Q[rows] @ K[keys].T.contiguous() / d ** 0.5
            P = torch.softmax(S, 1)
            want = P @ V[keys]
            err = (buf["op"][0, h, rows].double() - want).abs()
            # probabilities and outputs rounded to bf16 (2^-8 each, relative); logits below 10 in fp32.  (No number: not below)
            over.append((~(err <= 2.0 ** -8 * (P @ V[keys].abs() + want.abs()) + 1e-4)).any())
            off.append((buf["lse"][0, h, rows].double() - torch.logsumexp(S, 1)).abs().max())
        assert not torch.stack(over).any(), (h, torch.stack(over).nonzero().flatten()[:8])
        assert torch.stack(off).max() <= 1e-4, h
    plan.close()


# (rows and columns of the grid, block, block_k, head_dim, heads) -> (rows of a workgroup, wavefronts that share a list)
GRIDS = {(15, 22, 64, 64, 128, 200): (64, 1), (49, 50, 128, 64, 128, 12): (64, 2), (9, 73, 64, 64, 128, 1): (64, 4),
         (58, 69, 128, 128, 128, 41): (128, 1), (71, 87, 128, 64, 128, 5): (128, 2), (49, 50, 128, 64, 128, 27): (128, 1),
         (270, 280, 256, 128, 128, 40): (256, 1), (27, 37, 64, 64, 64, 100): (64, 1), (30, 50, 64, 64, 64, 23): (64, 2),
         (9, 73, 64, 64, 64, 17): (64, 4), (49, 50, 64, 64, 64, 1): (64, 8), (49, 50, 128, 128, 64, 24): (128, 2)}


def grid_plan(shape):
    h, w, block, block_k, d, heads = shape
    return rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=h, W=w, block=block, block_k=block_k, sparsity=0.3, window=(1, 8, 8),
                    qkv_layout=rf2.RF2_LAYOUT_BNHD)


def test_cuts_of_the_grids(tmp_path):
    (tmp_path / "cut.cpp").write_text(SOURCE)
    lib = str(tmp_path / "cut.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", os.path.join(b.ROOT, "include"),
                    "-I", b.CSRC, str(tmp_path / "cut.cpp"), "-o", lib], check=True)
    fn, out = C.CDLL(lib).cut, (C.c_int * 5)()
    for shape, want in GRIDS.items():
        plan = grid_plan(shape)
        fn(C.byref(plan.cfg), C.byref(plan.info), out)
        assert tuple(out)[:2] == want and (out[3] > 0) == (shape[:2] == (49, 50) and shape[5] == 27), shape
        assert plan.info.N % shape[2], shape                          # a ragged last block
        assert plan.rf2_plan_perm()[0].tolist() != list(range(plan.info.N)), shape
        plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", GRIDS, ids=lambda s: "x".join(map(str, s)))
def test_rows_land_where_they_belong(shape):
    """Output rows leave a wavefront whole, 16 bytes a lane: of a permuted grid, token-major, behind an address that is a multiple of 8
    bytes only, with a ragged last block, they are those of the plain exit in the tokens' own places, so are the log-sum-exps, nothing
    beside them is written, and they are softmax attention over the kept blocks."""
    block, block_k, d, heads = shape[2:]
    print(f"[case] {shape}", flush=True)
    plan = grid_plan(shape)
    i = plan.info
    tokens = i.N
    g = torch.Generator(device="cuda").manual_seed(19)
    q, k, v = (torch.randn(1, tokens, heads, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    idx, cnt = hp.lists_to_device(cut_tests.lists(plan, 7), i.k_row, i.n_blocks, "cuda")
    buf = plan.alloc("cuda", lse=True)
    plan.rf2_permute(q, k, v, buf["qp"], buf["kp"], buf["vp"])
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], idx, cnt, buf["op"], buf["lse"])
    n = tokens * heads * d
    around = torch.full((n + 512,), 7.5, dtype=torch.bfloat16, device="cuda")
    o = around[260:260 + n].view(1, tokens, heads, d)
    assert o.data_ptr() % 16 == 8
    lse_around = torch.full((heads * tokens + 128,), 7.5, device="cuda")
    lse = lse_around[64:64 + heads * tokens].view(1, heads, tokens)
    plan.rf2_block_sparse_attn_unpermuted(buf["qp"], buf["kp"], buf["vp"], idx, cnt, o, lse)
    perm = torch.from_numpy(plan.rf2_plan_perm()[0]).cuda().long()
    assert (perm != torch.arange(tokens, device="cuda")).any()
    assert torch.equal(o[:, perm].transpose(1, 2).view(torch.int16), buf["op"][:, :, :tokens].view(torch.int16))
    assert torch.equal(lse[:, :, perm], buf["lse"][:, :, :tokens])
    assert (around[:260] == 7.5).all() and (around[260 + n:] == 7.5).all()
    assert (lse_around[:64] == 7.5).all() and (lse_around[64 + heads * tokens:] == 7.5).all()
    inside = torch.arange(block_k)
    for h in sorted({0, heads - 1}):
        Q, K, V = (x[0, :, h][perm].double() for x in (q, k, v))
        for r in sorted({*range(0, i.n_blocks, max(1, i.n_blocks // 60 | 1)), i.n_blocks - 1}):
            rows = slice(r * block, min((r + 1) * block, tokens))
            count = int(cnt[0, h, r])
            cols = torch.arange(i.n_blocks_k) if count == i.n_blocks_k else idx[0, h, r, :count].long().cpu()
            keys = (cols[:, None] * block_k + inside).flatten()
            keys = keys[keys < tokens].cuda()
            got, got_lse = o[0, perm[rows], h].double(), lse[0, h, perm[rows]].double()
            if len(keys) == 0:
                assert not got.any() and torch.isneginf(got_lse).all(), (h, r)
                continue
            S = Q[rows] @ K[keys].T.contiguous() / d ** 0.5
            P = torch.softmax(S, 1)
            want = P @ V[keys]
            # probabilities and outputs rounded to bf16 (2^-8 each, relative); logits below 10 in fp32
            assert ((got - want).abs() <= 2.0 ** -8 * (P @ V[keys].abs() + want.abs()) + 1e-4).all(), (h, r)
            assert (got_lse - torch.logsumexp(S, 1)).abs().max() <= 1e-4, (h, r)
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(330, 64, 64, 128, 200), (2450, 128, 64, 128, 12), (657, 64, 64, 128, 1), (4001, 128, 128, 128, 41),
                                   (6177, 128, 64, 128, 5), (999, 64, 64, 64, 100), (1500, 64, 64, 64, 23), (657, 64, 64, 64, 17),
                                   (2450, 64, 64, 64, 1), (2450, 128, 128, 64, 24)], ids=lambda s: "x".join(map(str, s)))
def test_reference_moves_in_any_unit(shape):
    """Keys that outweigh all before them by more than 2^40 in one, two and three units of 32: the first ones of a head, the last
    ones with the ragged end, any others; also in units of the last block that lie behind the end of a wavefront's share."""
    tokens, block, block_k, d, heads = shape
    print(f"[case] {shape}", flush=True)
    plan = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3, window=(1, 1, 16))
    i = plan.info
    g = torch.Generator(device="cuda").manual_seed(23)
    q, k, v = (torch.randn(1, heads, tokens, d, generator=g, device="cuda") for _ in range(3))
    perm = torch.from_numpy(plan.rf2_plan_perm()[0]).cuda().long()
    units = (tokens + 31) // 32
    factor = torch.ones(heads, units, device="cuda")
    for h in range(heads):
        at = torch.randperm(units, generator=torch.Generator().manual_seed(h))[:3].sort()[0]
        at = torch.arange(3) if h == heads - 1 and heads > 1 else torch.arange(units - 3, units) if h == 0 else at
        factor[h, at] = torch.tensor([8.0, 20.0, 50.0], device="cuda")
    k[0][:, perm] *= factor.repeat_interleave(32, 1)[:, :tokens, None]
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    idx, cnt = hp.lists_to_device(cut_tests.lists(plan, 11), i.k_row, i.n_blocks, "cuda")
    buf = plan.alloc("cuda", lse=True)
    plan.rf2_permute(q, k, v, buf["qp"], buf["kp"], buf["vp"])
    buf["op"].fill_(float("nan"))
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], idx, cnt, buf["op"], buf["lse"])
    inside = torch.arange(block_k)
    for h in sorted({0, 1 % heads, heads // 2, heads - 1}):
        Q, K, V = (x[0, h][perm].double() for x in (q, k, v))
        for r in range(i.n_blocks):
            rows = slice(r * block, min((r + 1) * block, tokens))
            count = int(cnt[0, h, r])
            cols = torch.arange(i.n_blocks_k) if count == i.n_blocks_k else idx[0, h, r, :count].long().cpu()
            keys = (cols[:, None] * block_k + inside).flatten()
            keys = keys[keys < tokens].cuda()
            if len(keys) == 0:
                assert not buf["op"][0, h, rows].any(), (h, r)
                continue
            S = Q[rows] @ K[keys].T.contiguous() / d ** 0.5
            P = torch.softmax(S, 1)
            want = P @ V[keys]
            err = (buf["op"][0, h, rows].double() - want).abs()
            # probabilities and outputs rounded to bf16 (2^-8 each, relative); logits of 300 in fp32: 2^-24 x 300 a rounding, sums of
            # up to 128 products, the scale and the difference among them: 2e-3 of a probability
            assert (err <= (2.0 ** -8 + 2e-3) * (P @ V[keys].abs()) + 2.0 ** -8 * want.abs() + 1e-4).all(), (h, r, err.max())
            assert (buf["lse"][0, h, rows].double() - torch.logsumexp(S, 1)).abs().max() <= 2e-3, (h, r)
    plan.close()


def test_where_shares_meet(tmp_path):
    """Four shares of a list meet in launches of long lists over a long sequence, and only there."""
    (tmp_path / "cut.cpp").write_text("""#include "rf2_attn_cut.h"
extern "C" int meets(const rf2_config* c, const rf2_info* i) { return rf2_cut_stream(*c, *i).meets; }
""")
    lib = str(tmp_path / "cut.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", os.path.join(b.ROOT, "include"),
                    "-I", b.CSRC, str(tmp_path / "cut.cpp"), "-o", lib], check=True)
    fn = C.CDLL(lib).meets

    def meets(**kw):
        plan = rf2.Plan(**dict(dict(batch=1, heads=2, head_dim=128, T=1, H=1, W=57344, block=64, sparsity=0.5, window=(1, 1, 16)), **kw))
        found = fn(C.byref(plan.cfg), C.byref(plan.info)), plan.info.k_row
        plan.close()
        return found

    assert meets() == (1, 448) and meets(block_k=128) == (1, 224) and meets(batch=2, heads=1) == (1, 448)           # 28 MB of a head's K and V, 40 of all
    assert meets(W=57280) == (0, 447)
    assert meets(sparsity=0.7142) == (1, 256) and meets(sparsity=0.715) == (0, 255)      # 256 parts
    assert meets(block_k=128, sparsity=0.7142) == (1, 128) and meets(block_k=128, sparsity=0.715) == (0, 127)
    assert meets(heads=1, W=81920)[0] == 1 and meets(heads=1, W=81856)[0] == 0
    assert meets(heads=5)[0] == 1 and meets(heads=6)[0] == 0 and meets(batch=3, heads=2)[0] == 0
    assert meets(heads=6, W=90112)[0] == 1 and meets(heads=7, W=90048)[0] == 0 and meets(heads=8, W=118784)[0] == 0     # 44 MB each
    assert meets(cdf_threshold=0.7)[0] == 0 and meets(head_dim=64, W=118784)[0] == 0
    assert meets(block=128)[0] == 0 and meets(block=256, block_k=128)[0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(236, 243, 64, 2), (236, 243, 128, 3), (280, 205, 128, 2)], ids=lambda s: "x".join(map(str, s)))
def test_shares_that_meet(shape):
    """Lists of none, one to three, k_row and all blocks, with a last block of 4 keys (whose second part no wavefront has, of 128-key blocks) or 56:
    wavefronts with no part, with a part less than others and with many, as softmax attention over the kept blocks, by both exits."""
    rows_of_grid, columns, block_k, heads = shape
    print(f"[case] {shape}", flush=True)
    tokens, d = rows_of_grid * columns, 128
    plan = rf2.Plan(batch=1, heads=heads, head_dim=d, T=1, H=rows_of_grid, W=columns, block=64, block_k=block_k, sparsity=0.6, window=(1, 8, 8))
    i = plan.info
    assert i.k_row * block_k >= 256 * 64 and i.N_pad_k * 512 >= 28 << 20       # (as test_where_shares_meet has it)
    g = torch.Generator(device="cuda").manual_seed(29)
    q, k, v = (torch.randn(1, heads, tokens, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    idx, cnt = hp.lists_to_device(cut_tests.lists(plan, 13), i.k_row, i.n_blocks, "cuda")
    buf = plan.alloc("cuda", lse=True)
    plan.rf2_permute(q, k, v, buf["qp"], buf["kp"], buf["vp"])
    buf["op"].fill_(float("nan"))
    plan.rf2_block_sparse_attn(buf["qp"], buf["kp"], buf["vp"], idx, cnt, buf["op"], buf["lse"])
    o, lse = torch.full_like(buf["o"], float("nan")), torch.full((1, heads, tokens), float("nan"), device="cuda")
    plan.rf2_block_sparse_attn_unpermuted(buf["qp"], buf["kp"], buf["vp"], idx, cnt, o, lse)
    perm = torch.from_numpy(plan.rf2_plan_perm()[0]).cuda().long()
    assert (perm != torch.arange(tokens, device="cuda")).any()
    assert torch.equal(o[:, :, perm].view(torch.int16), buf["op"][:, :, :tokens].view(torch.int16))
    assert torch.equal(lse[:, :, perm], buf["lse"][:, :, :tokens])
    inside = torch.arange(block_k)
    for h in range(heads):
        Q, K, V = (x[0, h][perm].double() for x in (q, k, v))
        for r in (*range(0, i.n_blocks, 13), *range(i.n_blocks - 6, i.n_blocks)):
            rows = slice(r * 64, min((r + 1) * 64, tokens))
            count = int(cnt[0, h, r])
            cols = torch.arange(i.n_blocks_k) if count == i.n_blocks_k else idx[0, h, r, :count].long().cpu()
            keys = (cols[:, None] * block_k + inside).flatten()
            keys = keys[keys < tokens].cuda()
            if len(keys) == 0:
                assert not buf["op"][0, h, rows].any() and torch.isneginf(buf["lse"][0, h, rows]).all(), (h, r)
                continue
            S = Q[rows] @ K[keys].T.contiguous() / d ** 0.5
            P = torch.softmax(S, 1)
            want = P @ V[keys]
            err = (buf["op"][0, h, rows].double() - want).abs()
            # probabilities and outputs rounded to bf16 (2^-8 each, relative); logits below 10 in fp32
            assert (err <= 2.0 ** -8 * (P @ V[keys].abs() + want.abs()) + 1e-4).all(), (h, r, err.max())
            assert (buf["lse"][0, h, rows].double() - torch.logsumexp(S, 1)).abs().max() <= 1e-4, (h, r)
    plan.close()
