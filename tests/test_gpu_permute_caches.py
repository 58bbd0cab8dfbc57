"""The permutation and its inverse on both sides of the sizes from which they stream past the caches: a layer of many heads is
bit for bit what its first and last head are on their own (the smallest layer, kept in the caches)."""
import os
import re

import pytest
import torch

from paper_2512_24086_amd import build as b
from paper_2512_24086_amd import rf2

TOKENS, BLOCK = 4099, 128           # ragged last blocks
# heads, d, token-major -> 2: what the permutation reads and writes is kept, 1: what it writes, 0: neither; what its inverse reads
CASES = {(13, 128, False): (2, True), (14, 128, True): (1, True), (26, 128, True): (1, True), (27, 128, False): (0, True),
         (26, 64, True): (2, True), (27, 64, False): (1, True), (52, 64, False): (1, True), (53, 64, True): (0, True),
         (95, 128, False): (0, True), (96, 128, True): (0, False), (191, 64, True): (0, True), (192, 64, False): (0, False)}


def test_the_cases_lie_on_both_sides_of_every_limit():
    text = open(os.path.join(b.CSRC, "rf2_permute.hip")).read()
    limit = {n: int(x) << 20 for n, x in re.findall(r"(KEEP_[A-Z]+) = \(int64_t\)(\d+) << 20", text)}
    padded = -(-TOKENS // BLOCK) * BLOCK
    for (heads, d, _), (keep, keep_inverse) in CASES.items():
        row = heads * d * 2
        moved = (3 * TOKENS + padded + 2 * padded) * row
        assert keep == (2 if moved <= limit["KEEP_ALL"] else 1 if moved <= limit["KEEP_STORES"] else 0), (heads, d, moved)
        assert keep_inverse == (2 * TOKENS * row <= limit["KEEP_UNPERMUTE"]), (heads, d)
    for d in (64, 128):
        assert {c[0] for (_, x, _), c in CASES.items() if x == d} == {0, 1, 2}


@pytest.mark.gpu
@pytest.mark.parametrize("heads, d, bnhd", CASES)
def test_sizes_around_the_limits(heads, d, bnhd):
    print(f"[case] {heads} heads d {d}", flush=True)
    cfg = dict(batch=1, head_dim=d, T=1, H=1, W=TOKENS, block=BLOCK, sparsity=0.5, window=(1, 1, 16),
               qkv_layout=rf2.RF2_LAYOUT_BNHD if bnhd else rf2.RF2_LAYOUT_BHND)
    g = torch.Generator(device="cuda").manual_seed(3)
    shape = (1, TOKENS, heads, d) if bnhd else (1, heads, TOKENS, d)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    names = ("qp", "kp", "vp", "qbar", "kbar")
    plan, one = rf2.Plan(heads=heads, **cfg), rf2.Plan(heads=1, **cfg)
    buf, part = plan.alloc(), one.alloc()
    plan.rf2_permute(q, k, v, *(buf[n] for n in names))
    plan.rf2_unpermute(buf["qp"], buf["o"])
    assert torch.equal(buf["o"], q)
    for h in (0, heads - 1):
        x = [(t[:, :, h:h + 1] if bnhd else t[:, h:h + 1]).contiguous() for t in (q, k, v)]
        one.rf2_permute(*x, *(part[n] for n in names))
        for n in names:
            assert torch.equal(buf[n][:, h], part[n][:, 0]), (n, h)
    plan.close()
    one.close()
