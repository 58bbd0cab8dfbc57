"""The permutation and its inverse on both sides of the sizes from which they stream past the caches: a layer of many heads is
bit for bit what its first and last head are on their own (the smallest layer, kept in the caches)."""
import pytest
import torch

from paper_2512_24086_amd import rf2

pytestmark = pytest.mark.gpu


# heads of 4,099 tokens (ragged last blocks): bytes read and written in MB: 76 / 82, 158 / 164 of 80 and 160 kept by the
# permutation; 190 / 195 of 192 by its inverse
@pytest.mark.parametrize("heads, d, bnhd", [(12, 128, False), (13, 128, True), (25, 128, True), (26, 128, False), (51, 64, False),
                                            (52, 64, True), (95, 128, False), (97, 128, True)])
def test_sizes_around_the_limits(heads, d, bnhd):
    print(f"[case] {heads} heads d {d}", flush=True)
    cfg = dict(batch=1, head_dim=d, T=1, H=1, W=4099, block=128, sparsity=0.5, window=(1, 1, 16),
               qkv_layout=rf2.RF2_LAYOUT_BNHD if bnhd else rf2.RF2_LAYOUT_BHND)
    g = torch.Generator(device="cuda").manual_seed(3)
    shape = (1, 4099, heads, d) if bnhd else (1, heads, 4099, d)
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
