"""How the attention launches of the GPU tests are cut, evaluated on the host by the rule that the launches take: every kernel
instance of the dispatch has to be among them, and for products that are not finite every way to share a row's list."""
import ctypes as C
import os
import re
import subprocess

import pytest

from paper_2512_24086_amd import build as b
from paper_2512_24086_amd import inputs, rf2
from tests import test_gpu_attn_stream as stream
from tests import test_gpu_fullsize as fullsize
from tests.helpers import make_plan
from tests.test_gpu_attn_cut import NONFINITE, SHAPES

SOURCE = """#include "rf2_attn_cut.h"
extern "C" void cut(const rf2_config* c, const rf2_info* i, int* out) {
  const rf2_attn_cut x = rf2_cut_stream(*c, *i);
  out[0] = x.rows, out[1] = x.groups, out[2] = x.whole_slots > 0, out[3] = x.whole_heads;
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    """(head_dim, block_k, 64-row tiles of a workgroup, wavefronts that share a list, mixed) of a plan's attention launch."""
    folder = tmp_path_factory.mktemp("cut")
    (folder / "cut.cpp").write_text(SOURCE)
    lib = str(folder / "cut.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", os.path.join(b.ROOT, "include"),
                    "-I", b.CSRC, str(folder / "cut.cpp"), "-o", lib], check=True)
    fn = C.CDLL(lib).cut

    def of(plan):
        out = (C.c_int * 4)()
        fn(C.byref(plan.cfg), C.byref(plan.info), out)
        return plan.cfg.head_dim, plan.info.block_k, out[0] // 64, out[1], bool(out[2])
    return of


def plan_of(shape, **over):
    tokens, block, block_k, d, heads = shape
    return rf2.Plan(**dict(dict(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3,
                                window=(1, 1, 16)), **over))


def instances():
    """(head_dim, QH, KS) of the dispatch, and the pairs that may be mixed in a launch."""
    text = open(os.path.join(b.CSRC, "rf2_attn.hip")).read()
    body = text[text.index("int dispatch_cut("):]
    body = body[body.index("#define RF2_ATTN_CASE"):body.index("#undef RF2_ATTN_CASE")]
    both, rest = body.split("if constexpr (D == 128) {")
    of128, of64 = rest.split("} else {")
    found = {d: {(int(q), int(k)) for q, k in re.findall(r"RF2_ATTN_CASE\((\d), (\d)\)", both + own)}
             for d, own in ((128, of128), (64, of64))}
    assert found[128] >= {(1, 1), (2, 1)} and found[64] >= {(1, 1), (1, 8)}
    assert "if constexpr (D == 128 && QH == 2 && KS == 1)" in text      # (mixed_attn_kernel)
    return {(d, q, k) for d, pairs in found.items() for q, k in pairs}


def test_the_gpu_tests_reach_every_instance(cut):
    plans = [plan_of(s) for s in (*SHAPES, *stream.SHAPES, *stream.MIXED)]
    for (tokens, text, block, block_k, heads) in stream.HALVED:
        plans.append(plan_of((tokens, block, block_k, 128, heads), text_tokens=text, sparsity=0.7))
    for name in ("video720p_q256_k128", "video720p_q256_k64"):
        workload, sparsity, _ = fullsize.CASES[name]
        plans.append(make_plan(inputs.WORKLOADS[workload], sparsity=sparsity, **fullsize.EXTRA[name]))
    want = {(d, bk, q, k, False) for d, q, k in instances() for bk in (64, 128)} | {(128, bk, 2, 1, True) for bk in (64, 128)}
    got = {cut(p) for p in plans}
    assert got == want, (sorted(want - got), sorted(got - want))


def test_the_shapes_of_the_non_finite_tests_share_lists_in_every_way(cut):
    """(Four tiles of a 256-row block are two of 128 rows as far as a wavefront can see; only the largest launches have them.)"""
    want = {(d, q, k, False) for d, q, k in instances() if q < 4} | {(128, 2, 1, True)}
    got = {(c[0], *c[2:]) for c in map(cut, map(plan_of, NONFINITE))}
    assert got == want, (sorted(want - got), sorted(got - want))


# equal rows at d = 64, (tokens, heads, block, block_k, sparsity) -> one wavefront to a workgroup?  With more such workgroups than
# SIMDs, or than whole rounds and as many again, some SIMDs run two and the launch waits for those (us, 64 rows x 1 wavefront / best
# cut); with half of the places or nearly all of them taken it is the best cut, or as good
@pytest.mark.parametrize("shape, alone", [
    ((8424, 8, 256, 128, 0.61), False),         # 87.8 / 70.8
    ((6972, 10, 128, 0, 0.70), False),          # 58.8 / 49.2
    ((6090, 12, 128, 0, 0.59), False),          # 69.5 / 58.4
    ((11760, 6, 128, 0, 0.77), False),          # 76.8 / 63.8
    ((29412, 3, 128, 64, 0.89), False),         # 94.0 / 83.7
    ((10626, 19, 128, 0, 0.62), False),         # 237.5 / 216.5
    ((16256, 21, 256, 128, 0.61), False),       # 557.5 / 525.0
    ((2016, 32, 128, 0, 0.76), True),           # 13.5, the others 14.3 and more
    ((2450, 45, 256, 128, 0.65), True),         # 36.0, 38.5
    ((3025, 39, 256, 128, 0.83), True),         # 25.9, 28.8
    ((4320, 30, 128, 0, 0.66), True)],          # 55.6, 57.9
    ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else "")
def test_single_wavefronts_where_no_few_simds_hold_two(cut, shape, alone):
    tokens, heads, block, block_k, sparsity = shape
    assert (cut(plan_of((tokens, block, block_k, 64, heads), sparsity=sparsity))[2:4] == (1, 1)) is alone
