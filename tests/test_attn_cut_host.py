"""How the attention launches of the GPU tests are cut, evaluated on the host: every kernel instance that a plan can
reach has to be among them."""
import ctypes as C
import itertools
import os
import subprocess

import pytest

from paper_2512_24086_amd import build as b
from paper_2512_24086_amd import rf2
from tests.test_gpu_attn_cut import NONFINITE, SHAPES

SOURCE = """#include "rf2_attn_cut.h"
extern "C" void cut(const rf2_config* c, const rf2_info* i, int* rows, int* groups) {
  const rf2_attn_cut x = rf2_cut_attn(*c, *i);
  *rows = x.rows;
  *groups = x.groups;
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    """(head_dim, rows of a workgroup, block_k, groups) of a plan's attention launch."""
    folder = tmp_path_factory.mktemp("cut")
    (folder / "cut.cpp").write_text(SOURCE)
    lib = str(folder / "cut.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I", os.path.join(b.ROOT, "include"),
                    "-I", b.CSRC, str(folder / "cut.cpp"), "-o", lib], check=True)
    fn = C.CDLL(lib).cut

    def of(plan):
        rows, groups = C.c_int(), C.c_int()
        fn(C.byref(plan.cfg), C.byref(plan.info), C.byref(rows), C.byref(groups))
        return plan.cfg.head_dim, rows.value, plan.info.block_k, groups.value
    return of


def plan_of(shape, **over):
    tokens, block, block_k, d, heads = shape
    return rf2.Plan(**dict(dict(batch=1, heads=heads, head_dim=d, T=1, H=1, W=tokens, block=block, block_k=block_k, sparsity=0.3,
                                window=(1, 1, 16)), **over))


def test_the_gpu_tests_reach_every_instance(cut):
    want = set(itertools.product((64, 128), (64, 128, 256), (64, 128), (1,))) \
        | set(itertools.product((64, 128), (64, 128), (64, 128), (2,))) | set(itertools.product((64,), (64, 128), (64, 128), (4,)))
    got = {cut(plan_of(s)) for s in SHAPES}
    assert got == want, (sorted(want - got), sorted(got - want))


def test_the_shapes_of_the_non_finite_tests_have_several_groups(cut):
    assert all(cut(plan_of(s))[3] > 1 for s in NONFINITE)
    assert {cut(plan_of(s))[3] for s in NONFINITE} == {2, 4}


# (tokens, block, block_k, head_dim, heads, sparsity) -> groups, rows of equal length.  What the busiest shader engine gets is
# behind it: at d = 128 two groups (at d = 64 four) leave one workgroup to a compute unit, 8 to an engine.
@pytest.mark.parametrize("shape, groups", [
    ((31 * 64, 64, 64, 128, 8, 0.0), 2), ((25 * 64, 64, 64, 128, 9, 0.0), 1), ((13 * 64, 64, 64, 128, 17, 0.0), 1),
    ((33 * 64, 64, 64, 128, 7, 0.0), 2), ((63 * 128, 128, 128, 128, 4, 0.3), 2), ((51 * 128, 128, 128, 128, 5, 0.3), 1),
    ((31 * 64, 64, 64, 64, 16, 0.5), 2), ((25 * 64, 64, 64, 64, 20, 0.5), 1), ((63 * 64, 64, 64, 64, 4, 0.3), 4),
    ((85 * 64, 64, 64, 64, 3, 0.3), 2), ((63 * 128, 128, 64, 64, 4, 0.3), 4), ((51 * 128, 128, 64, 64, 5, 0.3), 2)],
    ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_groups_only_where_every_engine_has_room(cut, shape, groups):
    *shape, sparsity = shape
    assert cut(plan_of(shape, sparsity=sparsity))[3] == groups


def video(**kw):
    return rf2.Plan(**dict(dict(batch=1, heads=20, head_dim=128, T=1, H=1, W=1, block=64, sparsity=0.8), **kw))


# many short rows beside a few all-column ones: workgroups by parts of the longest list decide
@pytest.mark.parametrize("kw, groups", [
    (dict(head_dim=64, H=53, W=77, text_tokens=269, sparsity=0.82), 2),              # 1,360 workgroups, 68 parts
    (dict(head_dim=64, H=43, W=102, heads=4, text_tokens=222, sparsity=0.86), 4),    # 288, 72
    (dict(head_dim=64, H=86, W=86, heads=40, text_tokens=244, sparsity=0.91, block_k=128), 1),     # 4,800, 120
    (dict(H=31, W=71, text_tokens=194, sparsity=0.77), 1),                           # 760, 38
    (dict(head_dim=64, T=26, H=5, W=13, heads=24, sink_frames=1, sparsity=0.51), 1), # 648, 27, hardly a tail
    (dict(head_dim=64, T=26, H=12, W=10, heads=32, sink_frames=1, sparsity=0.76), 1),        # 1,568, 49
    (dict(H=57, W=75, heads=10, text_tokens=300, sparsity=0.85), 2)])                # 720, 72
def test_groups_only_where_short_rows_are_few_beside_the_longest_list(cut, kw, groups):
    assert cut(video(**kw))[3] == groups


# cumulative mass, equal rows: the threshold says how many of the columns a flat row keeps
@pytest.mark.parametrize("shape, tau, groups", [
    ((29 * 64, 128, 64, 128, 2), 0.1, 1), ((29 * 64, 128, 64, 128, 2), 0.9, 2), ((25 * 64, 64, 64, 64, 1), 0.1, 1),
    ((71 * 64, 64, 64, 64, 5), 0.1, 1), ((71 * 64, 64, 64, 64, 3), 0.9, 4), ((12 * 64, 128, 64, 64, 2), 0.1, 1)])
def test_groups_of_cumulative_mass_launches_follow_the_threshold(cut, shape, tau, groups):
    assert cut(plan_of(shape, cdf_threshold=tau))[3] == groups


# 256-row Q blocks of equal length: two workgroups each where that fills the compute units better
@pytest.mark.parametrize("shape, rows", [
    ((65 * 256, 256, 128, 128, 1), 128), ((33 * 256, 256, 128, 128, 5), 256), ((65 * 256, 256, 128, 128, 4), 128),
    ((65 * 256, 256, 128, 128, 6), 256), ((9 * 256, 256, 128, 128, 14), 128), ((33 * 256, 256, 128, 128, 40), 256),
    ((65 * 256, 256, 128, 64, 3), 256), ((65 * 256, 256, 128, 64, 4), 128), ((65 * 256, 256, 128, 64, 6), 256),
    ((122 * 256, 256, 128, 64, 5), 256), ((65 * 256, 256, 128, 64, 40), 256)])
def test_halves_only_where_they_fill_the_compute_units_better(cut, shape, rows):
    assert cut(plan_of(shape, sparsity=0.5))[1] == rows
