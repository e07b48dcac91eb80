"""A batch launch that the caller captured, replayed with other leaves staged.

The graph bakes in grids and LDS sizes; the number of leaves, their sizes (up to
the largest seen), their policy and with them the actions per tile and the values
that a tile holds may change between replays, under every schedule, with one
model or several.  Each replay is compared with one-leaf calls; the program's own
eager work runs in between.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, collect, gpu_leaf_desc, ids_dev, to_dev

pytestmark = pytest.mark.gpu

FIELDS = ("n_children", "perm", "steps", "ids", "r_mean")
CHILD = ("child_z", "child_n", "child_off", "child_u0", "child_l0")
SCHEDULES = [None, (256, 2, 0), (64, 0, 1), (128, 1, 1)]


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


MODELS = {
    "driving": (lambda: W.pednav_model(6, 5, 3), W.pednav_leaf),
    "rocks": (lambda: W.rocksample_model(7, 8, 3), W.rocksample_leaf),
    "two": (lambda: W.mars_model(7, 4, 3), W.mars_leaf),
    "nav": (lambda: W.nav_model(1), W.nav_leaf),
}
# what is staged at the capture and then, as (model, leaves, sizes, policy): more leaves than workspaces are for
# (driving), more actions per tile, values per scenario instead of shared ones, fewer and smaller leaves again; several
# models
CASES = {
    "driving": [[("driving", 9, [300, 13], 0)], [("driving", 530, [300, 14, 5, 13], 0)], [("driving", 40, [264], 2)],
                [("driving", 2, [300], 0)]],
    "rocks": [[("rocks", 12, [300, 40], 0)], [("rocks", 12, [300, 40], 2)], [("rocks", 300, [300, 64, 65, 1], 0)],
              [("rocks", 150, [290, 64], 1)]],
    "two": [[("two", 5, [130, 40], 0)], [("two", 5, [130, 40], 2)], [("two", 60, [130, 64, 65, 1], 0)],
            [("two", 60, [129, 64], 2)]],
    "nav": [[("nav", 9, [300, 40], 0)], [("nav", 9, [300, 40], 2)], [("nav", 270, [300, 64, 65, 1], 0)],
            [("nav", 270, [260, 64, 2], 2)], [("nav", 1, [300], 0)]],
    "several": [[("rocks", 12, [300], 0), ("driving", 9, [300], 0), ("nav", 9, [300], 0)],
                [("rocks", 12, [300, 2], 2), ("driving", 9, [300, 2], 2), ("nav", 9, [300, 2], 2)],
                [("rocks", 12, [1, 257], 1), ("driving", 9, [14, 300], 0), ("nav", 9, [260], 0)]],
}


def build(models, spec, seed):
    items = []
    for name, count, sizes, policy in spec:
        m = models[name]
        for i in range(count):
            n = sizes[i % len(sizes)]
            lf = MODELS[name][1](m.desc, n + 2, n, seed + i, depth=1 + i % 5, p_term=0.1)
            par, pids = to_dev(oracle.parent_states(m.desc, lf)), ids_dev(lf["ids"])
            leaf, out, idx = gpu_leaf_desc(m, par, pids, lf["idx"], lf["depth"], lf["last_action"], seed, 2,
                                           cfg_pair(policy, 9, 90, 1)[1], per_pair=False)
            items.append((leaf, out, (par, pids, idx), m))
    return items


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("case", list(CASES))
def test_replays_with_other_leaves(ctx, case, schedule):
    from paper_1802_06215_amd import Batch
    models = {k: ctx.upload_model(MODELS[k][0]()) for k in sorted({s[0] for spec in CASES[case] for s in spec})}
    groups = [build(models, spec, 60 + 500 * j) for j, spec in enumerate(CASES[case])]
    refs = []
    for items in groups:
        for it in items:
            ctx.expand_leaf([it[0]])
        torch.cuda.synchronize()
        refs.append([collect(it[3], it[1]) for it in items])
    most = max(len(g) for g in groups)
    b = Batch(ctx, most, most * 100)
    b.set_leaves([it[0] for it in groups[0]])
    if schedule:
        b.set_schedule(*schedule)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.launch()
    for j in list(range(len(groups))) + [0, 1]:
        items = groups[j]
        for it in items:
            for f in FIELDS + CHILD:
                getattr(it[1], f).fill_(-7)
        b.set_leaves([it[0] for it in items])
        for _ in range(2):
            g.replay()
            junk = torch.randn(1 << 12, device="cuda").sum()
        torch.cuda.synchronize()
        assert torch.isfinite(junk)
        for i, (it, r) in enumerate(zip(items, refs[j])):
            got = collect(it[3], it[1])
            for f in FIELDS:
                assert np.array_equal(got[f].view(np.uint8), r[f].view(np.uint8)), (j, i, f)
            for act, nc in enumerate(got["n_children"]):
                for f in CHILD:
                    u, v = got[f][act, :nc], r[f][act, :nc]
                    assert np.array_equal(u.view(np.uint8), v.view(np.uint8)), (j, i, act, f)
    b.close()
    torch.cuda.synchronize()


@pytest.mark.parametrize("schedule", [(256, 2, 0), (64, 1, 0)])
def test_one_persistent_graph_serves_any_number_of_leaves(ctx, schedule):
    """The library's own graph: driving leaves few and many, eager results between."""
    from paper_1802_06215_amd import Batch
    models = {"driving": ctx.upload_model(MODELS["driving"][0]())}
    b = Batch(ctx, 530, 530 * 3)
    b.use_graph(True)
    b.set_schedule(*schedule)
    for j, spec in enumerate(CASES["driving"] * 2):
        items = build(models, spec, 60 + 500 * j)
        for it in items:
            ctx.expand_leaf([it[0]])
        torch.cuda.synchronize()
        ref = [collect(it[3], it[1]) for it in items]
        for it in items:
            for f in FIELDS + CHILD:
                getattr(it[1], f).fill_(-7)
        b.set_leaves([it[0] for it in items])
        for _ in range(2):
            b.launch()
        torch.cuda.synchronize()
        for it, r in zip(items, ref):
            got = collect(it[3], it[1])
            for f in FIELDS:
                assert np.array_equal(got[f].view(np.uint8), r[f].view(np.uint8)), (j, f)
    b.close()
