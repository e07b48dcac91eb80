"""Tiles that take several actions of a leaf: many leaves in one batch (wide
tiles) against one-leaf calls (narrow tiles), bit for bit, and against the
oracle on some of them, at sizes around the 64-scenario chunks."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, collect, compare_leaf, gpu_leaf_desc, ids_dev, to_dev

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 127, 130]


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


def check(ctx, desc, make, count, cfgs, seed, sizes=SIZES, oracle_every=37):
    """`count` leaves of one model batched, alone and (every so many) by the oracle, per-pair outputs included."""
    from paper_1802_06215_amd import Batch
    m = ctx.upload_model(desc)
    items = []
    for i in range(count):
        n = sizes[i % len(sizes)]
        lf = make(desc, max(sizes), n, seed + i, depth=1 + i % 7)
        par_np = oracle.parent_states(desc, lf)
        par, pids = to_dev(par_np), ids_dev(lf["ids"])
        leaf, out, idx = gpu_leaf_desc(m, par, pids, lf["idx"], lf["depth"], lf["last_action"], seed, 2, cfgs[1],
                                       per_pair=i % 3 == 0)
        items.append((lf, par_np, leaf, out, (par, pids, idx)))
    for it in items:
        ctx.expand_leaf([it[2]])
    torch.cuda.synchronize()
    alone = [collect(m, it[3]) for it in items]
    for it in items:
        for f in ("child_u0", "child_l0", "r_mean", "perm", "n_children", "steps", "ids"):
            getattr(it[3], f).fill_(-7)
    b = Batch(ctx, count, count * desc["n_actions"])
    b.set_leaves([it[2] for it in items])
    b.launch()
    torch.cuda.synchronize()
    for i, it in enumerate(items):
        got = collect(m, it[3])
        for f in ("n_children", "perm", "steps", "ids"):
            assert np.array_equal(got[f], alone[i][f]), (i, f)
        for f in ("r_mean",) + (("r", "z", "U", "L", "child_of") if it[3].per_pair else ()):
            u, v = got[f], alone[i][f]
            assert np.array_equal(u.view(v.dtype), v) or np.array_equal(u.view(np.uint32), v.view(np.uint32)), (i, f)
        for a, nc in enumerate(got["n_children"]):
            for f in ("child_z", "child_n", "child_off", "child_u0", "child_l0"):
                u, v = got[f][a, :nc], alone[i][f][a, :nc]
                assert np.array_equal(u, v), (i, a, f)
        if i % oracle_every == 0:
            lf = it[0]
            ref = oracle.expand_leaf(desc, cfgs[0], it[1], lf["ids"].astype(np.uint32), lf["idx"], lf["depth"],
                                     lf["last_action"], seed, 2, per_pair=True)
            compare_leaf(desc, got, ref, len(lf["idx"]))
    b.close()


# (grid, landmarks, p_fail, policy, max_steps, max_depth, leaves): nine
# actions per tile from 256 leaves, three from 86; rollouts cut at 0, 1, 2
# and 300 steps (moves failing so often that a walk needs several windows of
# 64 failure words); the smallest and the largest map
NAV = [
    (13, 8, 0.03, 0, 1 << 30, 90, 260),
    (13, 8, 0.03, 0, 1 << 30, 90, 90),
    (13, 8, 0.9, 0, 300, -1, 260),
    (13, 8, 0.9, 0, 300, 120, 3),
    (16, 100, 0.1, 0, 1 << 30, 90, 260),
    (5, 1, 0.03, 0, 60, -1, 260),
    (13, 8, 0.03, 0, 0, -1, 260),
    (13, 8, 0.03, 0, 1, -1, 90),
    (13, 8, 0.03, 0, 2, -1, 3),
    (13, 8, 0.03, 2, 40, -1, 260),
    (13, 8, 0.03, 1, 20, -1, 90),
]


@pytest.mark.parametrize("case", NAV)
def test_navigation_tiles(ctx, case):
    grid, marks, p_fail, policy, steps, horizon, count = case
    desc = dict(W.nav_model(3, n=grid, n_landmarks=marks), p_fail=p_fail)
    check(ctx, desc, W.nav_leaf, count, cfg_pair(policy, steps, horizon, 4), 500)
