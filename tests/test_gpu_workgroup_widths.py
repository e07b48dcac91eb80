"""Rock tiles as wide as they get, under workgroup sizes that are no powers of
two: a schedule's width may be any multiple of 64, and no output depends on it.

A tile's children are spread over the workgroup's lanes (225 of them with 25
actions of two robots), so a width that does not divide the work evenly must
still reach every child.  All child outputs are wiped before each launch, and
compared with one-leaf calls (an action or a few per tile) and the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, collect, compare_leaf, gpu_leaf_desc, ids_dev, to_dev

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 130]
SCHEDULES = [(64, 0, 0), (128, 2, 0), (192, 0, 0), (192, 2, 0), (256, 0, 1), (320, 0, 0), (384, 0, 1), (448, 2, 0),
             (512, 0, 0)]
CHILD = ("child_z", "child_n", "child_off", "child_u0", "child_l0")
FIELDS = ("n_children", "perm", "steps", "ids", "r_mean")


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


# (robots, grid, rocks, policy, leaves): rows of 25, 16 and 5 actions of the
# second robot on one tile; one robot's 25 actions on one tile; values per
# scenario (a policy that runs step by step)
CASES = [
    (2, 20, 20, 0, 21),
    (2, 11, 11, 0, 32),
    (2, 7, 0, 0, 110),
    (2, 20, 20, 2, 21),
    (1, 31, 20, 0, 500),
]


@pytest.mark.parametrize("case", CASES)
def test_children_under_every_width(ctx, case):
    from paper_1802_06215_amd import Batch
    robots, grid, rocks, policy, count = case
    desc = (W.rocksample_model if robots == 1 else W.mars_model)(grid, rocks, 3)
    make = W.rocksample_leaf if robots == 1 else W.mars_leaf
    m = ctx.upload_model(desc)
    A = desc["n_actions"]
    # a tile takes a whole row only from this many (leaf, action) pairs on
    assert count * A > (5 + rocks - 1) * 2 * 256
    cfgs = cfg_pair(policy, 12 if policy else 1 << 30, 90)
    items = []
    for i in range(count):
        n = SIZES[i % len(SIZES)]
        lf = make(desc, max(SIZES), n, 40 + i, depth=1 + i % 7, p_term=0.1)
        par_np = oracle.parent_states(desc, lf)
        par, pids = to_dev(par_np), ids_dev(lf["ids"])
        leaf, out, idx = gpu_leaf_desc(m, par, pids, lf["idx"], lf["depth"], lf["last_action"], 40, 2, cfgs[1], False)
        items.append((lf, par_np, leaf, out, (par, pids, idx)))
    for it in items:
        ctx.expand_leaf([it[2]])
    torch.cuda.synchronize()
    alone = [collect(m, it[3]) for it in items]
    for i in range(0, count, 1 + count // 4):
        lf = items[i][0]
        ref = oracle.expand_leaf(desc, cfgs[0], items[i][1], lf["ids"].astype(np.uint32), lf["idx"], lf["depth"],
                                 lf["last_action"], 40, 2, per_pair=True)
        compare_leaf(desc, alone[i], ref, len(lf["idx"]))
    b = Batch(ctx, count, count * A)
    b.set_leaves([it[2] for it in items])
    for schedule in SCHEDULES:
        print("schedule", schedule, flush=True)
        for it in items:
            for f in CHILD + FIELDS:
                getattr(it[3], f).fill_(-7)
        b.set_schedule(*schedule)
        b.launch()
        torch.cuda.synchronize()
        for i, it in enumerate(items):
            got = collect(m, it[3])
            for f in FIELDS:
                assert np.array_equal(got[f].view(np.uint8), alone[i][f].view(np.uint8)), (schedule, i, f)
            for a, nc in enumerate(got["n_children"]):
                for f in CHILD:
                    u, v = got[f][a, :nc], alone[i][f][a, :nc]
                    assert np.array_equal(u.view(np.uint8), v.view(np.uint8)), (schedule, i, a, f)
    b.close()
