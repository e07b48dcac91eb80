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


# (pedestrians, policy, max_steps, sigma_h, speed, leaves, sizes): every lane
# split (4, 8 and 16 lanes per scenario; 3, 8, 9, 16, 17, 32 pedestrians),
# sorts of one wavefront, one block and several, rollouts of 0, 1 and 17
# steps, no heading noise and steps past every goal (the general operations)
DRIVING = [
    (3, 0, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (8, 0, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (9, 2, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 17, 0.3, 1.2, 40, [1, 2, 3, 4, 11, 12, 13]),
    (17, 1, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (32, 0, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (0, 0, 17, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 0, 0.3, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 1, 0.0, 1.2, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 17, 0.3, 90.0, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 17, 5.0, 0.0, 30, [1, 5, 16, 17, 64, 65, 130]),
    (16, 0, 5, 0.3, 1.2, 2, [257, 513, 1024, 2048]),
    (16, 0, 5, 0.3, 1.2, 300, [1, 130, 257]),
]


@pytest.mark.parametrize("case", DRIVING)
def test_driving_tiles(ctx, case):
    peds, policy, steps, sigma, speed, count, sizes = case
    desc = dict(W.pednav_model(peds, 5, 3), sigma_h=sigma, ped_speed=speed)
    check(ctx, desc, W.pednav_leaf, count, cfg_pair(policy, steps, -1, 1), 900, sizes)


def test_pedestrian_steps_at_the_ends_of_the_range(ctx):
    """Pedestrians on their goal, a hair from it, straight above it, and far away: the middle range of the step's
    root and quotients and the general operations beside it, bit for bit with the oracle."""
    desc = W.pednav_model(16, 5, 3)
    n = 64
    lf = W.pednav_leaf(desc, n, n, 5, depth=3)
    gx, gy = desc["goal_x"][lf["goal"]], desc["goal_y"][lf["goal"]]
    off = np.array([0.0, 1e-9, 1e-4, 0.5999999, 0.6, 0.6000001, 1.0, 1e6, 1e12, 1e25, -1e-40, 3e-30, 2.0, 1e19, -7.0, 0.0],
                   np.float32)[:, None]
    lf["px"] = (gx - off).astype(np.float32)
    lf["py"] = np.where(np.arange(n)[None, :] % 3 == 0, gy, np.where(np.arange(n)[None, :] % 3 == 1, gy - off, gy + 3)
                        ).astype(np.float32)
    m = ctx.upload_model(desc)
    cfgs = cfg_pair(0, 10)
    par = oracle.parent_states(desc, lf)
    from gpu_util import run_gpu_leaf
    for last in (-1, 0):
        gpu = run_gpu_leaf(ctx, m, par, lf["ids"], lf["idx"], lf["depth"], last, 41, 3, cfgs[1])
        ref = oracle.expand_leaf(desc, cfgs[0], par, lf["ids"].astype(np.uint32), lf["idx"], lf["depth"], last, 41, 3,
                                 per_pair=True)
        compare_leaf(desc, gpu, ref, n)


# (robots, grid, rocks, policy, max_steps, shared cells, leaves): tiles of one
# action up to a row; no rocks and the most; the shared-cell sums and the
# per-scenario ones; rollouts of 0 and 1 steps
ROCKS = [
    (1, 7, 8, 0, 1 << 30, True, 40),
    (1, 7, 8, 0, 1 << 30, True, 300),
    (1, 7, 8, 0, 1 << 30, False, 300),
    (1, 31, 20, 0, 1 << 30, True, 60),
    (1, 5, 0, 0, 1 << 30, True, 60),
    (1, 7, 8, 2, 30, True, 100),
    (1, 7, 8, 2, 30, False, 100),
    (1, 7, 8, 1, 30, True, 100),
    (1, 7, 8, 0, 0, True, 60),
    (1, 7, 8, 0, 1, False, 60),
    (2, 7, 4, 0, 1 << 30, True, 21),
    (2, 7, 4, 0, 1 << 30, True, 100),
    (2, 7, 4, 0, 1 << 30, False, 100),
    (2, 31, 20, 0, 1 << 30, True, 3),
    (2, 5, 0, 0, 1 << 30, True, 60),
    (2, 7, 4, 2, 20, True, 21),
    (2, 7, 4, 2, 20, False, 21),
    (2, 7, 4, 1, 20, True, 21),
    (2, 7, 4, 0, 1, False, 21),
]


@pytest.mark.parametrize("case", ROCKS)
def test_rock_tiles(ctx, case):
    robots, grid, rocks, policy, steps, shared, count = case
    desc = (W.rocksample_model if robots == 1 else W.mars_model)(grid, rocks, 3)
    if robots == 1:
        make = lambda d, n_par, n, seed, depth: W.rocksample_leaf(d, n_par, n, seed, depth=depth, shared_cell=shared,  # noqa: E731
                                                                  p_term=0.1)
    else:
        make = lambda d, n_par, n, seed, depth: W.mars_leaf(d, n_par, n, seed, depth=depth, shared_cells=shared,  # noqa: E731
                                                            p_term=0.1)
    # the constant policy samples (robot 2, when there are two)
    check(ctx, desc, make, count, cfg_pair(policy, steps, 90, 4), 700, oracle_every=11)


@pytest.mark.parametrize("n", [0, 1, 2048])
@pytest.mark.parametrize("robots", [1, 2])
def test_rock_tiles_at_the_ends(ctx, robots, n):
    desc = W.rocksample_model(7, 8, 3) if robots == 1 else W.mars_model(7, 4, 3)
    make = W.rocksample_leaf if robots == 1 else W.mars_leaf
    check(ctx, desc, make, 3, cfg_pair(0, 1 << 30, 90), 800, sizes=[n, max(n, 1)], oracle_every=1)
