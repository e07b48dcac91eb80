"""Driving states whose speed level lies above the model's top (a state holds
eight bits of it): the car cannot accelerate, keeps its speed, and slows down by
a level when it brakes, in a leaf's expansion and in rollouts."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, close, compare_leaf, ids_dev, run_gpu_leaf, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("policy,action", [(0, 0), (1, 0), (1, 1), (1, 2), (2, 0)])
@pytest.mark.parametrize("peds", [3, 16])
def test_levels_above_the_top(ctx, peds, policy, action):
    desc = dict(W.pednav_model(peds, 5, 3), path_len=400.0)
    m = ctx.upload_model(desc)
    n = 70
    cfgs = cfg_pair(policy, 12, -1, action)
    for last in (-1, 0, 2):
        lf = W.pednav_leaf(desc, n, n, 9, depth=2, p_term=0.0)
        lf["level"] = (np.arange(n) % 12).astype(np.int32)  # the top is 4
        par = oracle.parent_states(desc, lf)
        gpu = run_gpu_leaf(ctx, m, par, lf["ids"], lf["idx"], 2, last, 41, 3, cfgs[1])
        ref = oracle.expand_leaf(desc, cfgs[0], par, lf["ids"].astype(np.uint32), lf["idx"], 2, last, 41, 3,
                                 per_pair=True)
        compare_leaf(desc, gpu, ref, n)
    depths = np.full(n, 2, np.int32)
    _, L, steps = ctx.rollout_bounds(m, cfgs[1], to_dev(par), ids_dev(lf["ids"]), torch.from_numpy(depths).cuda(), 41, 3)
    _, ref_l, ref_steps, scale = oracle.rollout_bounds(desc, cfgs[0], par, lf["ids"].astype(np.uint32), depths, 41, 3,
                                                       with_abs=True)
    assert np.array_equal(steps.cpu().numpy(), ref_steps)
    close(L.cpu().numpy(), ref_l, scale, "L")
