"""Rock models with small discounts on the largest grid: the bounds' terms
10 gamma^d keep their relative precision however small they are.

Robots at the west edge of a 31-cell grid, so that the way out is 30 steps and
rocks are up to 60 away; scenarios whose rocks are all bad have the exit's term
alone.  The tolerance is that of every other comparison with the oracle (1e-5
of the value).
"""
import numpy as np
import pytest
import torch  # noqa: F401

import oracle
import workloads as W
from gpu_util import cfg_pair, compare_leaf, run_gpu_leaf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("gamma", [0.2, 0.3, 0.5, 0.7, 1.0])
@pytest.mark.parametrize("robots", [1, 2])
def test_bounds_of_far_robots(ctx, robots, gamma, shared):
    desc = (W.rocksample_model if robots == 1 else W.mars_model)(31, 20, 3, gamma)
    m = ctx.upload_model(desc)
    cfgs = cfg_pair(0, 1 << 30, 90)
    n = 40
    for seed in range(3):
        if robots == 1:
            lf = W.rocksample_leaf(desc, n, n, seed, p_term=0.1, shared_cell=shared)
            lf["x"] = 0 if shared else np.arange(n) % 3
        else:
            lf = W.mars_leaf(desc, n, n, seed, p_term=0.1, shared_cells=shared)
            x = np.zeros(n, np.int64) if shared else np.arange(n) % 3
            gone = [np.full(n, seed == 1, np.int64) | lf["term"], np.full(n, seed == 2, np.int64) | lf["term"]]
            lf["pos"] = (x, lf["pos"][1], x, lf["pos"][3], gone[0], gone[1])
        lf["rocks"][: n // 2] = False
        par = oracle.parent_states(desc, lf)
        gpu = run_gpu_leaf(ctx, m, par, lf["ids"], lf["idx"], 3, -1, 41, 3, cfgs[1], per_pair=seed == 0)
        ref = oracle.expand_leaf(desc, cfgs[0], par, lf["ids"].astype(np.uint32), lf["idx"], 3, -1, 41, 3, per_pair=True)
        compare_leaf(desc, gpu, ref, n)
