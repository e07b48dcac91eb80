"""Rollouts run step by step and stand-alone bounds against the oracle.

Rollouts of more than 64 steps (the discount powers of a wavefront's lanes are
then read again), from different depths within one wavefront, cut at 0 and 1
steps; the smallest and largest grids, no rocks and the most, every lane split
of the driving model.  Steps equal; U and L as elsewhere: 1e-5 of the value, or
of the sum of the rewards' magnitudes.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, host, ids_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


MODELS = {
    "rs7": lambda: W.rocksample_model(7, 8, 3),
    "rs31": lambda: W.rocksample_model(31, 20, 3),
    "rs5": lambda: W.rocksample_model(5, 0, 3),
    "mars7": lambda: W.mars_model(7, 4, 3),
    "mars31": lambda: W.mars_model(31, 20, 3),
    "mars5": lambda: W.mars_model(5, 0, 3),
    "nav13": lambda: dict(W.nav_model(3, n=13, n_landmarks=8), p_fail=0.5),
    "nav16": lambda: W.nav_model(3, n=16, n_landmarks=100),
    "nav5": lambda: W.nav_model(3, n=5, n_landmarks=1),
    "ped0": lambda: W.pednav_model(0, 5, 3),
    "ped8": lambda: W.pednav_model(8, 5, 3),
    "ped9": lambda: W.pednav_model(9, 5, 3),
    "ped17": lambda: W.pednav_model(17, 5, 3),
    "ped32": lambda: W.pednav_model(32, 5, 3),
}


def states_of(name, desc, n):
    if name.startswith("rs"):
        lf = W.rocksample_leaf(desc, n, n, 5, shared_cell=False, p_term=0.1)
    elif name.startswith("mars"):
        lf = W.mars_leaf(desc, n, n, 5, shared_cells=False, p_term=0.1)
    elif name.startswith("nav"):
        lf = W.nav_leaf(desc, n, n, 5)
    else:
        lf = W.pednav_leaf(desc, n, n, 5, p_term=0.1)
    return oracle.parent_states(desc, lf), lf["ids"]


@pytest.mark.parametrize("name", sorted(MODELS))
@pytest.mark.parametrize("policy", [0, 1, 2])
def test_bounds(ctx, name, policy):
    desc = MODELS[name]()
    m = ctx.upload_model(desc)
    n = 259 if name.startswith("ped") else 1030
    st, ids = states_of(name, desc, n)
    depths = (np.arange(n) % 37).astype(np.int32)
    for steps, horizon in ((300, -1), (1 << 30, 90), (1, -1), (0, 90)):
        if name.startswith("ped") and steps == 300:
            steps = 70
        ocfg, hcfg = cfg_pair(policy, steps, horizon, 1 if name.startswith("ped") else 4)
        U, L, ns = ctx.rollout_bounds(m, hcfg, to_dev(st), ids_dev(ids), torch.from_numpy(depths).cuda(), 12, 1)
        torch.cuda.synchronize()
        rU, rL, rs, rabs = oracle.rollout_bounds(desc, ocfg, st, ids, depths, 12, 1, with_abs=True)
        assert np.array_equal(host(ns), rs), (steps, horizon)
        assert np.all(np.abs(host(U) - rU) <= 1e-5 * np.abs(rU) + 1e-30), (steps, horizon)
        assert np.all(np.abs(host(L) - rL) <= 1e-5 * np.maximum(np.abs(rL), rabs) + 1e-30), (steps, horizon)


@pytest.mark.parametrize("name", ["rs7", "rs31", "rs5", "mars7", "mars5", "nav13", "nav5"])
@pytest.mark.parametrize("count", [3, 120])
def test_tiles_of_long_rollouts(ctx, name, count):
    """Leaves expanded with constant and random rollouts of up to 200 steps: tiles of one and of several actions."""
    from test_gpu_tile_actions import check
    desc = MODELS[name]()
    make = {"rs": W.rocksample_leaf, "ma": W.mars_leaf, "na": W.nav_leaf}[name[:2]]
    for policy in (1, 2):
        check(ctx, desc, make, count, cfg_pair(policy, 200, -1, 3), 800, [1, 2, 7, 11, 64, 65, 130], oracle_every=29)
