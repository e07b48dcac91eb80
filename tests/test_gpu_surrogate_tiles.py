"""Surrogate expansion of few, many and very small leaves, bit for bit.

Up to eight leaves take tiles of 32 rows with the features formed in the tile,
more of them tiles of 128 rows leaf by leaf, and many leaves of few rows a
features pass of their own; RockSample leaves value the distinct successors
only.  Whichever it is, the value of an (action, scenario) is the forward pass
over the features of its stepped state, and a child's l0 is the same as when
its leaf is expanded alone.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import bits, cfg_pair, gpu_leaf_desc, ids_dev, to_dev

pytestmark = pytest.mark.gpu
HORIZON = 90


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


# (models, leaves, sizes): packs; leaf by leaf; a features pass of its own;
# grids of 5 and 31 cells, no rocks (five actions, five successors) and twenty
CASES = [
    (["rs15"], 3, [1, 5, 6]),
    (["rs15", "rs5", "ped6", "rs31"], 8, [22, 43, 300]),
    (["rs15"], 12, [64, 127, 128, 129, 300]),
    (["rs15", "rs5", "ped6", "rs31"], 30, [100, 213, 340]),
    (["rs15", "rs5", "ped6", "rs31"], 60, [1, 2, 5]),
    (["rs31"], 9, [2048]),
]
MODELS = {
    "rs15": lambda: W.rocksample_model(15, 15, 2),
    "rs5": lambda: W.rocksample_model(5, 0, 2),
    "rs31": lambda: W.rocksample_model(31, 20, 2),
    "ped6": lambda: W.pednav_model(6, 5, 3),
}


@pytest.mark.parametrize("case", CASES)
def test_surrogate_tiles(ctx, case):
    from paper_1802_06215_amd import Mlp, hdx as H
    names, count, sizes = case
    net = Mlp(ctx, seed=11)
    hcfg = cfg_pair(0, 50, HORIZON)[1]
    models = {k: ctx.upload_model(MODELS[k]()) for k in names}
    leaves, outs, keep = [], [], []
    for i in range(count):
        name = names[i % len(names)]
        desc, n = models[name].desc, sizes[i % len(sizes)]
        if name == "ped6":
            lf = W.pednav_leaf(desc, n + 3, n, 50 + i, p_term=0.1)
        else:
            lf = W.rocksample_leaf(desc, n + 3, n, 50 + i, depth=3 + i % 5, p_term=0.1, shared_cell=i % 2 == 0)
        parent, pids = to_dev(oracle.parent_states(desc, lf)), ids_dev(lf["ids"])
        leaf, out, k = gpu_leaf_desc(models[name], parent, pids, lf["idx"], lf["depth"], lf["last_action"], 7, 1, hcfg)
        leaves.append((leaf, models[name], lf["depth"], n))
        outs.append(out)
        keep.append((parent, pids, k))
    ctx.expand_leaf_surrogate([q[0] for q in leaves], net, HORIZON)
    torch.cuda.synchronize()
    together = [(o.child_l0.cpu().numpy().copy(), o.L.cpu().numpy().copy(), o.n_children.cpu().numpy().copy())
                for o in outs]
    for (leaf, m, depth, n), o, (l0, L, nc) in zip(leaves, outs, together):
        A = m.desc["n_actions"]
        sp = {k: v[..., :A * n].contiguous() for k, v in o.sprime.items()}
        y = net.forward(H.features(ctx, m, sp, torch.full((A * n,), depth + 1, dtype=torch.int32, device="cuda"), HORIZON))
        assert np.array_equal(bits(L[:, :n].reshape(-1)), bits(y.cpu().numpy()))
        ctx.expand_leaf_surrogate([leaf], net, HORIZON)
        torch.cuda.synchronize()
        alone = o.child_l0.cpu().numpy()
        for a in range(A):
            assert np.array_equal(bits(alone[a, :nc[a]]), bits(l0[a, :nc[a]]))
    net.close()
