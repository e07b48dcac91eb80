"""Surrogate expansions whose leaves write their states to one buffer: a caller
that has no use for them may give every leaf the same, and the other outputs do
not depend on it."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, gpu_leaf_desc, ids_dev, to_dev

pytestmark = pytest.mark.gpu
HORIZON = 90


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


# packs, tiles leaf by leaf, a features pass of its own; all leaves on one
# buffer, neighbours overlapping by half, and one leaf inside another's
@pytest.mark.parametrize("layout", ["one", "half", "inside"])
@pytest.mark.parametrize("count,sizes", [(5, [1, 40, 200]), (20, [130, 257]), (30, [1, 2, 5])])
def test_states_on_one_buffer(ctx, count, sizes, layout):
    from paper_1802_06215_amd import Mlp
    net = Mlp(ctx, seed=3)
    desc = W.rocksample_model(15, 15, 2)
    m = ctx.upload_model(desc)
    rng = np.random.default_rng(4)
    leaves, outs, keep = [], [], []
    for i in range(count):
        n = sizes[i % len(sizes)]
        lf = W.rocksample_leaf(desc, n + 3, n, 70 + i, depth=3 + i % 5, p_term=0.1)
        par, pids = to_dev(oracle.parent_states(desc, lf)), ids_dev(lf["ids"])
        leaf, out, k = gpu_leaf_desc(m, par, pids, lf["idx"], lf["depth"], lf["last_action"], 7, 1,
                                     cfg_pair(0, 50, HORIZON)[1], per_pair=False)
        leaves.append(leaf)
        outs.append(out)
        keep.append((par, pids, k))

    def results():
        torch.cuda.synchronize()
        return [(o.child_l0.cpu().numpy().copy(), o.child_u0.cpu().numpy().copy(), o.n_children.cpu().numpy().copy())
                for o in outs]

    ctx.expand_leaf_surrogate(leaves, net, HORIZON)
    want = results()
    buf = torch.empty(max(sizes) * (count + 1), dtype=torch.int32, device="cuda")
    order = rng.permutation(count)
    for i, leaf in enumerate(leaves):
        at = {"one": 0, "half": int(order[i]) * (max(sizes) // 2), "inside": int(i == count // 2)}[layout]
        if layout == "inside" and i not in (0, count // 2):
            at = int(order[i] + 1) * max(sizes)
        leaf.states_out.w = buf.data_ptr() + 4 * at
        outs[i].child_l0.fill_(-7)
    ctx.expand_leaf_surrogate(leaves, net, HORIZON)
    for (l0, u0, nc), (wl0, wu0, wnc) in zip(results(), want):
        assert np.array_equal(nc, wnc)
        for a, k in enumerate(nc):
            assert np.array_equal(l0[a, :k].view(np.uint32), wl0[a, :k].view(np.uint32))
            assert np.array_equal(u0[a, :k], wu0[a, :k])
    net.close()
