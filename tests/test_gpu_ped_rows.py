"""Driving leaves expanded by one workgroup each and by two kernels.

Few leaves take their scenarios to any free CU and group them in a second
kernel, with a workspace between the two; 512 leaves and more, leaves of up to
twelve scenarios, and captured calls take a workgroup per leaf.  Results are the
same bit for bit, with more calls in flight than there are workspaces, from
several threads and streams, in replayed graphs and under every schedule.
"""
import threading

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import cfg_pair, collect, gpu_leaf_desc, ids_dev, to_dev

pytestmark = pytest.mark.gpu

FIELDS = ("n_children", "perm", "steps", "ids", "r_mean")
CHILD = ("child_z", "child_n", "child_off", "child_u0", "child_l0")


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


def build(m, count, sizes, policy=0, seed=60):
    items = []
    for i in range(count):
        n = sizes[i % len(sizes)]
        lf = W.pednav_leaf(m.desc, n + 2, n, seed + i, depth=1 + i % 5, p_term=0.1)
        par, pids = to_dev(oracle.parent_states(m.desc, lf)), ids_dev(lf["ids"])
        leaf, out, idx = gpu_leaf_desc(m, par, pids, lf["idx"], lf["depth"], lf["last_action"], seed, 2,
                                       cfg_pair(policy, 9, -1, 1)[1], per_pair=i % 2 == 0)
        items.append((leaf, out, (par, pids, idx)))
    torch.cuda.synchronize()
    return items


def clear(items):
    for it in items:
        for f in FIELDS:
            getattr(it[1], f).fill_(-7)
        for f in CHILD:
            getattr(it[1], f).fill_(-7)
    torch.cuda.synchronize()


def same(a, b):
    for f in FIELDS:
        assert np.array_equal(a[f].view(np.uint8), b[f].view(np.uint8)), f
    for act, nc in enumerate(a["n_children"]):
        for f in CHILD:
            assert np.array_equal(a[f][act, :nc], b[f][act, :nc]), f


@pytest.mark.parametrize("peds,sizes", [(3, [13, 17, 30]), (16, [13, 40, 65]), (32, [12, 13, 33])])
def test_many_leaves_whole(ctx, peds, sizes):
    """520 leaves (a workgroup each), against one-leaf calls (two kernels) and the oracle."""
    from test_gpu_tile_actions import check
    check(ctx, W.pednav_model(peds, 5, 3), W.pednav_leaf, 520, cfg_pair(0, 9, -1, 1), 900, sizes, oracle_every=130)


def test_calls_in_flight_on_threads_and_streams(ctx):
    m = ctx.upload_model(W.pednav_model(16, 5, 3))
    items = build(m, 40, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    clear(items)
    errors = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            for _ in range(3):
                for i in range(t, len(items), 4):
                    if i % 8 == t:
                        ctx.expand_leaf_noalloc([items[i][0]], stream)
                    else:
                        ctx.expand_leaf([items[i][0]], stream)
            stream.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    torch.cuda.synchronize()
    for it, r in zip(items, ref):
        same(collect(m, it[1]), r)


def test_captured_calls(ctx):
    """A captured leaf replayed beside eager calls; captured together with many leaves of a staged call."""
    m = ctx.upload_model(W.pednav_model(16, 5, 3))
    items = build(m, 3, [100, 60, 13])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.expand_leaf([items[0][0]])
    for _ in range(3):
        clear(items)
        g.replay()
        ctx.expand_leaf([items[1][0], items[2][0]])
        torch.cuda.synchronize()
        for it, r in zip(items, ref):
            same(collect(m, it[1]), r)


def test_batches_that_change_size(ctx):
    """One batch object: few leaves, many, few again, larger ones; eager, as a graph, and under persistent schedules."""
    from paper_1802_06215_amd import Batch
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    groups = [build(m, 9, [30, 13]), build(m, 530, [14, 13], seed=700), build(m, 20, [12, 5]), build(m, 12, [300, 20]),
              build(m, 40, [64])]
    refs = []
    for items in groups:
        for it in items:
            ctx.expand_leaf([it[0]])
        torch.cuda.synchronize()
        refs.append([collect(m, it[1]) for it in items])
    for graph in (False, True):
        for schedule in (None, (256, 2, 0), (64, 0, 1)):
            b = Batch(ctx, 530, 530 * 3)
            b.use_graph(graph)
            for items, ref in zip(groups + groups[:1], refs + refs[:1]):
                clear(items)
                b.set_leaves([it[0] for it in items])
                if schedule:
                    b.set_schedule(*schedule)
                for _ in range(2):
                    b.launch()
                torch.cuda.synchronize()
                for it, r in zip(items, ref):
                    same(collect(m, it[1]), r)
            b.close()
