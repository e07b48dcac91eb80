"""Driving calls keep to their own stream: a call does not wait for work that
another stream has still before it, and asks nothing about streams that are gone;
nor does staging a batch wait for the GPU.

A stream is kept busy with a spinning kernel of bounded length, and calls are
queued behind it.
"""
import ctypes
import threading
import time
from types import SimpleNamespace

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


def build(m, count, sizes, seed=60):
    items = []
    for i in range(count):
        n = sizes[i % len(sizes)]
        lf = W.pednav_leaf(m.desc, n + 2, n, seed + i, depth=1 + i % 5, p_term=0.1)
        par, pids = to_dev(oracle.parent_states(m.desc, lf)), ids_dev(lf["ids"])
        leaf, out, idx = gpu_leaf_desc(m, par, pids, lf["idx"], lf["depth"], lf["last_action"], seed, 2,
                                       cfg_pair(0, 9, -1, 1)[1], per_pair=False)
        items.append((leaf, out, (par, pids, idx)))
    torch.cuda.synchronize()
    return items


def wipe(items):
    for it in items:
        for f in FIELDS + CHILD:
            getattr(it[1], f).fill_(-7)
    torch.cuda.synchronize()


def same(a, b):
    for f in FIELDS:
        assert np.array_equal(a[f].view(np.uint8), b[f].view(np.uint8)), f
    for act, nc in enumerate(a["n_children"]):
        for f in CHILD:
            assert np.array_equal(a[f][act, :nc], b[f][act, :nc]), f


def spin_for(seconds):
    """Cycles of torch's spinning kernel that last about so long."""
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t = time.perf_counter()
    torch.cuda._sleep(1_000_000)
    torch.cuda.synchronize()
    return int(1_000_000 * seconds / (time.perf_counter() - t))


def busy_and_free():
    """Two streams of which the second runs while the first spins (streams may share a hardware queue)."""
    cycles = spin_for(0.3)
    busy = torch.cuda.Stream()
    for _ in range(8):
        free = torch.cuda.Stream()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(cycles)
            spun = torch.cuda.Event()
            spun.record()
        with torch.cuda.stream(free):
            torch.zeros(64, device="cuda")
        free.synchronize()
        apart = not spun.query()
        torch.cuda.synchronize()
        if apart:
            return busy, free, cycles
    pytest.skip("no two streams run side by side here")


def spin(busy, cycles):
    with torch.cuda.stream(busy):
        torch.cuda._sleep(cycles)
        spun = torch.cuda.Event()
        spun.record()
    return spun


@pytest.mark.parametrize("call", ["expand_leaf", "expand_leaf_noalloc"])
def test_a_call_does_not_wait_for_another_stream(ctx, call):
    m = ctx.upload_model(W.pednav_model(16, 5, 3))
    items = build(m, 12, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    busy, free, cycles = busy_and_free()
    wipe(items)
    spun = spin(busy, cycles)
    for it in items[:10]:
        getattr(ctx, call)([it[0]], busy)
    for it in items[10:]:
        getattr(ctx, call)([it[0]], free)
    free.synchronize()
    assert not spun.query(), "a call waited for the work of another stream"
    torch.cuda.synchronize()
    for it, r in zip(items, ref):
        same(collect(m, it[1]), r)


def test_more_streams_than_workspaces(ctx):
    """Seventy streams with calls in flight on all of them (more than there are workspaces), twice over."""
    hip = ctypes.CDLL("libamdhip64.so")
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    items = build(m, 140, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    # (torch's streams are drawn from a pool of 32)
    streams = []
    for _ in range(70):
        handle = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0
        streams.append(torch.cuda.ExternalStream(handle.value))
    for _ in range(2):
        wipe(items)
        for i, it in enumerate(items):
            ctx.expand_leaf([it[0]], streams[i % 70])
        torch.cuda.synchronize()
        for it, r in zip(items, ref):
            same(collect(m, it[1]), r)
    for s in streams:
        assert hip.hipStreamDestroy(ctypes.c_void_p(s.cuda_stream)) == 0


def test_streams_that_are_destroyed(ctx):
    """Streams destroyed with calls on them, new ones (which may get the same handles) right after: destroying a stream
    waits for its work, and nothing is asked about a stream that is gone."""
    hip = ctypes.CDLL("libamdhip64.so")
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    items = build(m, 30, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    wipe(items)
    cycles = spin_for(0.2)
    for i, it in enumerate(items):
        handle = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0
        stream = torch.cuda.ExternalStream(handle.value)
        if i == 0:
            with torch.cuda.stream(stream):
                torch.cuda._sleep(cycles)
        ctx.expand_leaf([it[0]], stream)
        t = time.perf_counter()
        assert hip.hipStreamDestroy(handle) == 0
        if i == 0:
            took = time.perf_counter() - t
            assert took > 0.1, took
    torch.cuda.synchronize()
    for it, r in zip(items, ref):
        same(collect(m, it[1]), r)


def test_the_per_thread_stream(ctx):
    """hipStreamPerThread is one handle for a stream of every thread: calls on it do not share a workspace."""
    per_thread = SimpleNamespace(cuda_stream=2)
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    items = build(m, 40, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    wipe(items)
    errors = []

    def work(t):
        try:
            for _ in range(3):
                for it in items[t::4]:
                    ctx.expand_leaf([it[0]], per_thread)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for it, r in zip(items, ref):
        same(collect(m, it[1]), r)


def test_calls_beside_a_capture(ctx):
    """Calls and staging on other threads while this one captures: neither the capture nor they are disturbed."""
    from paper_1802_06215_amd import Batch
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    items = build(m, 40, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    wipe(items)
    streams = [torch.cuda.Stream() for _ in range(12)]
    x = torch.ones(64, device="cuda")
    b = Batch(ctx, 20, 60)
    errors = []

    def work():
        try:
            for i, it in enumerate(items[:20]):
                ctx.expand_leaf([it[0]], streams[i % 12])
            b.set_leaves([it[0] for it in items[20:]], streams[0])
            b.launch(streams[0])
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        y = x * 2
        t = threading.Thread(target=work)
        t.start()
        t.join()
        y = y + 1
    assert not errors, errors
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(y, torch.full((64,), 3.0, device="cuda"))
    for it, r in zip(items, ref):
        same(collect(m, it[1]), r)
    b.close()


def test_staging_does_not_wait_for_the_gpu(ctx):
    from paper_1802_06215_amd import Batch
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    groups = [build(m, 9, [30, 13]), build(m, 40, [300, 20]), build(m, 200, [70])]
    refs = []
    for items in groups:
        for it in items:
            ctx.expand_leaf([it[0]])
        torch.cuda.synchronize()
        refs.append([collect(m, it[1]) for it in items])
        wipe(items)
    busy, free, cycles = busy_and_free()
    b = Batch(ctx, 200, 600)
    for items, ref in zip(groups, refs):
        spun = spin(busy, cycles)
        b.set_leaves([it[0] for it in items], free)
        waited = spun.query()
        b.launch(free)
        free.synchronize()
        for it, r in zip(items, ref):
            same(collect(m, it[1]), r)
        assert not waited, "staging waited for the work of another stream"
        torch.cuda.synchronize()
    b.close()


def test_calls_after_a_search(ctx):
    """A search's streams are gone when it returns: calls on other streams after it, and another search."""
    m = ctx.upload_model(W.pednav_model(6, 5, 3))
    items = build(m, 20, [100, 33, 250, 14])
    for it in items:
        ctx.expand_leaf([it[0]])
    torch.cuda.synchronize()
    ref = [collect(m, it[1]) for it in items]
    from paper_1802_06215_amd import hdx as H
    for batch in (0, 4):
        ctx.search(m, W.pednav_belief(m.desc), K=100, n_threads=8, batch_leaves=batch, max_trials=200, time_budget_s=5.0,
                   arena_bytes=1 << 28, rollout=H.rollout_cfg(0, 9, -1))
        wipe(items)
        for i, it in enumerate(items):
            ctx.expand_leaf([it[0]], torch.cuda.Stream() if i % 2 else None)
        torch.cuda.synchronize()
        for it, r in zip(items, ref):
            same(collect(m, it[1]), r)
