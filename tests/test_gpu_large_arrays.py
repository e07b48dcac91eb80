"""State arrays of more rows than one launch has threads for.

A launch is limited to 2^32 threads.  Calls that give a row several threads
(features: eight; driving bounds: four or more) take longer arrays in pieces.
"""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_06215_amd import Context
    c = Context(0)
    yield c
    c.close()


def room(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip("needs %d GiB of device memory" % gib)


def pieces(n):
    """The first rows, some in the middle, and the last, beyond the 2^32nd thread."""
    return [(0, 300), (n // 2 - 150, 300), (n - 300, 300)]


def test_features_of_many_rows(ctx):
    from paper_1802_06215_amd import hdx as H
    room(100)
    n = (1 << 29) + 40  # eight threads a row
    m = ctx.upload_model(W.rocksample_model(15, 15, 2))
    w = torch.randint(0, 1 << 25, (n,), dtype=torch.int32, device="cuda")
    depths = torch.randint(0, 90, (n,), dtype=torch.int32, device="cuda")
    X = H.features(ctx, m, dict(w=w), depths, 90)
    for at, count in pieces(n):
        want = H.features(ctx, m, dict(w=w[at:at + count].contiguous()), depths[at:at + count].contiguous(), 90)
        assert torch.equal(X[at:at + count], want)
    del X, w, depths
    torch.cuda.empty_cache()


def test_driving_bounds_of_many_states(ctx):
    from paper_1802_06215_amd import hdx as H
    room(60)
    n = (1 << 30) + 40  # four lanes a state
    m = ctx.upload_model(W.pednav_model(0, 5, 3))
    st = dict(s=torch.rand(n, device="cuda") * 40, car=torch.randint(0, 5, (n,), dtype=torch.int32, device="cuda"))
    st.update(px=torch.zeros((0, n), device="cuda"), py=torch.zeros((0, n), device="cuda"),
              goal=torch.zeros((0, n), dtype=torch.uint8, device="cuda"))
    ids = torch.randint(0, 500, (n,), dtype=torch.int32, device="cuda")
    depths = torch.randint(0, 50, (n,), dtype=torch.int32, device="cuda")
    cfg = H.rollout_cfg(0, 2, -1)
    got = ctx.rollout_bounds(m, cfg, st, ids, depths, 7, 1)
    for at, count in pieces(n):
        part = {k: v[..., at:at + count].contiguous() for k, v in st.items()}
        want = ctx.rollout_bounds(m, cfg, part, ids[at:at + count].contiguous(), depths[at:at + count].contiguous(), 7, 1)
        for g, w in zip(got, want):
            assert torch.equal(g[at:at + count], w)
    del got, st, ids, depths
    torch.cuda.empty_cache()
