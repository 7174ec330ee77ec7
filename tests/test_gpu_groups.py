"""fnn_reciprocal on small maps with up to 256 seeds: one workgroup per 32 seeds walks them through all iterations.  Sizes at the
edges of its groups, tiles and chunks and on both sides of the lines; exactly representable maps, so everything equals
the oracle bit for bit, whichever route a call takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
from gpu_helpers import check_reciprocal_exact, dev, exact_maps, host

pytestmark = pytest.mark.gpu

FEW, MANY = {24: 280, 32: 180}, {24: 210, 32: 145}   # tiles, up to 64 workgroups and up to 256


def traced(a, b, seeds, max_iter, compute, **kw):
    fnn.fnn_trace_begin(256)
    try:
        out = fnn.fnn_reciprocal(a, b, seeds, max_iter=max_iter, compute=compute, **kw)
        torch.cuda.synchronize()
    finally:
        names = [name for name, _ in fnn.fnn_trace_end(256)]
    return {k: host(v) for k, v in out.items()}, "recip_groups_kernel" in names


@pytest.mark.parametrize("n,m,n_seeds,batch,max_iter,d,compute,kw,groups", [
    (1, 2, 97, 1, 10, 24, "f16", {}, True),                 # one tile; every seed the same pixel
    (513, 3000, 128, 3, 10, 24, "f16", {}, True),           # 17 and 94 tiles over 16 waves, whole groups
    (3000, 511, 129, 2, 10, 24, "bf16", {}, True),          # one seed in the last group
    (2100, 1999, 255, 1, 3, 10, "f16", {}, True),           # 16-channel rows
    (2100, 1999, 256, 1, 3, 30, "bf16", {}, True),          # 32-channel rows
    (2100, 1999, 257, 1, 3, 24, "f16", {}, False),
    (700, 650, 200, 2, 1, 24, "f16", {}, True),             # a single iteration
    (700, 650, 200, 2, 0, 24, "f16", {}, False),
    (700, 650, 256, 32, 4, 24, "f16", {}, True),            # a workgroup for every compute unit
    (700, 650, 225, 33, 4, 24, "f16", {}, False),
    (32 * FEW[24], 7000, 100, 16, 4, 24, "f16", {}, True),
    (32 * FEW[24] + 1, 7000, 100, 16, 4, 24, "f16", {}, False),
    (32 * MANY[24], 4100, 97, 17, 4, 24, "f16", {}, True),
    (32 * MANY[24] + 1, 4100, 97, 17, 4, 24, "f16", {}, False),
    (3000, 32 * FEW[32], 100, 1, 4, 32, "bf16", {}, True),
    (3000, 32 * FEW[32] + 1, 100, 1, 4, 32, "bf16", {}, False),
    (3000, 32 * MANY[32], 200, 10, 4, 32, "bf16", {}, True),
    (3000, 32 * MANY[32] + 1, 200, 10, 4, 32, "bf16", {}, False),
    (1500, 1400, 200, 2, 6, 24, "f16", {"l2": True}, True),
    (1500, 1400, 200, 2, 6, 24, "f32", {}, False),          # costly products keep the launch sequence
    (1500, 1400, 200, 2, 6, 24, "f16", {"split": True}, False),
])
def test_every_group_of_seeds_walks_like_the_oracle(n, m, n_seeds, batch, max_iter, d, compute, kw, groups):
    maps = [exact_maps(n + m + k, n, m, d) for k in range(min(batch, 3))]
    seeds = np.random.default_rng(n_seeds).integers(0, n, size=(len(maps), n_seeds)).astype(np.int32)
    pick = [k % len(maps) for k in range(batch)]
    a, b = (dev(np.stack([maps[k][side] for k in pick])) for side in (0, 1))
    got, took = traced(a, b, dev(seeds[pick]), max_iter, compute, **kw)
    assert took == groups
    for p in {0, batch // 2, batch - 1}:
        check_reciprocal_exact(got, p, oracle.reciprocal(*maps[pick[p]], seeds[pick[p]], max_iter, **({"metric": "l2"} if kw.get("l2") else {})))


@pytest.mark.parametrize("max_iter", [10, 40])
def test_seeds_that_move_to_the_last_iteration(max_iter):
    """The score along u, v, u + 1, v + 1, ... rises at every step: a seed moves one pixel on in every iteration."""
    d = 24
    a, b = np.zeros((960, d), dtype=np.float32), np.zeros((960, d), dtype=np.float32)
    b[:d] = np.eye(d)
    for t in range(d):
        a[t, t] = 2 * t + 1
        if t:
            a[t, t - 1] = 2 * t
    seeds = (np.arange(200, dtype=np.int32) % d)[None]
    got, took = traced(dev(a)[None], dev(b)[None], dev(seeds), max_iter, "f16")
    assert took
    assert np.array_equal(got["seed_i"][0], np.minimum(seeds[0] + max_iter - 1, d - 1))
    check_reciprocal_exact(got, 0, oracle.reciprocal(a, b, seeds[0], max_iter))


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_indices_stay_inside_maps_that_are_not_numbers(value):
    n, m, n_seeds = 3000, 2977, 200
    a, b = exact_maps(n, n, m, 24)
    a[::7], b[-1:] = value, value
    got, took = traced(dev(a)[None], dev(b)[None], dev(np.arange(n_seeds, dtype=np.int32) * 15)[None], 6, "f16")
    assert took
    assert got["seed_i"].min() >= 0 and got["seed_i"].max() < n and got["seed_j"].min() >= 0 and got["seed_j"].max() < m
    assert 0 <= got["n_pairs"][0] <= n_seeds


def test_maps_used_in_place_keep_the_launch_sequence():
    a, b = exact_maps(3, 1024, 992, 24)
    seeds = np.random.default_rng(1).integers(0, 1024, size=(1, 130)).astype(np.int32)
    want = oracle.reciprocal(a, b, seeds[0], 10)
    for dtype, groups in ((torch.float16, False), (torch.float32, True)):
        got, took = traced(dev(a)[None].to(dtype), dev(b)[None].to(dtype), dev(seeds), 10, "f16")
        assert took == groups
        check_reciprocal_exact(got, 0, want)
