"""fnn_reciprocal on small pairs: the whole iteration runs in one workgroup per pair (search, reciprocity test,
compaction and the sorted match set behind workgroup barriers).  Sizes at the edges of its blocks, tiles and
chunks and on both sides of the line where the launch sequence takes over; exactly representable maps, so
everything must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
from gpu_helpers import check_reciprocal_exact, dev, exact_maps, host

pytestmark = pytest.mark.gpu


def traced(a, b, seeds, max_iter, compute, **kw):
    fnn.fnn_trace_begin(128)
    try:
        out = fnn.fnn_reciprocal([dev(x) for x in a], [dev(x) for x in b], dev(seeds), max_iter=max_iter, compute=compute, **kw)
        torch.cuda.synchronize()
    finally:
        kinds = [name for name, _ in fnn.fnn_trace_end(128)]
    return {k: host(v) for k, v in out.items()}, "recip_walk_kernel" in kinds


@pytest.mark.parametrize("compute,kw,d", [("f16", {}, 24), ("bf16", {}, 10), ("f32", {}, 24), ("f32", {}, 5), ("f16", {"split": True}, 24),
                                          ("f16", {"split": True}, 32), ("f16", {}, 32)])
@pytest.mark.parametrize("n,m,n_seeds,max_iter,walks", [    # walks: with 16 or 24 channels, with 32, with wide rows or fp32 products
    (1, 1, 1, 10, (True, True, True)),              # a single pixel on either side
    (33, 31, 33, 10, (True, True, False)),          # one pixel past a tile; 33 seeds: a second, nearly empty query block
    (500, 1537, 65, 3, (True, True, False)),        # 49 tiles over the chunks, 3 blocks
    (2048, 512, 64, 2, (True, True, False)),        # image 1 the larger one
    (512, 512, 256, 10, (False, False, False)),     # 8 blocks: the launch sequence
    (700, 768, 32, 10, (True, True, True)),         # both sides of the lines: 24 tiles, one block
    (769, 700, 32, 10, (True, True, False)),
    (3840, 3800, 30, 10, (True, True, False)),      # 120 tiles
    (3841, 3800, 30, 10, (True, False, False)),
    (5600, 5599, 33, 10, (True, False, False)),     # 175 tiles, two blocks
    (5601, 5599, 33, 10, (False, False, False)),
    (3072, 3071, 48, 0, (False, False, False)),     # no iteration allowed: the launch sequence
])
def test_small_pairs_walk_in_one_workgroup(compute, kw, d, n, m, n_seeds, max_iter, walks):
    maps = [exact_maps(n + m + k, n, m, d) for k in range(3)]
    rng = np.random.default_rng(n_seeds)
    seeds = rng.integers(0, n, size=(3, n_seeds)).astype(np.int32)
    got, walked = traced([x[0] for x in maps], [x[1] for x in maps], seeds, max_iter, compute, **kw)
    assert walked == walks[2 if compute == "f32" or kw else (1 if d > 24 else 0)]
    for p in range(3):
        check_reciprocal_exact(got, p, oracle.reciprocal(*maps[p], seeds[p], max_iter))


@pytest.mark.parametrize("n_seeds,walks", [(95, True), (96, True), (97, False), (1000, False), (1023, False), (1024, False), (1025, False)])
def test_both_sides_of_the_line_agree(n_seeds, walks):
    a, b = exact_maps(41, 992, 1000, 24)
    b = np.concatenate([b[:990], a[:10]])
    a, b = a[:960], b[:960]                   # 30 tiles: up to 3 blocks of seeds walk
    seeds = np.random.default_rng(3).integers(0, 960, size=(1, n_seeds)).astype(np.int32)
    got, walked = traced([a], [b], seeds, 10, "f16")
    assert walked == walks
    check_reciprocal_exact(got, 0, oracle.reciprocal(a, b, seeds[0], 10))


@pytest.mark.parametrize("n_seeds", [96, 256])       # one workgroup per pair, launch sequence
def test_seeds_that_move_to_the_last_iteration(n_seeds):
    """The slowest walk there is: the score along u, v, u + 1, v + 1, ... rises at every step, so a seed moves one pixel
    on in every iteration and none settles before the end of the chain."""
    d = 24
    a, b = np.zeros((960, d), dtype=np.float32), np.zeros((960, d), dtype=np.float32)
    b[:d] = np.eye(d)
    for t in range(d):
        a[t, t] = 2 * t + 1
        if t:
            a[t, t - 1] = 2 * t
    seeds = (np.arange(n_seeds, dtype=np.int32) % d)[None]
    for max_iter in (10, 40):
        got, walked = traced([a], [b], seeds, max_iter, "f16")
        assert walked == (n_seeds == 96)
        assert np.array_equal(got["seed_i"][0], np.minimum(seeds[0] + max_iter - 1, d - 1))
        check_reciprocal_exact(got, 0, oracle.reciprocal(a, b, seeds[0], max_iter))
