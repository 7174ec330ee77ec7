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
@pytest.mark.parametrize("n,m,n_seeds,max_iter,walks", [
    (1, 1, 1, 10, True),            # a single pixel on either side
    (33, 31, 33, 10, True),         # one pixel past a tile; 33 seeds: a second, nearly empty query block
    (500, 1537, 65, 3, True),       # 49 tiles over the chunks, 3 blocks
    (2048, 512, 64, 2, True),       # image 1 the larger one
    (512, 512, 256, 10, True),
    (3072, 3071, 48, 0, False),     # no iteration allowed: the launch sequence
])
def test_small_pairs_walk_in_one_workgroup(compute, kw, d, n, m, n_seeds, max_iter, walks):
    maps = [exact_maps(n + m + k, n, m, d) for k in range(3)]
    rng = np.random.default_rng(n_seeds)
    seeds = rng.integers(0, n, size=(3, n_seeds)).astype(np.int32)
    got, walked = traced([x[0] for x in maps], [x[1] for x in maps], seeds, max_iter, compute, **kw)
    price = 5 if compute == "f32" or kw else 1
    products = -(-n_seeds // 32) * -(-max(n, m) // 32)
    assert walked == (walks and products * price <= 100 * max_iter)
    for p in range(3):
        check_reciprocal_exact(got, p, oracle.reciprocal(*maps[p], seeds[p], max_iter))


@pytest.mark.parametrize("n_seeds,walks", [(1000, True), (1023, True), (1024, True), (1025, False)])
def test_both_sides_of_the_line_agree(n_seeds, walks):
    a, b = exact_maps(41, 992, 1000, 24)      # 32 tiles: up to 31 blocks of seeds stay within the rule at ten iterations
    b = np.concatenate([b[:990], a[:10]])
    a, b = a[:960], b[:960]                   # 30 tiles: 32 blocks (1024 seeds) walk, 33 do not
    seeds = np.random.default_rng(3).integers(0, 960, size=(1, n_seeds)).astype(np.int32)
    got, walked = traced([a], [b], seeds, 10, "f16")
    assert walked == walks
    check_reciprocal_exact(got, 0, oracle.reciprocal(a, b, seeds[0], 10))
