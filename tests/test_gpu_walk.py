"""fnn_reciprocal on small pairs: the whole iteration runs in one workgroup per pair (search, reciprocity test,
compaction and the sorted match set behind workgroup barriers).  Sizes at the edges of its blocks, tiles and
chunks and on both sides of the line where the launch sequence takes over; exactly representable maps, so
everything must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
import synth_inputs as synth
from gpu_helpers import GAP_ROUNDED, check_reciprocal_exact, check_reciprocal_pinned, dev, exact_maps, host

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


@pytest.mark.parametrize("walks,w,h,sub", [(True, 40, 28, 4), (False, 48, 40, 4)])     # 3 and 4 blocks of seeds
@pytest.mark.parametrize("compute", ["f16", "bf16"])
def test_squared_distance_on_both_routes(walks, w, h, sub, compute):
    a, b = synth.exact_pair(77, w, h, 24)
    seeds = synth.grid_seeds(w, h, sub)
    got, walked = traced([a], [b], seeds[None], 10, compute, l2=True)
    assert walked == walks
    check_reciprocal_exact(got, 0, oracle.reciprocal(a, b, seeds, 10, metric="l2"))


@pytest.mark.parametrize("walks,n_seeds", [(True, 90), (False, 130)])
@pytest.mark.parametrize("compute,dtype,d", [("f16", torch.float16, 24), ("bf16", torch.bfloat16, 16), ("f16", torch.float16, 32)])
def test_maps_used_in_place_on_both_routes(walks, n_seeds, compute, dtype, d):
    """Whole 32-pixel tiles of packed rows in the compute format, stacked: no prepared copy, and no padding behind the last row."""
    maps = [exact_maps(60 + k, 1024, 992, d) for k in range(2)]
    seeds = np.random.default_rng(n_seeds).integers(0, 1024, size=(2, n_seeds)).astype(np.int32)
    stack = [dev(np.stack([m[side] for m in maps])).to(dtype) for side in range(2)]
    fnn.fnn_trace_begin(128)
    out = fnn.fnn_reciprocal(stack[0], stack[1], dev(seeds), max_iter=10, compute=compute)
    torch.cuda.synchronize()
    names = [name for name, _ in fnn.fnn_trace_end(128)]
    assert names[0] == ("recip_walk_kernel" if walks else "prep_kernel") and ("recip_walk_kernel" in names) == walks
    for p in range(2):
        check_reciprocal_exact({k: host(v) for k, v in out.items()}, p, oracle.reciprocal(*maps[p], seeds[p], 10))


def test_normalised_pair_on_both_routes():
    a, b, _ = synth.warped_pair(61, 40, 30, 24)
    rng = np.random.default_rng(5)
    a, b = (x * rng.uniform(0.1, 9.0, size=(x.shape[0], 1)).astype(np.float32) for x in (a, b))
    ra, rb = (oracle.round_fp16(oracle.normalize(x)) for x in (a, b))
    for seeds, walks in ((np.arange(0, 1200, 13, dtype=np.int32), True), (np.arange(0, 1200, 9, dtype=np.int32), False)):
        got, walked = traced([a], [b], seeds[None], 10, "f16", normalize=True)
        assert walked == walks
        check_reciprocal_pinned(got, 0, oracle.reciprocal(ra, rb, seeds, 10), ra, rb, GAP_ROUNDED)
