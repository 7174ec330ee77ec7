"""The late iterations of a walk are one launch whose workgroups meet at barriers of their own.  The same call with a
workspace that ends where that launch's control words would begin has every iteration in launches: both must give the same bits."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2503_10017_amd as fnn
from gpu_helpers import check_reciprocal_exact, dev, exact_maps, host
from test_gpu_coarse import one_step_bytes
import oracle

pytestmark = pytest.mark.gpu


def wandering_maps(seed, batch, n, m, d):
    """Two unrelated fields that vary slowly along the pixels: seeds climb from neighbour to neighbour for several iterations."""
    gen = torch.Generator().manual_seed(seed)

    def field(pixels):
        knots = torch.randn((batch, d, pixels // 24 + 2), generator=gen)
        x = torch.nn.functional.interpolate(knots, size=pixels, mode="linear", align_corners=True)
        return torch.nn.functional.normalize(x, dim=1).permute(0, 2, 1).contiguous()

    return field(n).cuda(), field(m).cuda()


def run(a, b, seeds, max_iter, compute, tail, full=None, **kw):
    (batch, n, d), m = a.shape, b.shape[1]
    ns = seeds.shape[1]
    whole = fnn.fnn_workspace_bytes_opts(batch, n, m, d, ns, compute, max_iter, **kw)
    ws = torch.full((whole if full or tail else one_step_bytes("reciprocal", batch, n, m, d, ns, compute, **kw),), 0xA5, dtype=torch.uint8, device="cuda:0")
    fnn.fnn_trace_begin(256)
    try:
        out = fnn.fnn_reciprocal(a, b, seeds, max_iter, compute, workspace=ws, **kw)
        torch.cuda.synchronize()
    finally:
        names = [name for name, _ in fnn.fnn_trace_end(256)]
    assert ("recip_tail_kernel" in names) == tail
    return {k: host(v) for k, v in out.items()}, names


@pytest.mark.parametrize("batch,n,m,n_seeds,compute,d,max_iter,option", [
    (1, 9001, 9333, 256, "f16", 24, 10, None),    # a walk of few seeds from the first search on; a partial tile on either side
    (1, 9001, 20011, 257, "f16", 24, 10, None),   # from the second iteration on
    (1, 9001, 9333, 512, "bf16", 24, 4, None),    # the most that a workgroup keeps; seeds still moving at the end
    (1, 9001, 9333, 513, "f16", 24, 10, None),    # one more: from the third on
    (3, 16400, 12345, 5000, "f16", 24, 10, None),  # many seeds, then few
    (2, 9001, 9333, 8192, "f16", 24, 6, None),
    (1, 30000, 20011, 4000, "f16", 24, 10, None),  # 256 workgroups while many seeds move, 78 for few (above, 32: the least)
    (40, 2100, 1999, 700, "f16", 24, 10, None),   # six workgroups per pair
    (64, 1000, 777, 300, "f16", 24, 7, None),     # four
    (1, 9001, 9333, 600, "f16", 16, 10, None),
    (1, 9001, 9333, 600, "bf16", 32, 10, None),
    (1, 9001, 9333, 600, "f32", 5, 10, None),
    (1, 9001, 9333, 600, "f32", 16, 10, None),
    (2, 9001, 9333, 600, "f32", 24, 10, None),
    (1, 9001, 9333, 200, "f32", 30, 10, None),
    (1, 9001, 9333, 600, "f16", 24, 10, "l2"),
    (1, 9001, 9333, 600, "f16", 16, 10, "split"),   # rows of 48 channels
    (1, 9001, 9333, 600, "f16", 20, 10, "split"),   # 64
    (2, 9001, 9333, 600, "f16", 24, 10, "split"),   # 80
    (1, 9001, 9333, 600, "f16", 32, 10, "split"),   # 96
])
def test_one_launch_and_many_give_the_same(batch, n, m, n_seeds, compute, d, max_iter, option):
    a, b = wandering_maps(n_seeds + d, batch, n, m, d)
    gen = torch.Generator().manual_seed(d)
    seeds = torch.randint(0, n, (batch, n_seeds), generator=gen, dtype=torch.int32).cuda()
    kw = {option: True} if option else {}
    one, _ = run(a, b, seeds, max_iter, compute, True, **kw)
    many, names = run(a, b, seeds, max_iter, compute, False, **kw)
    assert names.count("resolve_step_kernel") == max_iter
    for k in many:
        assert np.array_equal(one[k], many[k]), (k, int(np.sum(one[k] != many[k])))
    late = (many["seed_iter"] >= 3) | (many["seed_iter"] < 0)
    assert late.any()  # the maps are of the kind that this is about


@pytest.mark.parametrize("batch,n_seeds,max_iter,launched", [
    (1, 256, 10, 0),
    (1, 257, 10, 1),
    (1, 512, 10, 1),
    (1, 513, 10, 2),
    (48, 3072, 10, 2),
    (48, 3073, 10, 3),
    (48, 3073, 5, 3),     # two iterations are left
    (48, 3073, 4, None),  # one: four launches are as good
    (1, 513, 4, 2),
    (1, 513, 3, None),
])
def test_the_iteration_that_the_launch_begins_with(batch, n_seeds, max_iter, launched):
    n = 9001 if batch == 1 else 2100
    a, b = wandering_maps(n_seeds, batch, n, n - 101, 24)
    seeds = torch.randint(0, n, (batch, n_seeds), generator=torch.Generator().manual_seed(batch), dtype=torch.int32).cuda()
    one, names = run(a, b, seeds, max_iter, "f16", launched is not None, full=True)
    assert names.count("resolve_step_kernel") == (max_iter if launched is None else launched)
    many, _ = run(a, b, seeds, max_iter, "f16", False)
    for k in many:
        assert np.array_equal(one[k], many[k]), (k, int(np.sum(one[k] != many[k])))


@pytest.mark.parametrize("n_seeds", [1, 32, 33, 64, 65, 96, 97, 129, 225])
@pytest.mark.parametrize("compute,option,scale", [("f16", None, 1.0), ("f16", "split", 1.0), ("f32", None, 1e-12), ("f16", "l2", 1.0)])
def test_blocks_of_queries_dealt_to_the_waves(n_seeds, compute, option, scale):
    """One, two, three (by ones where rows are narrow or products in fp32, by twos where rows are wide) and more blocks of queries (of fp32, odd numbers
    by ones), whole ones and one more query; scores of every sign and size start from what the search before found."""
    a, b = (x * scale for x in wandering_maps(n_seeds, 2, 9001, 9333, 24))
    seeds = torch.randint(0, 9001, (2, n_seeds), generator=torch.Generator().manual_seed(n_seeds), dtype=torch.int32).cuda()
    kw = {option: True} if option else {}
    one, names = run(a, b, seeds, 10, compute, True, **kw)
    assert "search_kernel" not in names
    many, _ = run(a, b, seeds, 10, compute, False, **kw)
    for k in many:
        assert np.array_equal(one[k], many[k]), (k, int(np.sum(one[k] != many[k])))


@pytest.mark.parametrize("n_seeds", [300, 1100])
def test_ties_and_rows_that_are_not_finite(n_seeds):
    a, b = exact_maps(31, 9001, 9333, 24)
    seeds = np.random.default_rng(n_seeds).integers(0, 9001, size=(1, n_seeds)).astype(np.int32)
    got, _ = run(dev(a)[None], dev(b)[None], dev(seeds), 10, "f16", True)
    check_reciprocal_exact(got, 0, oracle.reciprocal(a, b, seeds[0], 10))
    x, y = wandering_maps(5, 1, 9001, 9333, 24)
    x[0, ::7] = float("nan")
    y[0, 3::11] = float("inf")
    one, _ = run(x, y, dev(seeds), 10, "f16", True)
    many, _ = run(x, y, dev(seeds), 10, "f16", False)
    for k in many:
        assert np.array_equal(one[k], many[k]), k


@pytest.mark.parametrize("not_numbers", [0, 5, 32])
@pytest.mark.parametrize("m,n_seeds,compute,d", [(9333, 256, "f16", 24), (9344, 300, "bf16", 24), (9333, 300, "f32", 32), (9344, 60, "f16", 16)])
def test_scores_of_minus_infinity(m, n_seeds, compute, d, not_numbers):
    """Every score is minus infinity, or, of some rows or all of the last tile, not a number: which candidate is named does not hang on the route."""
    x, y = wandering_maps(8, 1, 9001, m, d)
    x[..., 0] = x[..., 0].abs() + 0.125
    y[..., 0] = -float("inf")
    first = (m - 1) // 32 * 32
    y[0, first:first + not_numbers] = float("nan")
    seeds = torch.randint(0, 9001, (1, n_seeds), generator=torch.Generator().manual_seed(d), dtype=torch.int32).cuda()
    one, _ = run(x, y, seeds, 10, compute, True)
    many, _ = run(x, y, seeds, 10, compute, False)
    for k in many:
        assert np.array_equal(one[k], many[k]), k
    assert (many["seed_j"] == min(first + not_numbers, m - 1)).all()


def test_calls_that_share_the_device():
    """Workgroups wait for one another only while they run, so launches of several streams may have the chip in any shares."""
    calls = []
    for i in range(4):
        a, b = wandering_maps(90 + i, 1 + i, 30000, 20011, 24)
        seeds = torch.randint(0, 30000, (1 + i, 400 + 300 * i), generator=torch.Generator().manual_seed(i), dtype=torch.int32).cuda()
        calls.append((a, b, seeds, torch.cuda.Stream()))
    want = [fnn.fnn_reciprocal(a, b, seeds, 10, "f16") for a, b, seeds, _ in calls]
    torch.cuda.synchronize()
    for _ in range(3):
        got = []
        for a, b, seeds, stream in calls:
            with torch.cuda.stream(stream):
                got.append(fnn.fnn_reciprocal(a, b, seeds, 10, "f16"))
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            for k in w:
                assert torch.equal(g[k], w[k]), k


def hip():
    """The HIP runtime that this process runs on."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return ctypes.CDLL(path)


@pytest.mark.parametrize("batch,n,m,n_seeds,option,first", [
    (2, 9001, 9333, 700, None, "prep"),
    (1, 9001, 9333, 600, "l2", "prep"),
    (16, 66000, 70001, 4000, None, "quantise_kernel"),
    (4, 66000, 70001, 4000, "split", "quantise_kernel"),
])
def test_seeds_that_the_launch_gives_up_are_no_matches(batch, n, m, n_seeds, option, first):
    """A call without its late iterations (taken out of the captured call on the host, as if every workgroup had left) has no match of
    a seed that they would have settled, whatever the caller's arrays held; with them back in, it is the call that it was."""
    a, b = wandering_maps(n_seeds, batch, n, m, 24)
    seeds = torch.randint(0, n, (batch, n_seeds), generator=torch.Generator().manual_seed(1), dtype=torch.int32).cuda()
    kw = {option: True} if option else {}
    ws = torch.empty(fnn.fnn_workspace_bytes_opts(batch, n, m, 24, n_seeds, "f16", 10, **kw), dtype=torch.uint8, device="cuda:0")
    fnn.fnn_trace_begin(64)
    out = fnn.fnn_reciprocal(a, b, seeds, 10, "f16", workspace=ws, **kw)
    torch.cuda.synchronize()
    names = [name for name, _ in fnn.fnn_trace_end(64)]
    assert names[0].startswith(first)
    want = {k: host(v) for k, v in out.items()}
    tail_from = names.count("resolve_step_kernel")

    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fnn.fnn_reciprocal(a, b, seeds, 10, "f16", out=out, workspace=ws, **kw)
    lib, raw, count = hip(), ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0 and count.value == len(names)
    nodes, run_it = (ctypes.c_void_p * len(names))(), ctypes.c_void_p()
    assert lib.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    assert lib.hipGraphInstantiate(ctypes.byref(run_it), raw, None, None, ctypes.c_size_t(0)) == 0
    tail = ctypes.c_void_p(nodes[names.index("recip_tail_kernel")])
    for enabled in (0, 1):
        for k, x in (("seed_i", 5), ("seed_j", 7), ("seed_iter", 3), ("pairs", -3), ("n_pairs", -3)):
            out[k].fill_(x)
        assert lib.hipGraphNodeSetEnabled(run_it, tail, ctypes.c_uint(enabled)) == 0
        torch.cuda.synchronize()
        assert lib.hipGraphLaunch(run_it, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        got = {k: host(v) for k, v in out.items()}
        settled = (want["seed_iter"] >= 0) & (want["seed_iter"] < (10 if enabled else tail_from))
        assert np.array_equal(got["seed_iter"], np.where(settled, want["seed_iter"], -1))
        for p in range(batch):
            done = settled[p]
            for k in ("seed_i", "seed_j"):
                assert np.array_equal(got[k][p][done], want[k][p][done]), k
            pairs = np.unique(np.stack([want["seed_i"][p][done], want["seed_j"][p][done]], axis=1), axis=0)
            assert np.array_equal(got["pairs"][p, :int(got["n_pairs"][p])], pairs)
        if enabled:
            for k in want:
                assert np.array_equal(got[k], want[k]), k
        else:
            assert not settled.all()
    assert lib.hipGraphExecDestroy(run_it) == 0
