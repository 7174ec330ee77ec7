"""fnn_reciprocal captured into a HIP graph (the library launches kernels only and clears its buffers with
kernels, so a call can be recorded once and replayed): every replay, with eager calls and new inputs in
between, must give what the eager call gives on the same inputs."""
import numpy as np
import pytest
import torch

import paper_2503_10017_amd as fnn
import synth_inputs as synth
from gpu_helpers import dev, unit_maps

pytestmark = pytest.mark.gpu

KEYS = ("seed_i", "seed_j", "seed_iter", "pairs", "n_pairs")


@pytest.mark.parametrize("width,height,stride,static", [(160, 120, 4, False), (256, 192, 4, False), (160, 120, 4, True)])
def test_graph_replays_match_eager_calls(width, height, stride, static):
    pairs = [synth.warped_pair(900 + i, width, height, 24)[:2] for i in range(3)]
    seeds = dev(synth.grid_seeds(width, height, stride))[None]
    n = width * height
    d1 = torch.empty((n, 24), dtype=torch.float32, device="cuda:0")
    d2 = torch.empty((n, 24), dtype=torch.float32, device="cuda:0")
    ws = torch.empty(fnn.fnn_workspace_bytes(1, n, n, 24, seeds.shape[1], "f16"), dtype=torch.uint8, device="cuda:0")

    def call(out):
        if static:
            return fnn.fnn_reciprocal_static(d1, d2, seeds, out, max_iter=10, compute="f16")
        return fnn.fnn_reciprocal(d1, d2, seeds, max_iter=10, compute="f16", out=out, workspace=ws)

    d1.copy_(dev(pairs[0][0]))
    d2.copy_(dev(pairs[0][1]))
    out = fnn.fnn_reciprocal(d1, d2, seeds, max_iter=10, compute="f16", workspace=ws)   # eager first: fills the launch caches
    call(out)
    torch.cuda.synchronize()

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out)
    for a, b in pairs + pairs[:1]:
        d1.copy_(dev(a))
        d2.copy_(dev(b))
        want = fnn.fnn_reciprocal(d1, d2, seeds, max_iter=10, compute="f16")     # eager, its own buffers
        torch.cuda.synchronize()
        for k in KEYS:
            out[k].fill_(-3)
        graph.replay()
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.equal(out[k], want[k]), k
        assert int(want["n_pairs"][0]) > 0


def test_dense_graph_replays_match_eager_calls():
    """The same for fnn_mutual_dense, at a size whose interior workgroups take the staged sweep (direct
    global->LDS loads) and whose edge workgroups take the unstaged one."""
    n, m = 9000, 5000
    maps = [unit_maps(700 + i, n, m, 24) for i in range(3)]
    d1 = torch.empty((n, 24), dtype=torch.float32, device="cuda:0")
    d2 = torch.empty((m, 24), dtype=torch.float32, device="cuda:0")
    ws = torch.empty(fnn.fnn_workspace_bytes(1, n, m, 24, 0, "f16"), dtype=torch.uint8, device="cuda:0")
    d1.copy_(dev(maps[0][0]))
    d2.copy_(dev(maps[0][1]))
    out = fnn.fnn_mutual_dense(d1, d2, "f16", workspace=ws)
    fnn.fnn_mutual_dense(d1, d2, "f16", out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fnn.fnn_mutual_dense(d1, d2, "f16", out=out, workspace=ws)
    for a, b in maps + maps[:1]:
        d1.copy_(dev(a))
        d2.copy_(dev(b))
        want = fnn.fnn_mutual_dense(d1, d2, "f16")
        torch.cuda.synchronize()
        for k in out:
            out[k].fill_(-3)
        graph.replay()
        torch.cuda.synchronize()
        for k in out:
            assert torch.equal(out[k], want[k]), k
        assert int(want["n_pairs"][0]) > 0


@pytest.mark.parametrize("op", ["nearest", "reciprocal", "dense"])
def test_graph_replays_of_calls_in_two_steps_match_eager_calls(op):
    """Calls that score in 8 bits first, with maps of other contrast in every replay: what decides between the ways on the device is found out
    afresh each time, on a workspace that the calls before have used."""
    n, m, batch = 66000, 70001, 4 if op == "dense" else 16
    gen = torch.Generator(device="cuda:0").manual_seed(17)

    def maps(alike):
        a = torch.nn.functional.normalize(torch.randn((batch, n, 24), generator=gen, device="cuda:0"), dim=2)
        if alike:
            a[::2] = a[::2, :1]
        b = torch.nn.functional.normalize(a[:, torch.randint(0, n, (m,), generator=gen, device="cuda:0")]
                                          + (0.0 if alike else 0.2) * torch.randn((batch, m, 24), generator=gen, device="cuda:0"), dim=2)
        return a, b

    seeds = torch.randint(0, n, (batch, 4000), generator=gen, device="cuda:0", dtype=torch.int32)
    d1, d2 = maps(False)
    compute = "f32" if op == "dense" else "f16"
    ws = torch.empty(fnn.fnn_workspace_bytes(batch, n, m, 24, 0 if op == "dense" else 4000, compute), dtype=torch.uint8, device="cuda:0")

    def call(out=None, workspace=ws):
        if op == "dense":
            return fnn.fnn_mutual_dense(d1, d2, compute, out=out, workspace=workspace)
        if op == "reciprocal":
            return fnn.fnn_reciprocal(d1, d2, seeds, max_iter=5, compute=compute, out=out, workspace=workspace)
        idx, score = fnn.fnn_nearest(d1, d2, q_idx=seeds, compute=compute, out_idx=out and out["idx"], out_score=out and out["score"], workspace=workspace)
        return {"idx": idx, "score": score}

    out = call()
    fnn.fnn_trace_begin(256)
    call(out)
    torch.cuda.synchronize()
    assert "refine_kernel" in [name for name, _ in fnn.fnn_trace_end(256)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out)
    for alike in (False, True, False, True, True):
        a, b = maps(alike)
        d1.copy_(a)
        d2.copy_(b)
        want = call(workspace=None)     # eager, its own buffers
        torch.cuda.synchronize()
        for k in out:
            out[k].fill_(-3)
        graph.replay()
        torch.cuda.synchronize()
        for k in out:
            assert torch.equal(out[k], want[k]), (alike, k)
