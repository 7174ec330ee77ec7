"""Large searches score everything in 8 bits first and multiply again, in the call's own format, only where a bound
says that the best candidate may be.  The same call with a workspace that ends where the 8-bit maps would begin runs in
one step: both must give the same bits, whatever the maps hold, and the trace says which way a call took."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
from gpu_helpers import check_nearest_against, check_reciprocal_exact, dev, exact_maps, host, unit_maps, GAP_ROUNDED, ROUNDERS, SCORE_TOL_ROUNDED

pytestmark = pytest.mark.gpu

ELEMENT = {"f32": 4, "f16": 2, "bf16": 2}


def up(x, to):
    return -(-x // to) * to


def channels(d, compute, l2=False, split=False):
    d = 3 * d if split else d + (0 if not l2 else 2 if compute == "f32" else 4)
    if compute == "f32":
        return up(d, 8)
    return 16 if d <= 16 else 24 if d <= 24 else up(d, 16)


def enough_pairs(nq, n, m, compute, d, **kw):
    """Pairs that make a call worth two steps, by the library's own estimate of both (nanoseconds)."""
    dp = channels(d, compute, kw.get("l2", False), kw.get("split", False))
    row, block = dp * ELEMENT[compute], 18.75 * dp if compute == "f32" else 46.0 if dp <= 32 else 1.64 * dp

    def gain(pixels):
        cells = pixels / 1024
        again = min(cells, 32.0 + 0.26 * (8.0 / d) ** 4 * cells if kw.get("l2") else 5.0 + 0.26 * (6.0 / d) ** 4 * cells)
        return -(-nq // 32) * -(-pixels // 32) / 1024.0 * (block * (1.0 - 1.5 * again / cells) - 28.0) - pixels * row / 4500.0

    maps = (n + m) * (row + 36) / 4500.0
    for batch in range(1, 65):
        if batch * gain(m) - 5000.0 - 4000.0 - batch * maps > 3000.0 and batch * (gain(m) + gain(n) - maps) - 14000.0 > 3000.0:
            return batch
    raise AssertionError("no batch is worth it")


def one_step_bytes(op, batch, n, m, d, nq, compute, **kw):
    """The workspace of a search in one step: prepared maps and keys, for the iteration its state too."""
    row = channels(d, compute, kw.get("l2", False), kw.get("split", False)) * ELEMENT[compute]
    maps = up(batch * up(n, 32) * row, 256) + up(batch * up(m, 32) * row, 256)
    if op == "nearest":
        return maps + up(batch * nq * 8, 256)
    words = up(batch * up(n, 32) // 32 * 4, 256)
    return maps + 2 * up(batch * nq * 8, 256) + 2 * words + 4 * up(batch * nq * 4, 256) + up(batch * 4, 256)


def run(op, a, b, queries, compute, two_steps, max_iter=6, **kw):
    batch, n, d = a.shape
    m = b.shape[1]
    nq = n if queries is None else queries.shape[1]
    small = one_step_bytes(op, batch, n, m, d, nq, compute, **kw)
    full = fnn.fnn_workspace_bytes_opts(batch, n, m, d, nq, compute, max_iter, **{k: v for k, v in kw.items()})
    assert full > small
    ws = torch.full((full if two_steps else small,), 0xA5, dtype=torch.uint8, device="cuda:0")
    fnn.fnn_trace_begin(128)
    try:
        if op == "nearest":
            idx, score = fnn.fnn_nearest(a, b, q_idx=queries, compute=compute, workspace=ws, **kw)
            out = {"idx": idx, "score": score}
        else:
            out = fnn.fnn_reciprocal(a, b, queries, max_iter, compute, workspace=ws, **kw)
        torch.cuda.synchronize()
    finally:
        names = [name for name, _ in fnn.fnn_trace_end(128)]
    assert ("coarse_kernel" in names) == two_steps and ("refine_kernel" in names) == two_steps
    return {k: host(v) for k, v in out.items()}


def same(op, a, b, queries, compute, **kw):
    two, one = (run(op, a, b, queries, compute, x, **kw) for x in (True, False))
    for k in one:
        assert np.array_equal(two[k], one[k]), (k, int(np.sum(two[k] != one[k])))
    return two


@pytest.mark.parametrize("n,m,nq,compute,stored,d,kw", [
    (65536, 65536, 8192, "f16", "f32", 24, {}),                      # whole segments, raw rows
    (70011, 65537, 8193, "bf16", "f32", 24, {}),                     # one candidate in the last segment
    (66000, 70001, 5001, "f16", "f32", 21, {}),                      # channels padded: prepared first
    (66000, 68001, 9000, "bf16", "f16", 30, {}),                     # 32-channel rows
    (65551, 70017, 7000, "f16", "f16", 24, {}),                      # rows of the caller, not whole tiles
    (65568, 70016, 7000, "f16", "f16", 24, {}),                      # ... and where they are
    (33000, 36001, 1000, "f32", "f32", 24, {}),
    (33000, 36001, 1500, "f32", "f32", 8, {}),
    (33000, 35001, 700, "f32", "f32", 31, {}),
    (132000, 131100, 600, "f32", "bf16", 13, {"l2": True}),
    (66000, 70000, 3000, "f16", "f32", 24, {"split": True}),
    (66000, 70000, 2600, "f16", "f32", 13, {"split": True}),
    (130000, 140000, 9000, "f16", "f32", 8, {"split": True}),
    (130000, 140000, 9000, "f16", "f32", 10, {"split": True}),
    (66000, 70000, 2800, "f16", "f32", 32, {"split": True, "normalize": True}),
    (67000, 68000, 7000, "bf16", "f32", 24, {"normalize": True}),
])
@pytest.mark.parametrize("op", ["nearest", "reciprocal"])
def test_same_bits_in_two_steps_as_in_one(op, n, m, nq, compute, stored, d, kw):
    batch = enough_pairs(nq, n, m, compute, d, **kw)
    gen = torch.Generator(device="cuda:0").manual_seed(n + m + nq)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda:0")

    a = torch.nn.functional.normalize(normal(batch, n, d), dim=2)
    b = torch.nn.functional.normalize(normal(batch, m, d), dim=2)
    b[:, :n // 2] = torch.nn.functional.normalize(a[:, :n // 2] + 0.3 * b[:, :n // 2], dim=2)  # half the pixels have a partner
    if kw:  # raw rows
        a, b = a * torch.exp(0.3 * normal(batch, n, 1)), b * torch.exp(0.3 * normal(batch, m, 1))
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[stored]
    a, b = a.to(kind), b.to(kind)
    q = torch.randint(0, n, (batch, nq), generator=gen, device="cuda:0", dtype=torch.int32)
    got = same(op, a, b, q, compute, **kw)
    if op == "nearest" and not kw and stored == "f32" and compute != "f32":
        ra, rb = ROUNDERS[compute](host(a[0])), ROUNDERS[compute](host(b[0]))
        ri, rbest, rsecond = oracle.nearest(ra[host(q[0])], rb)
        check_nearest_against(got["idx"][0], got["score"][0], ri, rbest, rsecond, GAP_ROUNDED, SCORE_TOL_ROUNDED)
    if op == "nearest" and n in (65536, 65568):
        same(op, a, b, None, compute, **kw)  # every pixel a query


@pytest.mark.parametrize("compute", ["f16", "f32"])
def test_exact_maps_with_ties_match_the_oracle(compute):
    a, b = exact_maps(5, 65600, 66001, 24)
    b[7000:7400] = b[100:500]      # equal candidates in different segments: the lowest index wins
    q = np.arange(0, 65600, 9).astype(np.int32)
    batch = enough_pairs(len(q), len(a), len(b), compute, 24)
    ta, tb, tq = dev(a)[None].repeat(batch, 1, 1), dev(b)[None].repeat(batch, 1, 1), dev(np.tile(q, (batch, 1)))
    got = same("nearest", ta, tb, tq, compute)
    ri, rbest, _ = oracle.nearest(a[q], b)
    assert np.array_equal(got["idx"][-1], ri) and np.array_equal(got["score"][-1], rbest)
    got = same("reciprocal", ta, tb, tq, compute)
    check_reciprocal_exact(got, batch - 1, oracle.reciprocal(a, b, q, 6))


def _special(kind, rng, n, m):
    a, b = unit_maps(int(rng.integers(1 << 30)), n, m, 24)
    if kind == "all equal":
        a[:], b[:] = a[0], a[0]
    elif kind == "negative":                       # every score is below zero: padding must not win
        a, b = np.abs(a) + 0.1, -np.abs(b) - 0.1
    elif kind == "outlier":                        # one row far longer than the rest flattens its segment's 8-bit rows
        a[3], b[5000] = 3000.0 * a[3], 3000.0 * b[5000]
    elif kind == "zero rows":
        a[::3], b[:2048], b[-5:] = 0.0, 0.0, 0.0
    elif kind == "tiny":                           # below what fp16 calls normal
        a, b = a * np.float32(1e-4), b * np.float32(3e-5)
    elif kind == "lengths":
        a = a * np.exp(2.0 * rng.standard_normal((n, 1))).astype(np.float32)
        b = b * np.exp(2.0 * rng.standard_normal((m, 1))).astype(np.float32)
    elif kind == "beyond bounds":                  # squares that leave fp32's comfortable range
        a[:1000] *= np.float32(1e-17)
        b[:1000] *= np.float32(1e-18)
        a[1000:1200] *= np.float32(1e16)
        b[3000:3200] *= np.float32(1e17)
    elif kind == "not finite":
        a[::7, 3], a[5::7, 4], b[1::5, 7], b[2::50] = np.nan, np.inf, np.nan, -np.inf
    return a, b


SPECIAL = ["all equal", "negative", "outlier", "zero rows", "tiny", "lengths", "beyond bounds", "not finite"]


@pytest.mark.parametrize("kind,compute", [(k, c) for k in SPECIAL for c in ("f16", "bf16", "f32") if (k, c) != ("beyond bounds", "f16")])
def test_maps_that_strain_the_bounds(kind, compute):
    rng = np.random.default_rng(11)
    n, m = 65601, 66011
    batch = enough_pairs(7500, n, m, compute, 24)
    maps = [_special(kind, rng, n, m) for _ in range(min(batch, 3))]
    maps = [maps[p % len(maps)] for p in range(batch)]
    a, b = (dev(np.stack([x[i] for x in maps])) for i in (0, 1))
    q = dev(rng.integers(0, n, size=(batch, 7500)).astype(np.int32))
    q[:, :8] = 3
    if kind == "not finite":  # unspecified results, but indices inside the maps
        got = run("nearest", a, b, q, compute, True)
        assert got["idx"].min() >= 0 and got["idx"].max() < m
        got = run("reciprocal", a, b, q, compute, True)
        assert min(got["seed_i"].min(), got["seed_j"].min()) >= 0 and got["seed_i"].max() < n and got["seed_j"].max() < m
        return
    same("nearest", a, b, q, compute)
    same("reciprocal", a, b, q, compute)


def test_queries_in_more_than_one_launch():
    """The table of bounds covers as many queries at a time as 256 MB hold."""
    n, m, batch = 16400, 200000, 64
    a, b = unit_maps(77, n, m, 24)
    ta, tb = [dev(a).half()] * batch, [dev(b).half()] * batch
    nq = n
    full = fnn.fnn_workspace_bytes(batch, n, m, 24, nq, "f16")
    fnn.fnn_trace_begin(32)
    ws = torch.full((full,), 0xA5, dtype=torch.uint8, device="cuda:0")
    idx, score = fnn.fnn_nearest(ta, tb, compute="f16", workspace=ws)
    torch.cuda.synchronize()
    names = [name for name, _ in fnn.fnn_trace_end(32)]
    assert names.count("coarse_kernel") == 1 + (nq - 1) // max(8192, (128 << 20) // (196 * batch) // 1024 * 1024) > 1
    small = one_step_bytes("nearest", batch, n, m, 24, nq, "f16")
    want, wscore = fnn.fnn_nearest(ta, tb, compute="f16", workspace=ws[:small])
    assert torch.equal(idx, want) and torch.equal(score, wscore)


def test_small_and_narrow_calls_keep_one_step():
    a, b = unit_maps(3, 66000, 66000, 24)
    ta, tb = dev(a), dev(b)
    q = dev(np.arange(8192, dtype=np.int32))[None].repeat(32, 1)

    def two_steps(x, y, queries, compute, **kw):
        fnn.fnn_trace_begin(16)
        fnn.fnn_nearest([x] * len(queries), [y] * len(queries), q_idx=queries, compute=compute, **kw)
        torch.cuda.synchronize()
        return "coarse_kernel" in [name for name, _ in fnn.fnn_trace_end(16)]

    assert two_steps(ta, tb, q, "f16") and not two_steps(ta, tb, q[:, :2047].contiguous(), "f16")
    assert two_steps(ta, tb, q[:, :2047].contiguous(), "f32") and two_steps(ta, tb, q[:, :2047].contiguous(), "f16", split=True)
    assert not two_steps(ta, tb, q[:, :255].contiguous(), "f32")
    assert not two_steps(ta, tb[:16383], q, "f32") and two_steps(ta, tb[:16384], q, "f32")
    assert not two_steps(ta, tb, q[:1], "f16")                             # one pair of this size
    assert not two_steps(ta[:, :16], tb[:, :16], q, "f16")                # one matrix instruction as it is
    assert not two_steps(ta, tb, q, "f16", l2=True)                       # bounds too wide on a map of this size
    count = torch.full((32,), 8192, dtype=torch.int32, device="cuda:0")
    assert not two_steps(ta, tb, q, "f16", nq_active=count)               # live counts on the device


@pytest.mark.parametrize("fewer,more", [(3008, 3072), (4550, 4608), (2900, 3060)])
def test_kernel_width_follows_the_split_not_the_count(fewer, more):
    """Query counts whose blocks are dealt alike (the same blocks for the busiest wave of as many quads) take the same kernel."""
    gen = torch.Generator(device="cuda:0").manual_seed(fewer)
    a, b = (torch.randn((16, 131072, 24), generator=gen, device="cuda:0").half() for _ in range(2))
    width = []
    for nq in (fewer, more):
        q = torch.randint(0, 131072, (16, nq), generator=gen, device="cuda:0", dtype=torch.int32)
        fnn.fnn_trace_begin(16)
        idx, score = fnn.fnn_nearest(a, b, q_idx=q, compute="f16")
        torch.cuda.synchronize()
        width.append([detail for name, _, detail in fnn.fnn_trace_end(16, details=True) if name == "coarse_kernel"])
        ws = torch.empty(one_step_bytes("nearest", 16, 131072, 131072, 24, nq, "f16"), dtype=torch.uint8, device="cuda:0")
        want, wscore = fnn.fnn_nearest(a, b, q_idx=q, compute="f16", workspace=ws)
        assert torch.equal(idx, want) and torch.equal(score, wscore)
    assert width[0] == width[1] and len(width[0]) == 1


def alike_maps(kind, n, gen):
    """Maps of which the 8-bit scores rule out little: one descriptor throughout, or descriptors of three dimensions."""
    if kind == "equal":
        return torch.nn.functional.normalize(torch.randn((1, 24), generator=gen, device="cuda:0"), dim=1).repeat(n, 1)
    few = torch.randn((n, 3), generator=gen, device="cuda:0") @ torch.randn((3, 24), generator=gen, device="cuda:0")
    return torch.nn.functional.normalize(few, dim=1)


@pytest.mark.parametrize("n,nq,batch,compute,d", [
    (131072, 3072, 16, "f16", 24),    # whole cells
    (100001, 4001, 10, "bf16", 24),   # half cells
    (66000, 7000, 15, "f16", 29),
    (196608, 196608, 1, "f16", 24),   # long chunks
    (34000, 17000, 8, "bf16", 24),    # few cells
])
@pytest.mark.parametrize("op", ["nearest", "reciprocal"])
def test_pairs_that_look_alike_beside_pairs_that_do_not(op, n, nq, batch, compute, d):
    """Every pair of a batch is searched its own way, with the same keys."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a = torch.nn.functional.normalize(torch.randn((batch, n, 24), generator=gen, device="cuda:0"), dim=2)
    b = a[:, torch.randperm(n, generator=gen, device="cuda:0")] + 0.1 * torch.randn((batch, n, 24), generator=gen, device="cuda:0")
    for p in range(0, batch, 3):
        a[p] = alike_maps("equal" if p % 2 else "rank 3", n, gen)
        b[p] = a[p, torch.randperm(n, generator=gen, device="cuda:0")]
    a, b = (x.repeat(1, 1, 2)[:, :, :d].contiguous() for x in (a, torch.nn.functional.normalize(b, dim=2)))
    q = torch.randint(0, n, (batch, nq), generator=gen, device="cuda:0", dtype=torch.int32)
    same(op, a, b, q, compute)


@pytest.mark.parametrize("batch,step", [(16, 64), (1, 1)])
@pytest.mark.parametrize("kind", ["equal", "rank 3"])
def test_maps_without_contrast_are_given_up(kind, batch, step):
    """Every cell of such maps is multiplied again, and scoring all of them in 8 bits first took 1.6 to 1.9 times the one step's time.  (The 8-bit maps and the
    scores up to the votes remain, and a second step that is not quite as fast as the one.)  16 pairs of seeds, and every pixel of one pair."""
    n = 196608
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    a = torch.stack([alike_maps(kind, n, gen) for _ in range(batch)])
    b = a[:, torch.randperm(n, generator=gen, device="cuda:0")].contiguous()
    q = torch.arange(0, n, step, device="cuda:0", dtype=torch.int32)[None].repeat(batch, 1)
    op = "nearest" if step == 1 else "reciprocal"
    ws = torch.empty(fnn.fnn_workspace_bytes(batch, n, n, 24, q.shape[1], "f16"), dtype=torch.uint8, device="cuda:0")
    small = ws[:one_step_bytes(op, batch, n, n, 24, q.shape[1], "f16")]

    def least(workspace):
        times = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            if op == "nearest":
                fnn.fnn_nearest(a, b, q_idx=q, compute="f16", workspace=workspace)
            else:
                fnn.fnn_reciprocal(a, b, q, 6, "f16", workspace=workspace)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    assert least(ws) < 1.45 * least(small)


@pytest.mark.parametrize("n,m,nq,compute,stored,d", [
    (400001, 390007, 6000, "f16", "f32", 24),
    (300000, 410000, 9001, "bf16", "f16", 28),     # the widest rows: 28 channels and four for the norms
])
@pytest.mark.parametrize("op", ["nearest", "reciprocal"])
def test_squared_distance_of_16_bit_rows_in_two_steps(op, n, m, nq, compute, stored, d):
    test_same_bits_in_two_steps_as_in_one(op, n, m, nq, compute, stored, d, {"l2": True})


@pytest.mark.parametrize("kw", [{}, {"split": True}])
@pytest.mark.parametrize("stride", [28, 40])
@pytest.mark.parametrize("op", ["nearest", "every", "reciprocal"])
def test_rows_apart_in_memory(op, stride, kw):
    """fp32 rows of 24 channels with others behind them are read where they are, 16 bytes at a time."""
    n, m, nq = 66003, 70001, 7000
    batch = enough_pairs(nq, n, m, "f16", 24, **kw)
    gen = torch.Generator(device="cuda:0").manual_seed(stride)
    a, b = (torch.randn((batch, rows, stride), generator=gen, device="cuda:0") for rows in (n, m))
    a, b = a[:, :, :24], b[:, :, :24]
    assert a.stride(1) == stride
    q = torch.randint(0, n, (batch, nq), generator=gen, device="cuda:0", dtype=torch.int32)
    packed = (a.contiguous(), b.contiguous())
    name, queries = ("nearest", None) if op == "every" else (op, q)
    got, want = same(name, a, b, queries, "f16", **kw), run(name, *packed, queries, "f16", True, **kw)
    for k in want:
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("kind,compute,kw", [(k, "f16", {"split": True}) for k in SPECIAL if k != "beyond bounds"] +
                         [(k, "f32", {"l2": True}) for k in SPECIAL] +
                         [(k, "bf16", {"l2": True}) for k in ("outlier", "zero rows", "tiny", "lengths", "not finite")])
def test_wide_rows_that_strain_the_bounds(kind, compute, kw):
    rng = np.random.default_rng(13)
    n, m = (65601, 66011) if compute != "bf16" else (262200, 270011)
    batch = enough_pairs(7500, n, m, compute, 24, **kw)
    maps = [_special(kind, rng, n, m) for _ in range(min(batch, 2))]
    maps = [maps[p % len(maps)] for p in range(batch)]
    a, b = (dev(np.stack([x[i] for x in maps])) for i in (0, 1))
    q = dev(rng.integers(0, n, size=(batch, 7500)).astype(np.int32))
    q[:, :8] = 3
    if kind == "not finite":
        got = run("reciprocal", a, b, q, compute, True, **kw)
        assert min(got["seed_i"].min(), got["seed_j"].min()) >= 0 and got["seed_i"].max() < n and got["seed_j"].max() < m
        return
    same("nearest", a, b, q, compute, **kw)
    same("reciprocal", a, b, q, compute, **kw)


@pytest.mark.parametrize("compute", ["f16", "bf16"])
@pytest.mark.parametrize("n,m,batch", [(65536, 66560, 8), (70001, 66561, 8)])
def test_rows_that_the_quantise_launch_normalises(n, m, batch, compute):
    """Aligned fp32 rows of 24 channels are divided by the launch that quantises them, all others by a launch of its own; the prepared
    maps in the workspace are the same bits as those of one step."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.randn((batch, rows, 24), generator=gen, device="cuda:0") * torch.exp(torch.randn((batch, rows, 1), generator=gen, device="cuda:0"))
            for rows in (n, m))
    a[0, 7] = b[1, m - 1] = 0
    a[1, n - 1] = 1e-30
    seeds = torch.randint(0, n, (batch, 6000), generator=torch.Generator().manual_seed(1), dtype=torch.int32).cuda()
    maps = 48 * batch * (up(n, 32) + up(m, 32))
    kept = []
    for size in (fnn.fnn_workspace_bytes_opts(batch, n, m, 24, 6000, compute, 6, normalize=True), one_step_bytes("reciprocal", batch, n, m, 24, 6000, compute)):
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda:0")
        fnn.fnn_trace_begin(64)
        out = fnn.fnn_reciprocal(a, b, seeds, 6, compute, workspace=ws, normalize=True)
        torch.cuda.synchronize()
        names = [name for name, _ in fnn.fnn_trace_end(64)]
        kept.append((names[0], ws[:maps].clone(), {k: host(v) for k, v in out.items()}))
    assert [k[0] for k in kept] == ["quantise_kernel", "prep_kernel"]
    assert torch.equal(kept[0][1], kept[1][1])
    for k in kept[0][2]:
        assert np.array_equal(kept[0][2][k], kept[1][2][k]), k
