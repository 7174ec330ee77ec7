"""The dense mode on large maps: 8-bit scores with bounds first, then the second step of the searches in both directions.  With a
workspace that ends where the 8-bit maps would begin the same call forms every product in its own format: both must give the
same bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
from gpu_helpers import dev, exact_maps, host
from test_gpu_coarse import ELEMENT, SPECIAL, _special, channels, up

pytestmark = pytest.mark.gpu


def one_step_bytes(batch, n, m, d, compute, **kw):
    row = channels(d, compute, kw.get("l2", False), kw.get("split", False)) * ELEMENT[compute]
    n_pad, m_pad = up(n, 4096), up(m, 32)
    row_units, col_units = -(-m_pad // 128), n_pad // 128
    lists = up(n, 32) + 32 * row_units + m_pad + 32 * col_units
    units = 4 * batch * (row_units + col_units)
    sizes = [batch * n_pad * row, batch * m_pad * row, 8 * batch * (n + m), units, units, 4 * batch * lists, batch * lists // 8, 8 * batch,
             4 * batch * (-(-max(n, m) // 1024) + 1)]
    return sum(up(x, 256) for x in sizes)


def run(a, b, compute, two_steps, **kw):
    batch, n, d = a.shape
    m = b.shape[1]
    small = one_step_bytes(batch, n, m, d, compute, **kw)
    full = fnn.fnn_workspace_bytes_opts(batch, n, m, d, 0, compute, **kw)
    assert full > small + 1024
    ws = torch.full((full if two_steps else small,), 0xA5, dtype=torch.uint8, device="cuda:0")
    fnn.fnn_trace_begin(256)
    try:
        out = fnn.fnn_mutual_dense(a, b, compute, workspace=ws, **kw)
        torch.cuda.synchronize()
    finally:
        names = [name for name, _ in fnn.fnn_trace_end(256)]
    assert ("dense_select_kernel" in names) == two_steps
    return {k: host(v) for k, v in out.items()}, names


def same(a, b, compute, **kw):
    (two, names), (one, _) = (run(a, b, compute, x, **kw) for x in (True, False))
    for k in one:
        assert np.array_equal(two[k], one[k]), (k, int(np.sum(two[k] != one[k])))
    return two, names


@pytest.mark.parametrize("n,m,batch,compute,stored,d,kw", [
    (131072, 131072, 2, "f16", "f32", 24, {}),                  # whole segments, rows where they are
    (131073, 135169, 2, "bf16", "f32", 24, {}),                 # one pixel in the last segments
    (150000, 131071, 3, "f16", "f16", 21, {}),
    (131500, 141000, 4, "bf16", "f32", 29, {}),                 # 32-channel rows
    (65536, 40000, 1, "f32", "f32", 24, {}),
    (130001, 70000, 2, "f32", "bf16", 7, {}),
    (50000, 60001, 1, "f32", "f32", 32, {"normalize": True}),
    (400001, 390000, 1, "f32", "f32", 16, {"l2": True}),
    (66000, 65600, 1, "f16", "f32", 24, {"split": True}),
    (66000, 71000, 1, "f16", "f32", 11, {"split": True}),
    (300801, 310777, 1, "f16", "f32", 24, {"split": True}),     # segments of 4096 pixels that the quantise launch prepares, a wave's rows past the map
    (200000, 200001, 2, "f16", "f32", 9, {"split": True}),
    (90000, 404000, 1, "f16", "f32", 24, {"normalize": True}),  # wide cells
    (404123, 17000, 2, "f32", "f32", 24, {}),
])
def test_same_bits_in_two_steps_as_in_one(n, m, batch, compute, stored, d, kw):
    gen = torch.Generator(device="cuda:0").manual_seed(n + m)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda:0")

    a = torch.nn.functional.normalize(normal(batch, n, d), dim=2)
    b = torch.nn.functional.normalize(normal(batch, m, d), dim=2)
    k = min(n, m) // 2
    b[:, :k] = torch.nn.functional.normalize(a[:, :k] + 0.3 * b[:, :k], dim=2)  # half the pixels have a partner
    if kw:
        a, b = a * torch.exp(0.2 * normal(batch, n, 1)), b * torch.exp(0.2 * normal(batch, m, 1))
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[stored]
    same(a.to(kind), b.to(kind), compute, **kw)


@pytest.mark.parametrize("n,m,compute", [(300801, 30001, "f16"), (307201, 17000, "bf16")])
def test_raw_rows_normalised_where_they_are_read_twice(n, m, compute):
    """Segments of 4096 pixels: the quantise launch divides a row for its segment's scale and once more for the prepared map."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.nn.functional.normalize(torch.randn((1, rows, 24), generator=gen, device="cuda:0"), dim=2) for rows in (n, m))
    b[:, :m // 2] = torch.nn.functional.normalize(a[:, 7:7 + m // 2] + 0.3 * b[:, :m // 2], dim=2)
    for x in (a, b):
        x *= torch.exp(4.0 * torch.randn(x.shape[:2] + (1,), generator=gen, device="cuda:0"))
        x[:, 4095] = 0.0
        x[:, -1] = 0.0
    _, names = same(a, b, compute, normalize=True)
    assert "quantise_kernel" in names and not [name for name in names if name.startswith("prep")]


def test_ranges_of_segments_in_launches_of_their_own():
    """The table of bounds covers as many segments of image 1 as 128 MB hold."""
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    a = torch.nn.functional.normalize(torch.randn((5, 130000, 24), generator=gen, device="cuda:0"), dim=2)
    b = torch.nn.functional.normalize(a[:, torch.randperm(130000, generator=gen, device="cuda:0")] + 0.1 * torch.randn(a.shape, generator=gen, device="cuda:0"), dim=2)
    _, names = same(a, b, "bf16")
    assert names.count("dense_kernel") == 2    # 127 cells x 4096 x 2 bytes x 5 pairs: 25 of the 32 segments fit


def test_exact_maps_with_ties_match_the_oracle():
    a, b = exact_maps(8, 45000, 36000, 24)
    b[17000:17400] = b[100:500]
    a[20000:20100] = a[50:150]
    (got, _), ref = same(dev(a)[None], dev(b)[None], "f32"), oracle.mutual_dense(a, b)
    for k in ("nn12", "s12", "nn21", "s21"):
        assert np.array_equal(got[k][0], ref[k]), k
    assert np.array_equal(got["pairs"][0, :int(got["n_pairs"][0])], ref["pairs"])


@pytest.mark.parametrize("kind,compute", [(k, c) for k in SPECIAL for c in ("f16", "f32") if (k, c) != ("beyond bounds", "f16") and k != "not finite"])
def test_maps_that_strain_the_bounds(kind, compute):
    rng = np.random.default_rng(12)
    n, m, batch = (131100, 133000, 2) if compute == "f16" else (40001, 40100, 1)
    maps = [_special(kind, rng, n, m) for _ in range(batch)]
    a, b = (dev(np.stack([x[i] for x in maps])) for i in (0, 1))
    same(a, b, compute)


def _alike(kind, n, gen):
    """Maps of which the 8-bit scores rule out little: one descriptor throughout, or descriptors of three dimensions."""
    if kind == "equal":
        return torch.nn.functional.normalize(torch.randn((1, 24), generator=gen, device="cuda:0"), dim=1).repeat(n, 1)
    few = torch.randn((n, 3), generator=gen, device="cuda:0") @ torch.randn((3, 24), generator=gen, device="cuda:0")
    return torch.nn.functional.normalize(few, dim=1)


@pytest.mark.parametrize("n,m,compute,stored,d,kw", [
    (131072, 131072, "f16", "f32", 24, {}),
    (131073, 135169, "bf16", "f16", 24, {}),
    (131500, 141000, "bf16", "f32", 29, {}),
    (65537, 40000, "f32", "f32", 21, {}),
    (66000, 65600, "f16", "f32", 24, {"split": True}),
])
def test_pairs_that_look_alike_beside_pairs_that_do_not(n, m, compute, stored, d, kw):
    """Every pair of a batch goes its own way; the keys of both ways are resolved together."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a = torch.nn.functional.normalize(torch.randn((5, n, 24), generator=gen, device="cuda:0"), dim=2)
    b = torch.nn.functional.normalize(torch.randn((5, m, 24), generator=gen, device="cuda:0"), dim=2)
    for p, kind in ((0, "rank 3"), (2, "equal"), (4, "rank 3")):
        a[p] = _alike(kind, n, gen)
        b[p] = a[p, torch.randint(0, n, (m,), generator=gen, device="cuda:0")]
    a, b = (x.repeat(1, 1, 2)[:, :, :d].to({"f32": torch.float32, "f16": torch.float16}[stored]).contiguous() for x in (a, b))
    same(a, b, compute, **kw)


@pytest.mark.parametrize("kind", ["equal", "rank 3"])
def test_maps_without_contrast_take_no_longer_than_one_step(kind):
    """Every cell of such maps would be multiplied again: 2.2 times the one step's time.  (The sample, the 8-bit maps and the launches that
    leave the pair alone are 5 to 10 %.)"""
    n = 196608
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    a = _alike(kind, n, gen)
    b = a[torch.randperm(n, generator=gen, device="cuda:0")]
    ws = torch.empty(fnn.fnn_workspace_bytes(1, n, n, 24, 0, "f16"), dtype=torch.uint8, device="cuda:0")
    small = ws[:one_step_bytes(1, n, n, 24, "f16")]
    out = fnn.fnn_mutual_dense(a, b, "f16", workspace=ws)

    def least(workspace):
        return least_ms(lambda: fnn.fnn_mutual_dense(a, b, "f16", out=out, workspace=workspace))

    assert least(ws) < 1.4 * least(small)


def least_ms(call):
    times = []
    for _ in range(6):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        call()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end))
    return min(times)


@pytest.mark.parametrize("w,h,batch,feature,most", [(224, 168, 4, 32, 0.97), (192, 144, 4, 32, 0.97), (288, 216, 1, 128, 1.15)])
def test_lists_that_lie_together(w, h, batch, feature, most):
    """Neighbouring pixels need the same cells where a map's features are large, so some workgroups of the second step have long lists; shared out in short
    ranges they do not hold up a small call (0.89 and 0.87 of what one step takes; in ranges of 4096 queries 1.02 and 1.04; the last 1.04 to 1.12, with whole ranges in the
    candidates' second round 1.34)."""
    n, gen = w * h, torch.Generator(device="cuda:0").manual_seed(w)

    def field():
        coarse = torch.randn((batch, 24, h // feature + 2, w // feature + 2), generator=gen, device="cuda:0")
        x = torch.nn.functional.interpolate(coarse, size=(h, w), mode="bilinear", align_corners=True)
        return torch.nn.functional.normalize(x, dim=1).permute(0, 2, 3, 1).reshape(batch, n, 24).contiguous()

    a = field()
    b = torch.nn.functional.normalize(a.roll(w * 11 + 17, 1) + 0.1 * torch.randn(a.shape, generator=gen, device="cuda:0"), dim=2)
    same(a, b, "f16")
    ws = torch.empty(fnn.fnn_workspace_bytes(batch, n, n, 24, 0, "f16"), dtype=torch.uint8, device="cuda:0")
    small, out = ws[:one_step_bytes(batch, n, n, 24, "f16")], fnn.fnn_mutual_dense(a, b, "f16", workspace=ws)
    two, one = (least_ms(lambda: fnn.fnn_mutual_dense(a, b, "f16", out=out, workspace=x)) for x in (ws, small))
    assert two < most * one


def test_pairs_in_groups_that_share_their_tables():
    """The candidates' table covers as many pairs at a time as 512 MB hold: 38 pairs of 120000 pixels (14 MB each), so that 40 are two groups of 20.  A
    workspace that grew with batch x pixels x segments took 2.7 times as much for 64 pairs."""
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    n, m, batch = 118000, 120000, 40
    a = torch.nn.functional.normalize(torch.randn((batch, n, 24), generator=gen, device="cuda:0"), dim=2).half()
    b = torch.nn.functional.normalize(torch.randn((batch, m, 24), generator=gen, device="cuda:0"), dim=2).half()
    b[:, :n // 2] = a[:, :n // 2]
    for p in (1, 19, 20, 39):   # in either group, and next to the line between them
        a[p] = _alike("rank 3", n, gen).half()
    _, names = same(a, b, "f16")
    assert names.count("dense_alike_kernel") == 2

    def size(pairs):
        return fnn.fnn_workspace_bytes(pairs, n, m, 24, 0, "f16") - one_step_bytes(pairs, n, m, 24, "f16")

    per_pair = 36 * 2 * 122880 + 4096 * 24 * 2 * 30        # 8-bit maps and what little else every pair has
    assert size(64) - size(32) < 32 * per_pair + (64 << 20)


@pytest.mark.parametrize("n,m,compute,stored,d", [(400001, 390000, "f16", "f32", 24), (300000, 410000, "bf16", "f16", 28)])
def test_squared_distance_of_16_bit_rows_in_two_steps(n, m, compute, stored, d):
    test_same_bits_in_two_steps_as_in_one(n, m, 1, compute, stored, d, {"l2": True})


@pytest.mark.parametrize("kw", [{}, {"split": True}])
def test_rows_apart_in_memory(kw):
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    a, b = (torch.randn((2, rows, 28), generator=gen, device="cuda:0")[:, :, :24] for rows in (131100, 90001))
    got, _ = same(a, b, "f16", **kw)
    want, _ = run(a.contiguous(), b.contiguous(), "f16", True, **kw)
    for k in want:
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("kind,compute,kw", [(k, "f16", {"split": True}) for k in SPECIAL if k not in ("beyond bounds", "not finite")] +
                         [(k, "f32", {"l2": True}) for k in SPECIAL if k != "not finite"])
def test_wide_rows_that_strain_the_bounds(kind, compute, kw):
    rng = np.random.default_rng(14)
    n, m = (66001, 66100) if compute == "f16" else (200001, 210000)
    a, b = _special(kind, rng, n, m)
    same(dev(a)[None], dev(b)[None], compute, **kw)


@pytest.mark.parametrize("compute,kw", [("f16", {}), ("bf16", {}), ("f32", {}), ("f16", {"split": True})])
def test_indices_stay_inside_maps_that_are_not_finite(compute, kw):
    """Results are unspecified there, but every index lies in its map (or is -1) and every pair is a pair of pixels."""
    rng = np.random.default_rng(15)
    n, m = 131100, 133000
    a, b = _special("not finite", rng, n, m)
    got, _ = run(dev(a)[None], dev(b)[None], compute, True, **kw)
    for k, most in (("nn12", m), ("nn21", n)):
        assert got[k].min() >= -1 and got[k].max() < most
    count = int(got["n_pairs"][0])
    assert 0 <= count <= min(n, m)
    pairs = got["pairs"][0, :count]
    assert count == 0 or (pairs.min() >= 0 and pairs[:, 0].max() < n and pairs[:, 1].max() < m)


def traced(a, b, compute, **kw):
    fnn.fnn_mutual_dense(a, b, compute, **kw)
    torch.cuda.synchronize()
    fnn.fnn_trace_begin(256)
    try:
        fnn.fnn_mutual_dense(a, b, compute, **kw)
        torch.cuda.synchronize()
    finally:
        return fnn.fnn_trace_end(256, details=True)


def pass1_detail(a, b, compute, **kw):
    """Which 8-bit pass was launched: 2 keeps a maximum for every candidate, 3 one for three (or, pair by pair, for every candidate)."""
    return {detail for name, _, detail in traced(a, b, compute, **kw) if name == "dense_kernel"}


def ways(a, b, compute, **kw):
    """What the pairs of a call in two steps did there.  A launch without a pair of its own takes 4 us; the sweeps and lists of these sizes take 20 and more."""
    entries = traced(a, b, compute, **kw)
    took = {kind: [ms * 1e3 for name, ms, _ in entries if name == kind] for kind in ("dense_kernel", "dense_alike_kernel", "refine_kernel")}
    groups = {detail for name, _, detail in entries if name == "dense_kernel"} == {3}
    done = {"one step"} if max(took["dense_alike_kernel"]) > 15 else set()
    if max(took["dense_kernel"]) > 15:
        done.add("groups" if groups and took["refine_kernel"][-1] > 12 else "singles")
    return done


@pytest.mark.parametrize("n,m,batch,compute,d,kw,grouped", [
    (122881, 131073, 1, "f16", 24, {}, True),              # one pixel in the last cell of queries and in the last run of 1024 candidates
    (126976, 131071, 1, "bf16", 24, {}, True),             # the last group lacks a candidate
    (123904, 132064, 1, "f16", 24, {}, True),              # one tile in the last run
    (43008, 524288, 1, "f16", 24, {}, True),               # as few cells of queries as groups are taken for, wide cells of candidates
    (300001, 200100, 1, "bf16", 32, {}, True),             # cells of 2048 queries
    (131072, 131072, 1, "f16", 24, {"split": True}, True),
    (110000, 131072, 1, "f16", 24, {"split": True}, False),
    (131072, 70000, 1, "f32", 24, {}, False),
])
def test_maxima_of_three_candidates(n, m, batch, compute, d, kw, grouped):
    """A group's candidates have their partners in different cells, equal rows in different cells tie, and rows that are not finite are
    multiplied with everything."""
    gen = torch.Generator(device="cuda:0").manual_seed(n + 7 * m)
    a = torch.nn.functional.normalize(torch.randn((batch, n, d), generator=gen, device="cuda:0"), dim=2)
    b = torch.nn.functional.normalize(torch.randn((batch, m, d), generator=gen, device="cuda:0"), dim=2)
    at = torch.randperm(n, generator=gen, device="cuda:0")[:min(n, m) // 2]
    b[:, 1:2 * at.numel():2] = torch.nn.functional.normalize(a[:, at] + 0.3 * b[:, 1:2 * at.numel():2], dim=2)   # every second candidate
    a[:, n - 3000:n - 2000] = a[:, 1000:2000]                                    # the same row in two cells: the lower index wins
    b[:, m - 1] = a[:, 1500]
    got, _ = same(a, b, compute, **kw)
    assert pass1_detail(a, b, compute, **kw) == {3 if grouped else 2}
    assert (got["nn21"][:, m - 1] == 1500).all()
    assert ways(a, b, compute, **kw) == ({"groups"} if grouped else {"singles"})
    # a product of infinity is reached by no bound, and the lowest of two is the match (most of these maps, crowded in one orthant, are left to one
    # step; infinities in two steps: test_rows_without_bounds_among_rows_that_have_them)
    a, b = a.abs() + 0.01, b.abs() + 0.01  # no channel is 0: 0 times infinity is no number
    a[:, 5000] = a[:, n - 5] = float("inf")
    b[:, 77] = b[:, m - 40] = float("inf")
    got, _ = same(a, b, compute, **kw) if not kw else (None, None)
    if got:
        assert (got["nn21"] == 5000).sum() >= batch * (m - 2) and (got["nn12"] == 77).sum() >= batch * (n - 2)


@pytest.mark.parametrize("n,m,compute,d,kind,way", [
    (122881, 131073, "f16", 24, "infinite", "groups"),
    (300001, 200100, "bf16", 32, "infinite", "groups"),      # cells of 2048 queries
    (43008, 524288, "bf16", 24, "beyond bounds", "groups"),
    (126976, 131071, "bf16", 24, "beyond bounds", "groups"),
    (131072, 70000, "f32", 24, "beyond bounds", "singles"),
])
def test_rows_without_bounds_among_rows_that_have_them(n, m, compute, d, kind, way):
    """Two equal rows of either image have no bounds, in different cells, and win wherever a product with them is positive: the lower index is the match.  The rest
    keep the bounds that they have, so the pair stays in two steps."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.nn.functional.normalize(torch.randn((1, rows, d), generator=gen, device="cuda:0"), dim=2) for rows in (n, m))
    k = min(n, m) // 2
    b[:, :k] = torch.nn.functional.normalize(a[:, :k] + 0.3 * b[:, :k], dim=2)
    a[..., 0] += 0.002 * (a[..., 0] >= 0) - 0.001   # no row's channel 0 is 0, also in 16 bits: 0 times infinity is no number
    b[..., 0] += 0.002 * (b[..., 0] >= 0) - 0.001
    for x, at in ((a, (5000, n - 5)), (b, (77, m - 40))):
        row = x[0, at[0]].clone()
        if kind == "infinite":
            row[0] = float("inf")
        else:
            row *= 3e15 / row.abs().max()   # a square past the largest that the bounds hold for
        x[0, list(at)] = row
    assert ways(a, b, compute) == {way}
    got, _ = same(a, b, compute)
    for key, x, y, index, special in (("nn12", a, b[0, 77], 77, (5000, n - 5)), ("nn21", b, a[0, 5000], 5000, (77, m - 40))):
        x, y = (z.to({"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[compute]).double() for z in (x[0], y))
        positive = (x[:, 0] > 0) if kind == "infinite" else (x @ y > 1e12)   # far above any other product
        positive[list(special)] = False   # ... but theirs with one another
        assert positive.sum() > x.shape[0] // 3 and (got[key][0][positive.cpu().numpy()] == index).all(), key


@pytest.mark.parametrize("n,m,compute,d,kw", [
    (196608, 196608, "f16", 24, {}),
    (122881, 131073, "bf16", 24, {}),
    (43008, 524288, "f16", 24, {}),       # wide cells of candidates
    (300001, 200100, "bf16", 32, {}),     # cells of 2048 queries
    (131072, 131072, "f16", 24, {"split": True}),
])
def test_rows_whose_lengths_vary_keep_a_maximum_for_every_candidate(n, m, compute, d, kw):
    """A group's bound is that of its longest row, which reaches past the best of the others."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.nn.functional.normalize(torch.randn((1, rows, d), generator=gen, device="cuda:0"), dim=2) for rows in (n, m))
    k = min(n, m) // 2
    b[:, :k] = torch.nn.functional.normalize(a[:, :k] + 0.3 * b[:, :k], dim=2)
    assert ways(a, b, compute, **kw) == {"groups"}
    for x in (a, b):
        x *= torch.exp(0.4 * torch.randn(x.shape[:2] + (1,), generator=gen, device="cuda:0"))
    assert ways(a, b, compute, **kw) == {"singles"}
    same(a, b, compute, **kw)


@pytest.mark.parametrize("n,batch,compute", [(27648, 4, "f16"), (62208, 1, "bf16")])
def test_small_maps_whose_lengths_vary_take_two_steps(n, batch, compute):
    """What is paid for before the samples speak is a tenth of these calls, and no reason to leave them to one step (four of 27648 pixels: 392 us, in two 295)."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.nn.functional.normalize(torch.randn((batch, n, 24), generator=gen, device="cuda:0"), dim=2) for _ in range(2))
    b[:, :n // 2] = torch.nn.functional.normalize(a[:, :n // 2] + 0.3 * b[:, :n // 2], dim=2)
    for x in (a, b):
        x *= torch.exp(0.3 * torch.randn((batch, n, 1), generator=gen, device="cuda:0"))
    assert ways(a, b, compute) == {"singles"}
    same(a, b, compute)


@pytest.mark.parametrize("n,batch,few,want", [
    (27648, 4, (0, 2), {"one step"}),        # half of the call would take two steps
    (27648, 16, (3,), {"groups"}),
    (196608, 3, (1,), {"one step", "groups"}),   # large pairs go their own way where that gains much
])
def test_small_pairs_of_a_call_go_the_same_way(n, batch, few, want):
    """Launches that take a part of a call's small pairs leave most of the chip idle."""
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    a, b = (torch.nn.functional.normalize(torch.randn((batch, n, 24), generator=gen, device="cuda:0"), dim=2) for _ in range(2))
    b[:, :n // 2] = torch.nn.functional.normalize(a[:, :n // 2] + 0.3 * b[:, :n // 2], dim=2)
    for p in few:
        a[p] = _alike("rank 3", n, gen)
        b[p] = a[p, torch.randperm(n, generator=gen, device="cuda:0")]
    assert ways(a, b, "f16") == want
    same(a, b, "f16")


def test_pairs_whose_lengths_vary_beside_pairs_that_do_not():
    """Every way of a large pair, in one call."""
    n, gen = 196608, torch.Generator(device="cuda:0").manual_seed(4)
    a, b = (torch.nn.functional.normalize(torch.randn((3, n, 24), generator=gen, device="cuda:0"), dim=2) for _ in range(2))
    b[:, :n // 2] = torch.nn.functional.normalize(a[:, :n // 2] + 0.3 * b[:, :n // 2], dim=2)
    for x in (a, b):
        x[1] *= torch.exp(0.4 * torch.randn((n, 1), generator=gen, device="cuda:0"))
    a[2] = _alike("rank 3", n, gen)
    b[2] = a[2, torch.randperm(n, generator=gen, device="cuda:0")]
    assert ways(a, b, "bf16") == {"one step", "groups"}
    same(a, b, "bf16")


@pytest.mark.parametrize("n,m,batch,compute,d,kw,two_steps", [
    (27648, 27648, 4, "f16", 24, {}, True),      # maps that are not whole runs of 4096 queries
    (27648, 27648, 1, "f16", 24, {}, False),     # ... one pair of them
    (37632, 36864, 4, "bf16", 24, {}, True),     # a maximum for every candidate
    (49152, 49152, 4, "f16", 24, {}, True),      # whole
    (49152, 49152, 1, "f16", 24, {}, False),
    (27648, 27649, 8, "f16", 32, {}, True),
    (16384, 16384, 4, "f16", 24, {}, False),
])
def test_which_small_maps_take_two_steps(n, m, batch, compute, d, kw, two_steps):
    gen = torch.Generator(device="cuda:0").manual_seed(n + m)
    a = torch.nn.functional.normalize(torch.randn((batch, n, d), generator=gen, device="cuda:0"), dim=2)
    b = torch.nn.functional.normalize(torch.randn((batch, m, d), generator=gen, device="cuda:0"), dim=2)
    k = min(n, m) // 2
    b[:, :k] = torch.nn.functional.normalize(a[:, :k] + 0.3 * b[:, :k], dim=2)
    if two_steps:
        same(a, b, compute, **kw)
    else:
        fnn.fnn_trace_begin(64)
        fnn.fnn_mutual_dense(a, b, compute, **kw)
        torch.cuda.synchronize()
        assert "dense_select_kernel" not in [name for name, _ in fnn.fnn_trace_end(64)]
