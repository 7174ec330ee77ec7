"""What the matching path is timed on: calls that a user of libfnn makes, over the range of their sizes and options.

Sizes are those of the benchmark's configurations (64x48, 512x384 alone and in batches of 16, 1024x768; 24 channels,
every 8th pixel a seed, at most ten iterations) and generic ones around them.  The maps are what a dense matching head
emits: unit rows (raw rows where the call normalises them itself), image 2 = image 1 seen through a random homography,
with noise -- the benchmark's generator, on the GPU.  ``grain`` is the size in pixels of a map's features: 1 is that
generator as it stands (every pixel on its own), 4 gives maps in which neighbouring pixels resemble each other, as
those of a trained head do.
"""
import math

import torch

import paper_2503_10017_amd as fnn

STORAGE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ELEMENT = {"f32": 4, "f16": 2, "bf16": 2}

# width and height of the two images, pairs in the call, channels, format of the caller's maps and of the products
BASE = {"op": "reciprocal", "w1": 512, "h1": 384, "w2": 512, "h2": 384, "batch": 1, "d": 24, "maps": "f32", "compute": "f16",
        "step": 8, "max_iter": 10, "option": "", "grain": 1}


def _case(name, **kw):
    return {"name": name, **BASE, **kw}


def listed():
    return [
        # thumbnails, a preview or a unit test of a pipeline: launches and latency only
        _case("reciprocal_tiny", w1=64, h1=48, w2=64, h2=48),
        # one pair at a time, as an online localiser or tracker matches: the paper's latency figure
        _case("reciprocal_one", grain=4),
        # the throughput case: the pairs of a scene graph, matched 16 to a call
        _case("reciprocal_batch", batch=16),
        # one pair of large images
        _case("reciprocal_large", w1=1024, h1=768, w2=1024, h2=768, compute="bf16"),
        # raw head outputs of two cameras of different, ragged size, a few pairs, normalised by the call
        _case("reciprocal_raw_ragged", w1=517, h1=389, w2=433, h2=301, batch=4, compute="bf16", option="normalize", grain=4),
        # fp32-grade matching for a reconstruction: two-term fp16 products, and fp32 products
        _case("reciprocal_split", batch=4, option="split"),
        _case("reciprocal_f32", batch=2, compute="f32", step=16),
        # descriptors that are not unit rows, ranked by distance; maps stored as fp16
        _case("reciprocal_l2", batch=2, maps="f16", option="l2"),
        # one-directional searches: a seed grid in every pair of a batch, and a flow field with every pixel a query
        _case("nearest_batch", op="nearest", batch=16, maps="f16"),
        _case("nearest_every_pixel", op="nearest", step=1, grain=4),
        # the exhaustive match set of one pair, at the usual and at the large size
        _case("dense_one", op="dense"),
        _case("dense_large", op="dense", w1=1024, h1=768, w2=1024, h2=768, compute="bf16", grain=4),
    ]


def _queries(case):
    """Queries or seeds of one pair: the grid of every step-th pixel in x and y."""
    return -(-case["w1"] // case["step"]) * -(-case["h1"] // case["step"])


def _products(case):
    """Scores of the call's first (and, for a walk, second) search or of its dense sweep, times what one costs in fp16."""
    n, m = case["w1"] * case["h1"], case["w2"] * case["h2"]
    rows = n if case["op"] == "dense" else _queries(case) * (2 if case["op"] == "reciprocal" else 1)
    price = 6.0 if case["compute"] == "f32" else (2.5 if case["option"] == "split" else 1.0)
    return case["batch"] * rows * m * price


def draw(rng):
    def size(low, high):
        return round(math.exp(rng.uniform(math.log(low), math.log(high))))

    most = _products({**BASE, "op": "dense", "w1": 1024, "h1": 768, "w2": 1024, "h2": 768})
    while True:
        case = dict(BASE)
        case["op"] = rng.choice(["reciprocal", "reciprocal", "nearest", "dense"])
        case["w1"], case["h1"] = size(64, 1024), size(48, 768)
        if rng.random() < 0.5:  # two images of one camera, or of two
            case["w2"], case["h2"] = case["w1"], case["h1"]
        else:
            case["w2"], case["h2"] = size(64, 1024), size(48, 768)
        case["batch"] = rng.choice([1, 1, 2, 4, 16, rng.randint(1, 32)])
        case["d"] = rng.choice([24, 24, 24, 16, 32, rng.randint(4, 31)])
        case["compute"] = rng.choice(["f16", "f16", "bf16", "f32"])
        case["maps"] = rng.choice(["f32", "f32", case["compute"]])
        case["option"] = rng.choice(["", "", "", "normalize", "l2", "split"])
        if case["option"] == "split":
            case["compute"], case["maps"] = "f16", "f32"
        if case["option"] == "l2":
            case["d"] = min(case["d"], 28)
        case["step"] = 1 if case["op"] == "dense" else rng.choice([4, 8, 8, 16] + ([1] if case["op"] == "nearest" else []))
        case["max_iter"] = rng.choice([10, 10, 5, 2])
        case["grain"] = rng.choice([1, 4])
        n, m = case["w1"] * case["h1"], case["w2"] * case["h2"]
        if _products(case) <= most and case["batch"] * (n + m) <= 16 * 2 * 512 * 384:
            return case


def _pair(case, gen, dev):
    """Two maps as the benchmark's generator makes them (unit rows, fp32), image 2 of another size if the case says so."""
    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev)

    w1, h1, w2, h2, d, grain = (case[k] for k in ("w1", "h1", "w2", "h2", "d", "grain"))

    def field(h, w):
        if grain == 1:
            return normal(1, d, h, w)
        coarse = normal(1, d, -(-h // grain) + 1, -(-w // grain) + 1)
        return torch.nn.functional.interpolate(coarse, size=(h, w), mode="bilinear", align_corners=True)

    one = torch.nn.functional.normalize(field(h1, w1), dim=1)
    # the four corners of image 2 land within 15 % of image 1's corners: the homography through those points
    corner = torch.tensor([[-1.0, -1.0], [1.0, -1.0], [1.0, 1.0], [-1.0, 1.0]], dtype=torch.float64)
    jitter = torch.rand((4, 2), generator=gen, device=dev).cpu().double() * 0.6 - 0.3
    rows, right = [], []
    for (x, y), (u, v) in zip(corner.tolist(), (corner + jitter).tolist()):
        rows += [[x, y, 1, 0, 0, 0, -u * x, -u * y], [0, 0, 0, x, y, 1, -v * x, -v * y]]
        right += [u, v]
    hom = torch.linalg.solve(torch.tensor(rows, dtype=torch.float64), torch.tensor(right, dtype=torch.float64))
    hom = torch.cat([hom, torch.ones(1, dtype=torch.float64)]).reshape(3, 3).to(dev, torch.float32)
    ys, xs = torch.meshgrid(torch.linspace(-1, 1, h2, device=dev), torch.linspace(-1, 1, w2, device=dev), indexing="ij")
    at = torch.stack([xs, ys, torch.ones_like(xs)], dim=-1) @ hom.T
    at = at[..., :2] / at[..., 2:]
    seen = torch.nn.functional.grid_sample(one, at[None], mode="bilinear", align_corners=True)
    inside = (at.abs() <= 1).all(dim=-1)
    two = torch.where(inside, seen, field(h2, w2)) + 0.1 * normal(1, d, h2, w2)
    two = torch.nn.functional.normalize(two, dim=1)

    def rows_of(x):
        return x[0].permute(1, 2, 0).reshape(-1, d)

    return rows_of(one), rows_of(two)


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    n, m = case["w1"] * case["h1"], case["w2"] * case["h2"]
    kind = STORAGE[case["maps"]]
    d1 = torch.empty((case["batch"], n, case["d"]), dtype=kind, device=dev)
    d2 = torch.empty((case["batch"], m, case["d"]), dtype=kind, device=dev)
    for b in range(case["batch"]):
        one, two = _pair(case, gen, dev)
        if case["option"] in ("normalize", "l2"):  # raw head outputs, whose lengths vary from pixel to pixel
            spread = 0.1 if case["option"] == "l2" else 0.5
            one = one * torch.exp(spread * torch.randn((n, 1), generator=gen, device=dev))
            two = two * torch.exp(spread * torch.randn((m, 1), generator=gen, device=dev))
        d1[b], d2[b] = one, two
    state = {"case": dict(case), "d1": d1, "d2": d2}
    nq = 0 if case["op"] == "dense" else _queries(case)
    flags = {"normalize": case["option"] == "normalize", "l2": case["option"] == "l2", "split": case["option"] == "split"}
    if nq and (case["op"] == "reciprocal" or case["step"] > 1):
        grid = (torch.arange(0, case["h1"], case["step"], device=dev)[:, None] * case["w1"]
                + torch.arange(0, case["w1"], case["step"], device=dev)[None, :]).reshape(-1)
        state["seeds"] = grid.to(torch.int32)[None].repeat(case["batch"], 1)
    # what a serving program allocates once: the workspace and the result arrays
    need = fnn.fnn_workspace_bytes_opts(case["batch"], n, m, case["d"], nq, case["compute"], case["max_iter"], **flags)
    state["workspace"] = torch.empty(need, dtype=torch.uint8, device=dev)

    def ints(*shape):
        return torch.empty((case["batch"],) + shape, dtype=torch.int32, device=dev)

    def floats(*shape):
        return torch.empty((case["batch"],) + shape, dtype=torch.float32, device=dev)

    if case["op"] == "reciprocal":
        state["out"] = {"seed_i": ints(nq), "seed_j": ints(nq), "seed_iter": ints(nq), "pairs": ints(nq, 2), "n_pairs": ints()}
    elif case["op"] == "nearest":
        state["out"] = (ints(nq), floats(nq))
    else:
        state["out"] = {"nn12": ints(n), "s12": floats(n), "nn21": ints(m), "s21": floats(m), "pairs": ints(min(n, m), 2),
                        "n_pairs": ints()}
    return state


def run(state):
    case, out = state["case"], state["out"]
    kw = {"compute": case["compute"], "workspace": state["workspace"]}
    if case["option"]:
        kw[case["option"]] = True
    if case["op"] == "reciprocal":
        return fnn.fnn_reciprocal(state["d1"], state["d2"], state["seeds"], case["max_iter"], out=out, **kw)
    if case["op"] == "nearest":
        return fnn.fnn_nearest(state["d1"], state["d2"], q_idx=state.get("seeds"), out_idx=out[0], out_score=out[1], **kw)
    return fnn.fnn_mutual_dense(state["d1"], state["d2"], out=out, **kw)


def work(case):
    """Both maps read once, the seeds read and the results written; 2 d operations for every score of the searches
    that no seed can be spared (a walk's first search out and back: how many are live later depends on the data)."""
    n, m, batch, d = case["w1"] * case["h1"], case["w2"] * case["h2"], case["batch"], case["d"]
    maps = (n + m) * d * ELEMENT[case["maps"]]
    if case["op"] == "dense":
        return {"bytes": batch * (maps + 8 * (n + m) + 8 * min(n, m)), "flops": 2.0 * d * batch * n * m}
    nq = _queries(case)
    if case["op"] == "nearest":
        return {"bytes": batch * (maps + 4 * nq + 8 * nq), "flops": 2.0 * d * batch * nq * m}
    return {"bytes": batch * (maps + 4 * nq + 20 * nq), "flops": 2.0 * d * batch * nq * (n + m)}


def tolerance(case):
    """Indices are whole numbers: products of 16-bit values are exact in fp32 and ties go to the lowest index, so another
    order of the fp32 sums moves an index only where two scores lie within about 1e-7 of each other.  One such flip shifts
    the sorted match list behind it, so no share of differing values describes it: indices are held exactly, on inputs
    where the call's own runs agree.  Scores: at most 96 additions in fp32."""
    if case["op"] == "reciprocal":
        return "exact"
    return {"rel": 1e-6, "max": 1e-5}
