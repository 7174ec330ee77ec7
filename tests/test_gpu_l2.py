"""GPU parity of the squared-distance dist_func (FNN_FLAG_L2) against the oracle, through the C ABI.

The library reports score = -1/2 |a - b|^2 (larger is better); the oracle reports |a - b|^2.
On exactly representable maps (entries k/8) every term is exact in all three compute formats, so
indices and -2 * score must match the oracle bit for bit.  On raw Gaussian maps the comparison is
made against the oracle on inputs rounded like the library rounds them; then the two differ by
fp32 rounding only: the library sums <a,b> - |a|^2/2 - |b|^2/2 (about 30 terms, partial sums up to
(|a| + |b|)^2 / 2 < 128 for these maps, so at most about 32 * 2^-24 * 128 = 2.4e-4 in the score),
the oracle sums 24 squared differences.  Hence: indices equal wherever the oracle's distance gap
exceeds 2e-3, distances within 1e-3.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
import synth_inputs as synth
from gpu_helpers import ROUNDERS, check_reciprocal_exact, dev, exact_maps, host, unit_maps

pytestmark = pytest.mark.gpu

L2_GAP = 2e-3
L2_TOL = 1e-3


def raw_maps(seed, n, m, d):
    """Un-normalised N(0,1) descriptors; the second map holds noisy copies of rows of the first."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((n, d)).astype(np.float32)
    b = (a[rng.integers(0, n, size=m)] + 0.1 * rng.standard_normal((m, d))).astype(np.float32)
    return a, b


@pytest.mark.parametrize("compute", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n,m,d", [(1000, 3001, 24), (77, 4100, 12), (300, 300, 5), (64, 999, 28)])
def test_nearest_l2_exact_maps_bit_exact(compute, n, m, d):
    a, b = exact_maps(100 + d, n, m, d)
    gi, gs = fnn.fnn_nearest(dev(a), dev(b), compute=compute, l2=True)
    torch.cuda.synchronize()
    ri, rbest, _ = oracle.nearest_l2(a, b)
    assert np.array_equal(host(gi)[0], ri)
    assert np.array_equal(-2.0 * host(gs)[0], rbest)
    # and the dot-product answer is a different one on these maps
    di, _ = fnn.fnn_nearest(dev(a), dev(b), compute=compute)
    assert not np.array_equal(host(di)[0], ri)


def test_nearest_l2_widest_rows_and_limits():
    a, b = exact_maps(7, 200, 500, 30)
    gi, gs = fnn.fnn_nearest(dev(a), dev(b), compute="f32", l2=True)
    ri, rbest, _ = oracle.nearest_l2(a, b)
    assert np.array_equal(host(gi)[0], ri) and np.array_equal(-2.0 * host(gs)[0], rbest)
    with pytest.raises(fnn.FnnError) as err:
        fnn.fnn_nearest(dev(a), dev(b), compute="f16", l2=True)     # 30 + 4 channels do not fit
    assert err.value.status == 2
    a, b = exact_maps(8, 64, 64, 31)
    with pytest.raises(fnn.FnnError) as err:
        fnn.fnn_nearest(dev(a), dev(b), compute="f32", l2=True)     # 31 + 2 channels do not fit
    assert err.value.status == 2


@pytest.mark.parametrize("compute", ["f16", "bf16", "f32"])
def test_nearest_l2_raw_gaussian_maps(compute):
    a, b = raw_maps(5, 3000, 20000, 24)
    rng = np.random.default_rng(6)
    q = rng.integers(0, a.shape[0], size=1500).astype(np.int32)
    gi, gs = fnn.fnn_nearest(dev(a), dev(b), q_idx=dev(q)[None], compute=compute, l2=True)
    torch.cuda.synchronize()
    rnd = ROUNDERS[compute]
    ri, rbest, rsecond = oracle.nearest_l2(rnd(a)[q], rnd(b))
    gi, gd = host(gi)[0], -2.0 * host(gs)[0]
    clear = (rsecond - rbest) > L2_GAP
    assert clear.mean() > 0.9
    assert np.array_equal(gi[clear], ri[clear])
    assert np.abs(gd - rbest).max() <= L2_TOL
    # the maps are far from unit norm: the dot product picks other neighbours
    di, _ = fnn.fnn_nearest(dev(a), dev(b), q_idx=dev(q)[None], compute=compute)
    assert (host(di)[0] != ri).mean() > 0.2


@pytest.mark.parametrize("compute", ["f16", "f32"])
def test_l2_on_unit_maps_agrees_with_the_dot_product_mode(compute):
    a, b = unit_maps(11, 2000, 9000, 24)
    li, ls = fnn.fnn_nearest(dev(a), dev(b), compute=compute, l2=True)
    di, ds = fnn.fnn_nearest(dev(a), dev(b), compute=compute)
    torch.cuda.synchronize()
    rnd = ROUNDERS[compute]
    _, rbest, rsecond = oracle.nearest(rnd(a), rnd(b))
    clear = (rbest - rsecond) > 1e-3          # rounded vectors are only approximately unit-norm
    assert clear.mean() > 0.8
    assert np.array_equal(host(li)[0][clear], host(di)[0][clear])
    # |a - b|^2 = |a|^2 + |b|^2 - 2<a,b>, all three from the rounded vectors
    ra, rb = rnd(a).astype(np.float64), rnd(b).astype(np.float64)
    j = host(li)[0]
    want = ((ra - rb[j]) ** 2).sum(axis=1)
    assert np.abs(-2.0 * host(ls)[0] - want).max() <= 1e-5


@pytest.mark.parametrize("compute", ["f16", "bf16", "f32"])
def test_reciprocal_and_dense_l2_exact_maps(compute):
    w, h, d = 40, 28, 24
    d1, d2 = synth.exact_pair(77, w, h, d)
    seeds = synth.grid_seeds(w, h, 4)
    out = fnn.fnn_reciprocal(dev(d1), dev(d2), dev(seeds)[None], max_iter=10, compute=compute, l2=True)
    torch.cuda.synchronize()
    got = {k: host(v) for k, v in out.items()}
    ref = oracle.reciprocal(d1, d2, seeds, 10, metric="l2")
    check_reciprocal_exact(got, 0, ref)
    assert not np.array_equal(ref["seed_j"], oracle.reciprocal(d1, d2, seeds, 10)["seed_j"])

    dense = fnn.fnn_mutual_dense(dev(d1), dev(d2), compute=compute, l2=True)
    torch.cuda.synchronize()
    rd = oracle.mutual_dense(d1, d2, metric="l2")
    n_pairs = int(host(dense["n_pairs"])[0])
    assert np.array_equal(host(dense["nn12"])[0], rd["nn12"]) and np.array_equal(host(dense["nn21"])[0], rd["nn21"])
    assert np.array_equal(2.0 * host(dense["s12"])[0], rd["s12"]) and np.array_equal(2.0 * host(dense["s21"])[0], rd["s21"])
    assert np.array_equal(host(dense["pairs"])[0, :n_pairs], rd["pairs"])


def test_reciprocal_l2_raw_gaussian_batch():
    # two pairs in one call, ragged sizes, pinned-seed comparison on rounded inputs
    pairs = [raw_maps(40 + b, 48 * 36, 48 * 36, 24) for b in range(2)]
    seeds = synth.grid_seeds(48, 36, 4)
    out = fnn.fnn_reciprocal([dev(p[0]) for p in pairs], [dev(p[1]) for p in pairs],
                             dev(np.stack([seeds, seeds])), max_iter=10, compute="f16", l2=True)
    torch.cuda.synchronize()
    got = {k: host(v) for k, v in out.items()}
    for b, (d1, d2) in enumerate(pairs):
        ref = oracle.reciprocal(oracle.round_fp16(d1), oracle.round_fp16(d2), seeds, 10, metric="l2")
        pinned = ref["min_gap"] > L2_GAP
        assert pinned.mean() > 0.8
        for key in ("seed_i", "seed_j", "seed_iter"):
            assert np.array_equal(got[key][b][pinned], ref[key][pinned]), key
        n_pairs = int(got["n_pairs"][b])
        done = got["seed_iter"][b] >= 0
        want = np.unique(np.stack([got["seed_i"][b][done], got["seed_j"][b][done]], axis=1), axis=0)
        assert np.array_equal(got["pairs"][b, :n_pairs], want)


def test_normalize_then_l2():
    a, b = raw_maps(9, 1500, 6000, 24)
    gi, gs = fnn.fnn_nearest(dev(a), dev(b), compute="f16", normalize=True, l2=True)
    torch.cuda.synchronize()
    na, nb = oracle.round_fp16(oracle.normalize(a)), oracle.round_fp16(oracle.normalize(b))
    ri, rbest, rsecond = oracle.nearest_l2(na, nb)
    clear = (rsecond - rbest) > 1e-4
    assert clear.mean() > 0.9
    assert np.array_equal(host(gi)[0][clear], ri[clear])
    assert np.abs(-2.0 * host(gs)[0] - rbest).max() <= 1e-5


@pytest.mark.parametrize("storage", [torch.float32, torch.float16])
@pytest.mark.parametrize("n,m", [(60, 77), (2000, 2500)])     # one workgroup per pair, launch sequence
def test_rows_too_long_for_fp16_norm_terms(storage, n, m):
    """1/2 |x|^2 past 65504 does not fit one fp16 value: the remainder carries what it can, up to 131008, and longer
    rows are held there.  Whole numbers of at most 200: every term is exact in fp32, so the scores are known."""
    rng = np.random.default_rng(n)
    a, b = (np.rint(rng.uniform(-1, 1, size=(k, 24)) * np.linspace(20, 200, k)[:, None]) for k in (n, m))

    def term(x):
        t = -0.5 * (x * x).sum(axis=1)
        hi = np.maximum(t, -65504.0).astype(np.float16).astype(np.float64)
        return hi + np.maximum(t - hi, -65504.0).astype(np.float16).astype(np.float64)

    lengths = 0.5 * (a * a).sum(axis=1)
    assert (lengths < 65504).any() and (lengths > 131008).any() and ((lengths > 65504) & (lengths < 131008)).any()
    score = a @ b.T + term(a)[:, None] + term(b)[None]
    ta, tb = (dev(x.astype(np.float32)).to(storage) for x in (a, b))
    idx, best = fnn.fnn_nearest(ta, tb, compute="f16", l2=True)
    assert np.array_equal(host(idx)[0], score.argmax(axis=1)) and np.array_equal(host(best)[0], score.max(axis=1))
    seeds = np.arange(0, n, 3, dtype=np.int32)
    out = fnn.fnn_reciprocal(ta, tb, dev(seeds)[None], max_iter=10, compute="f16", l2=True)
    out = {k: host(v)[0] for k, v in out.items()}
    done = out["seed_iter"] >= 0
    assert done.any()
    assert np.array_equal(out["seed_j"], score.argmax(axis=1)[out["seed_i"]])
    assert np.array_equal(out["seed_i"][done], score.argmax(axis=0)[out["seed_j"][done]])
