"""The prepare step with options that need a whole row (FNN_FLAG_NORMALIZE, FNN_FLAG_L2, FNN_FLAG_SPLIT).  Many rows are
staged through LDS in runs of 256, copied whole where the map is 16-byte aligned and its rows lie close
together, element by element otherwise; few rows are prepared element by element or one per thread.  How
the caller stores a map must not change a single bit of the result: contiguous, strided and misaligned
storage of the same values are compared, at the edges of a run and -- fnn_mutual_dense, whose image 1 is
stored in another order -- of a super-block of 4096 pixels; and the exactly representable values of L2 and
SPLIT against the oracle.  Normalised rows are compared channel by channel with the oracle's, on Gaussian
rows whose sums round at every step (the header's exception, the norms of aligned fp32 rows, is held to
its bound).  Squared lengths likewise, against 64 bits."""
import hashlib

import numpy as np
import pytest
import torch

import oracle
import paper_2503_10017_amd as fnn
from gpu_helpers import dev, exact_maps, host

pytestmark = pytest.mark.gpu


def stored(x, dtype, stride, offset):
    """The rows of x, `stride` elements apart, the first one `offset` elements into its allocation."""
    n, d = x.shape
    flat = torch.full((offset + n * stride + 8,), 3.0, dtype=dtype, device="cuda:0")   # junk between the rows
    view = flat[offset:offset + n * stride].view(n, stride)[:, :d]
    view.copy_(x)
    return view


@pytest.mark.parametrize("option,compute,dtype", [("normalize", "f16", torch.float16), ("normalize", "bf16", torch.bfloat16),
                                                  ("normalize", "f32", torch.float16), ("l2", "f16", torch.float16),
                                                  ("l2", "bf16", torch.float32), ("l2", "f32", torch.float32),
                                                  ("split", "f16", torch.float32)])
@pytest.mark.parametrize("n,m,d", [(255, 257, 24), (256, 33, 17), (4097, 513, 8), (1, 4095, 5), (300, 290, 28)])
@pytest.mark.parametrize("batch", [1, 64])       # few rows and many: more than 32768 where n + m is 513 or more
def test_storage_does_not_change_the_result(option, compute, dtype, n, m, d, batch):
    a, b = exact_maps(n + m + d, n, m, d)
    ta, tb = dev(a).to(dtype), dev(b).to(dtype)
    want = dense = None
    for stride, offset in ((d, 0), (d + 5, 0), (d, 1), (d + 1, 3), (2 * d, 0), (3 * d + 1, 2)):
        sa, sb = stored(ta, dtype, stride, offset), stored(tb, dtype, stride, offset)
        sa, sb = [sa] * batch, [sb] * batch
        idx, score = (host(x) for x in fnn.fnn_nearest(sa, sb, compute=compute, **{option: True}))
        out = {k: host(v) for k, v in fnn.fnn_mutual_dense(sa, sb, compute=compute, **{option: True}).items()}
        if want is None:
            want, dense = (idx[0], score[0]), {k: v[0] for k, v in out.items()}
            if option != "normalize":
                ref = oracle.nearest_l2(a, b) if option == "l2" else oracle.nearest(a, b)
                assert np.array_equal(idx[0], ref[0])
                assert np.array_equal(-2.0 * score[0] if option == "l2" else score[0], ref[1])
        for p in range(batch):
            assert np.array_equal(idx[p], want[0]) and np.array_equal(score[p], want[1]), (stride, offset)
            for key in ("nn12", "s12", "nn21", "s21", "n_pairs", "pairs"):
                assert np.array_equal(out[key][p], dense[key]), (key, stride, offset)


def lengthy_maps(seed, n, d):
    """Gaussian rows of lengths between 0.05 and 20, one of them zero: sums of squares that round at every step."""
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((n, d)) * rng.uniform(0.05, 20.0, size=(n, 1))).astype(np.float32)
    x[n // 2] = 0.0
    return x


def prepared(x, compute, **kw):
    """The channels of every row as the prepare step leaves them: their products with the unit rows, one pair each."""
    unit = torch.eye(x.shape[1], dtype=x.dtype, device=x.device)
    score = fnn.fnn_nearest([x] * x.shape[1], [unit[k:k + 1] for k in range(x.shape[1])], compute=compute, **kw)[1]
    return host(score).T


@pytest.mark.parametrize("compute,kw", [("f32", {}), ("f16", {}), ("bf16", {}), ("f16", {"split": True})])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n,d", [(1030, 5), (30000, 5), (1030, 8), (20000, 8), (500, 16), (2100, 16), (1030, 17), (2000, 17), (200, 24), (1030, 24),
                                 (1500, 24), (200, 32), (1100, 32)])        # few rows and many (n rows in d pairs)
def test_normalised_rows_are_the_defined_ones_bit_for_bit(compute, kw, dtype, n, d):
    x = dev(lengthy_maps(d, n, d)).to(dtype)
    y = oracle.normalize(host(x.float()))
    want = {"f32": y, "f16": sum(oracle.split_fp16(y)) if kw else oracle.round_fp16(y), "bf16": oracle.round_bf16(y)}[compute]
    for stride, offset in ((d, 0), (d, 1), (d + 4, 0), (d + 1, 3), (3 * d + 1, 2)):
        got = prepared(stored(x, dtype, stride, offset), compute, normalize=True, **kw)
        if dtype == torch.float32 and d % 8 == 0 and stride % 4 == 0 and offset % 4 == 0 and not kw:
            # the header's exception.  Both sums of d rounded steps (and one rounded product) lie within (2 d + 1) 2^-24
            # of each other, their roots within half of that and one last place (2^-23), and both divisions round
            # (2^-24 each); in a 16-bit format that may carry a value over to its neighbour
            far = np.abs(got - want) > np.abs(want) * {"f32": (d + 4.5) * 2.0**-24, "f16": 2.0**-10, "bf16": 2.0**-7}[compute]
            assert not far.any() and (got == want).mean() > (0.5 if compute == "f32" else 0.999), (stride, offset)
        else:
            assert np.array_equal(got, want), (stride, offset)


@pytest.mark.parametrize("n", [1030, 40000])
@pytest.mark.parametrize("d", [5, 8, 16, 24, 28])
def test_squared_lengths_in_fp32(n, d):
    x = dev(lengthy_maps(d, n, d))
    want = -0.5 * (host(x).astype(np.float64) ** 2).sum(axis=1)
    zero = torch.zeros((1, d), device=x.device)
    for stride, offset in ((d, 0), (d, 1), (d + 4, 0), (d + 1, 3)):
        # against a zero row the score is the length's own term: d squares and d sums, each rounded at most once
        score = host(fnn.fnn_nearest(stored(x, torch.float32, stride, offset), zero, compute="f32", l2=True)[1])[0]
        assert (np.abs(score - want) <= np.abs(want) * 2 * d * 2.0**-24).all(), (stride, offset)


@pytest.mark.parametrize("d,digest", [(8, "f13ff72d1ab3a37a"), (16, "2098f6af11ee0c18"), (24, "cdf7abc18f34556b"), (32, "8875f89e7abb8ea3")])
def test_last_places_of_aligned_rows_stay(d, digest):
    """The header's exception: the second square is rounded, the others are fused steps on top of it, and the root is the hardware's.  Another order of the sum changes the
    last place of some rows and passes every bound, so the scores of these rows are pinned by their bits."""
    x = (np.random.default_rng(d).integers(-999, 1000, size=(20000, d)) / np.float32(997)).astype(np.float32)
    one_hot = np.eye(d, dtype=np.float32)   # length 1 exactly: the score is the largest channel of the normalised row
    idx, score = (host(y)[0] for y in fnn.fnn_nearest(dev(x)[None], dev(one_hot)[None], compute="f32", normalize=True))
    assert np.array_equal(idx, x.argmax(axis=1))
    assert hashlib.sha1(score.tobytes()).hexdigest()[:16] == digest
