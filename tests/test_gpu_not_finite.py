"""Maps whose scores are not numbers: the results are unspecified, but every index that comes back -- and every
index that the iteration feeds into its next search, its pixel bitmap and its pair list -- lies inside the
maps.  The sizes take each route of the iteration: one workgroup per pair, the launch sequence with the final sort
in LDS, and the staged first searches."""
import numpy as np
import pytest
import torch

import paper_2503_10017_amd as fnn
from gpu_helpers import dev, exact_maps, host

pytestmark = pytest.mark.gpu


def spoil(x, which, value):
    x = x.copy()
    if which == "all":
        x[:] = value
    elif which == "tail":            # the last, partial tile of the map
        x[-(x.shape[0] % 32 or 32):] = value
    else:                            # scattered rows
        x[::7] = value
    return x


@pytest.mark.parametrize("which", ["all", "tail", "some"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("batch,n,m,n_seeds,first", [(4, 70, 45, 40, ("recip_walk_kernel", 0)), (4, 3000, 2977, 600, ("search_kernel", 1)),
                                                     (32, 13000, 12345, 1600, ("search_kernel", 103))])
def test_indices_stay_inside_the_maps(which, value, batch, n, m, n_seeds, first):
    a, b = exact_maps(n, n, m, 24)
    ta, tb = dev(spoil(a, which, value)), dev(spoil(b, which, value))
    seeds = dev(np.arange(n_seeds, dtype=np.int32) * (n // n_seeds))[None].repeat(batch, 1)
    fnn.fnn_trace_begin(128)
    out = fnn.fnn_reciprocal([ta] * batch, [tb] * batch, seeds, max_iter=6, compute="f16")
    torch.cuda.synchronize()
    searches = [(name, detail) for name, _, detail in fnn.fnn_trace_end(128, details=True) if name != "prep_kernel"]
    assert searches[0] == first
    idx, _ = fnn.fnn_nearest([ta] * batch, [tb] * batch, q_idx=seeds, compute="f16")
    torch.cuda.synchronize()
    out = {k: host(v) for k, v in out.items()}
    for found, size in ((out["seed_i"], n), (out["seed_j"], m), (host(idx), m)):
        assert found.min() >= 0 and found.max() < size
    for p, count in enumerate(out["n_pairs"]):
        assert 0 <= count <= n_seeds
        listed = out["pairs"][p, :count]
        assert (listed >= 0).all() and (listed[:, 0] < n).all() and (listed[:, 1] < m).all()
