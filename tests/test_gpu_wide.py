"""Assignment and update at the widths and cluster counts of the wide kernels (kmeans_wide.hip) and the sorted update
in column slabs, at the sizes where their tiles and dispatch turn over, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from parity import CENTROID_RTOL, DEV, Kmeans, centroid_rel_err, centroids_used, label_mismatches, to_np32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,k,dtype", [
    (1, 129, 1, torch.float32),            # one row
    (15, 300, 15, torch.float16),          # part of a point tile, k == n
    (2500, 5, 3, torch.bfloat16),          # less than one K-step, odd width
    (2049, 132, 17, torch.float32),        # two centroid tiles, ragged last K-step
    (2047, 160, 33, torch.float16),        # three tiles, whole K-steps
    (32_767, 257, 48, torch.bfloat16),     # last size of the small workgroups ...
    (32_768, 131, 49, torch.float32),      # ... first of the large ones
    (131_071, 67, 16, torch.float32),      # last size with 16 points per wave ...
    (131_072, 67, 20, torch.float16),      # ... first with 64
    (9_001, 1024, 64, torch.float32),      # the widest row: records pass through LDS in panels
    (9_001, 392, 64, torch.float32),       # one K-step more than a panel holds
    (3_003, 96, 65, torch.bfloat16),       # a second block of centroids with one real centroid
    (12_000, 129, 130, torch.float32),     # two column slabs in the sorted update, segments in parts
    (2_000, 700, 300, torch.float16),      # six slabs, whole segments
])
def test_wide_lockstep(n, d, k, dtype):
    bf16 = dtype == torch.bfloat16
    g = torch.Generator().manual_seed(n + d)
    comps = max(2, min(k, 40))
    x = 2.0 * torch.randn(comps, d, generator=g)[torch.randint(0, comps, (n,), generator=g)] + torch.randn(n, d, generator=g)
    unit = 4 if dtype == torch.float32 else 8
    padded = torch.full((n, (d + unit - 1) // unit * unit + unit), float("nan"), dtype=dtype)   # never read as data
    padded[:, :d] = x.clamp_(min=0).to(dtype)
    X = padded.to(DEV)[:, :d]
    X32 = to_np32(X)
    rng = np.random.default_rng(n)
    C0 = X32[oracle.init_indices(n, n, k)].astype(np.float64) + 0.01 * rng.normal(size=(k, d))
    C0 = C0.astype(np.float32).astype(np.float64)
    used = centroids_used(C0, bf16)

    got, d2, obj = Kmeans(X, k).set_centroids(C0).assign()
    want, best, _, obj_or = oracle.assign(X32, used)
    differing, unexcused = label_mismatches(X32, used, got, want, best)
    assert unexcused == 0, f"{unexcused} of {differing} differing labels are not near-ties"
    terms = (X32.astype(np.float64) ** 2).sum(axis=1) + (used ** 2).sum(axis=1)[got]
    assert np.all(np.abs(d2 - best) <= 1e-5 * terms)      # the size of the terms that the expanded form cancels
    # the objective: what the terms cancel to, each carrying an fp32 rounding per K-step of 32 columns and a few more
    assert abs(obj - obj_or) <= 1e-6 * obj_or + (-(-d // 32) + 4) * 2.0**-24 * terms.sum()

    labels = rng.integers(0, k, size=n).astype(np.int32)
    if k >= 3:
        labels[labels == 1] = 0                            # an empty cluster keeps its centroid
    labels[::97] = -1 if n > 97 else labels[::97]           # rows of no cluster
    keep = labels >= 0
    C_or, counts_or, _ = oracle.update(X32[keep], labels[keep], C0)
    C_got, counts = Kmeans(X, k).update(labels, C0.astype(np.float32))
    np.testing.assert_array_equal(counts, counts_or)
    assert centroid_rel_err(C_got, C_or) <= CENTROID_RTOL


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,d,k", [(3_001, 132, 20), (140_000, 70, 49)])
def test_wide_infinities_stay_in_their_cluster(n, d, k, dtype):
    g = torch.Generator().manual_seed(n)
    unit = 4 if dtype == torch.float32 else 8
    padded = torch.full((n, (d + unit - 1) // unit * unit), float("nan"), dtype=dtype)
    padded[:, :d] = torch.randn(n, d, generator=g).to(dtype)
    C0 = torch.randn(k, d, generator=g).to(torch.bfloat16).float().numpy()
    clean, clean_d2, _ = Kmeans(padded.to(DEV)[:, :d], k).set_centroids(C0).assign()
    plants = [(5, 3, float("inf")), (40, d - 1, float("-inf")), (n - 1, 0, float("nan"))]
    for row, col, value in plants:
        padded[row, col] = value
    X = padded.to(DEV)[:, :d]
    got, d2, _ = Kmeans(X, k).set_centroids(C0).assign()
    odd = np.array([row for row, _, _ in plants])
    rest = np.delete(np.arange(n), odd)
    np.testing.assert_array_equal(got[rest], clean[rest])
    np.testing.assert_array_equal(d2[rest], clean_d2[rest])
    assert got[5] == np.nonzero(C0[:, 3] > 0)[0][0] and got[40] == np.nonzero(C0[:, d - 1] < 0)[0][0] and got[n - 1] == 0

    labels = np.random.default_rng(n).integers(0, k, size=n).astype(np.int32)
    labels[odd] = [1, 1, 2]
    C_or, counts_or, _ = oracle.update(to_np32(X), labels, C0.astype(np.float64))
    C_got, counts = Kmeans(X, k).update(labels, C0)
    np.testing.assert_array_equal(counts, counts_or)
    finite = np.isfinite(C_or)
    assert finite.sum() == k * d - 3
    np.testing.assert_array_equal(np.isfinite(C_got), finite)
    assert C_got[1, 3] == np.inf and C_got[1, d - 1] == -np.inf and np.isnan(C_got[2, 0])
    assert np.abs(C_got[finite] - C_or[finite]).max() <= CENTROID_RTOL * np.abs(C_or[finite]).max()
